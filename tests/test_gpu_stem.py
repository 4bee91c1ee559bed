"""First layers read straight from their staged input rows: forward where stride times channels is even, weight gradient where it is
six.  Rows wider than a tile, maps of one position, tiles cut by the last row and column, filters of one to eleven rows, every channel count,
paddings that put a run at odd and even offsets, output counts that fill no tile, and what stays with the kernels
for any alignment.  Reference: float64 from the bf16 inputs; forward one bf16 rounding (2^-8 of the value, fp32 sums of at most
300 products far below), weight gradients 2e-6 of the norm."""
import pytest

pytestmark = pytest.mark.gpu

# n, extents, c, k, filter, stride, padding, elements before the tensors' first
CASES = [
    (2, (30, 44), 3, 64, 7, 2, 3, 0), (1, (9, 8), 3, 64, 7, 2, 3, 0), (1, (1, 2), 3, 8, 3, 2, 1, 0), (1, (17, 300), 3, 40, 7, 2, 3, 0),
    (3, (33, 20), 3, 24, 3, 2, 1, 0), (2, (20, 26), 3, 56, 5, 2, 2, 0), (2, (12, 14), 3, 64, 7, 2, 0, 0), (1, (40, 52), 3, 64, 1, 2, 0, 0),
    (2, (13, 19), 4, 64, 3, 1, 1, 0), (1, (5, 260), 2, 8, 5, 1, 2, 0), (2, (16, 16), 2, 64, 3, 3, 1, 0), (1, (50, 70), 1, 8, 7, 6, 3, 0),
    (1, (34, 36), 1, 16, 11, 2, 5, 0), (2, (31, 34), 3, 40, 7, 2, 3, 1), (2, (22, 24), 3, 40, 7, 2, 3, 2),
]


@pytest.mark.parametrize("n,sp,c,k,f,stride,pad,off", CASES)
def test_forward_and_weight_gradient(n, sp, c, k, f, stride, pad, off):
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k + f)
    osp = tuple((e + 2 * pad - f) // stride + 1 for e in sp)

    def tensor(shape, mean):
        count = torch.Size(shape).numel()
        flat = torch.empty(count + 8, dtype=torch.bfloat16, device="cuda")
        return flat[off:off + count].view(shape).copy_(torch.randn(shape, generator=g, device="cuda") + mean)

    x, dy, w = tensor((n,) + sp + (c,), 0.0), tensor((n,) + osp + (k,), 0.5), tensor((f, f, c, k), 0.0)
    shift = torch.randn(k, generator=g, device="cuda")
    d = L.conv_desc(n, sp, c, k, (f, f), stride, pad, A.F_BIAS)
    need = [L.conv_workspace_bytes(d, which) for which in (A.CONV_FWD, A.CONV_WGRAD_BIAS)]
    ws = torch.full((max(need) + 4096,), 255, dtype=torch.uint8, device="cuda")
    y = torch.full((n,) + osp + (k,), float("nan"), dtype=torch.bfloat16, device="cuda")
    dw, db = torch.full((f, f, c, k), float("nan"), device="cuda"), torch.full((k,), float("nan"), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, shift.data_ptr(), None, y.data_ptr(), ws.data_ptr(), s)
    L.conv_wgrad_bias(d, x.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), ws.data_ptr(), s)
    torch.cuda.synchronize()
    assert bool((ws[max(need):] == 255).all())
    xp = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
    dyd = dy.double().reshape(-1, k)
    ref, refw = shift.double().expand((n,) + osp + (k,)).clone(), torch.empty((f, f, c, k), dtype=torch.float64, device="cuda")
    for r in range(f):
        for q in range(f):
            cut = xp[:, r:r + (osp[0] - 1) * stride + 1:stride, q:q + (osp[1] - 1) * stride + 1:stride]
            ref += (cut.reshape(-1, c) @ w[r, q].double()).view(ref.shape)
            refw[r, q] = cut.reshape(-1, c).t() @ dyd
    assert bool(((y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())
    assert float((dw.double() - refw).norm()) <= 2e-6 * float(refw.norm())
    assert float((db.double() - dyd.sum(0)).norm()) <= 2e-6 * float(dyd.sum(0).norm())
