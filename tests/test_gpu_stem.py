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


def sprinkle(x, g, every):
    """Infinities of both signs and NaN in place of one element in `every`, the corners of the first image among them."""
    import torch
    u = torch.rand(x.shape, generator=g, device="cuda") * every
    for i, v in enumerate((float("inf"), float("-inf"), float("nan"))):
        x[(u >= i / 3) & (u < (i + 1) / 3)] = v
    x[0, 0, 0, 0], x[0, -1, -1, -1], x[0, 0, -1, 0] = float("inf"), float("-inf"), float("inf")
    return x


@pytest.mark.parametrize("n,sp,c,k,f,stride,pad,off", [case for case in CASES if case[1] != (1, 2)] + [(1, (40, 52), 2, 64, 20, 2, 9, 0), (1, (9, 90), 4, 16, 1, 1, 0, 0)])
def test_forward_of_infinities_and_nan(n, sp, c, k, f, stride, pad, off):
    """They reach the outputs whose window contains them, and the others have the values that they have without them."""
    import torch
    import paper_1807_02037_amd as L
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k + f)
    osp = tuple((e + 2 * pad - f) // stride + 1 for e in sp)
    x = sprinkle(torch.randn((n,) + sp + (c,), generator=g, device="cuda"), g, 6 * f * f * c).to(torch.bfloat16)
    x = torch.empty(x.numel() + 8, dtype=torch.bfloat16, device="cuda")[off:off + x.numel()].view(x.shape).copy_(x)
    w = torch.randn((f, f, c, k), generator=g, device="cuda").to(torch.bfloat16)
    d = L.conv_desc(n, sp, c, k, (f, f), stride, pad, 0)
    ws = torch.empty(max(L.conv_workspace_bytes(d, L.abi.CONV_FWD), 256), dtype=torch.uint8, device="cuda")
    y = torch.empty((n,) + osp + (k,), dtype=torch.bfloat16, device="cuda")
    L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, y.data_ptr(), ws.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    xp, wd = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad)), w.double()
    ref = torch.zeros(y.shape, dtype=torch.float64, device="cuda")
    for r in range(f):
        for q in range(f):
            cut = xp[:, r:r + (osp[0] - 1) * stride + 1:stride, q:q + (osp[1] - 1) * stride + 1:stride]
            for e in range(c):                                  # element by element: a product of matrices may mix what is not finite
                ref += cut[..., e:e + 1] * wd[r, q, e]
    fin = torch.isfinite(ref)
    assert bool(fin.any()) and not bool(fin.all())
    yd = y.double()
    assert torch.equal(torch.nan_to_num(yd[~fin], 0.5, 1.0, -1.0), torch.nan_to_num(ref[~fin], 0.5, 1.0, -1.0))
    assert bool(((yd[fin] - ref[fin]).abs() <= 2.0 ** -8 * ref[fin].abs() + 1e-4).all())


@pytest.mark.parametrize("n,sp,c,k,f,stride,pad", [case[:7] for case in CASES if case[2] * case[5] == 6 and not case[7]] +
                         [(2, (48, 48), 3, 64, 7, 2, 3), (3, (33, 262), 3, 64, 7, 2, 3), (5, (70, 30), 3, 64, 3, 2, 1)])
def test_weight_gradient_of_infinities_and_nan(n, sp, c, k, f, stride, pad):
    """One pixel that is not finite, at the corners, edges and inside: it reaches the taps that read it, and the other entries have the
    values that they have without it."""
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k + f)
    h, w = sp
    osp = tuple((e + 2 * pad - f) // stride + 1 for e in sp)
    x = torch.randn((n,) + sp + (c,), generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn((n,) + osp + (k,), generator=g, device="cuda").to(torch.bfloat16)
    d = L.conv_desc(n, sp, c, k, (f, f), stride, pad, 0)
    ws = torch.empty(L.conv_workspace_bytes(d, A.CONV_WGRAD_BIAS), dtype=torch.uint8, device="cuda")
    dw, db = torch.empty((f, f, c, k), device="cuda"), torch.empty((k,), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    dyd = dy.double().cpu().reshape(-1, k)
    refb = dyd.sum(0)
    inf = float("inf")
    for a, r, q, v in [(0, 0, 0, inf), (n - 1, h - 1, w - 1, -inf), (0, h - 1, 0, float("nan")), (n - 1, 0, w - 1, inf), (0, h // 2, w - 2, inf), (0, max(h - 2, 0), w // 2, -inf),
                       (n - 1, h // 2, min(w // 2 + 1, w - 1), inf), (0, min(17, h - 1), min(33, w - 1), inf)]:
        xi = x.clone()
        xi[a, r, q, c - 1] = v
        L.conv_wgrad_bias(d, xi.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), ws.data_ptr(), s)
        torch.cuda.synchronize()
        xp = torch.nn.functional.pad(xi.double().cpu(), (0, 0, pad, pad, pad, pad))
        ref = torch.empty((f, f, c, k), dtype=torch.float64)
        for i in range(f):
            for j in range(f):
                cut = xp[:, i:i + (osp[0] - 1) * stride + 1:stride, j:j + (osp[1] - 1) * stride + 1:stride].reshape(-1, c)
                ref[i, j] = cut.t() @ dyd
        got, fin = dw.double().cpu(), torch.isfinite(ref)
        assert bool(fin.any())
        assert torch.equal(torch.nan_to_num(got[~fin], 0.5, 1.0, -1.0), torch.nan_to_num(ref[~fin], 0.5, 1.0, -1.0)), (a, r, q)
        assert float((got[fin] - ref[fin]).norm()) <= 2e-6 * float(ref[fin].norm()), (a, r, q)
        assert float((db.double().cpu() - refb).norm()) <= 2e-6 * float(refb.norm())


# extents, c, k, filter, stride, padding: two, three and four output rows of 64 channels that span more than 2^31 and 2^32 bytes
WIDE = [((4, 6000000), 2, 64, 3, 1, 1), ((5, 17000002), 1, 64, 3, 2, 1), ((4, 12000000), 2, 64, 3, 1, 1)]


@pytest.mark.parametrize("sp,c,k,f,stride,pad", WIDE)
def test_forward_on_rows_of_gigabytes(sp, c, k, f, stride, pad):
    """Every output row of images so wide that four of their rows leave 32-bit offsets, at the ends and in the middle."""
    import torch
    import paper_1807_02037_amd as L
    g = torch.Generator(device="cuda")
    g.manual_seed(sp[1])
    x = torch.empty((1,) + sp + (c,), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    w = torch.empty((f, f, c, k), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    oh, ow = [(e + 2 * pad - f) // stride + 1 for e in sp]
    assert oh * ow * k * 2 >= 1 << 31
    d = L.conv_desc(1, sp, c, k, (f, f), stride, pad, 0)
    ws = torch.empty(max(L.conv_workspace_bytes(d, L.abi.CONV_FWD), 256), dtype=torch.uint8, device="cuda")
    y = torch.full((oh, ow, k), float("nan"), dtype=torch.bfloat16, device="cuda")
    L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, y.data_ptr(), ws.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert not any(bool(torch.isnan(part).any()) for row in y for part in row.split(1 << 20))
    wd = w.double().cpu()
    for b in (0, 4194000, ow // 2, ow - 1500):
        e = min(ow, b + 1500)
        lo, hi = b * stride - pad, (e - 1) * stride - pad + f                    # input columns
        cols = x[0, :, max(lo, 0):min(hi, sp[1])].double().cpu()
        cols = torch.nn.functional.pad(cols, (0, 0, max(-lo, 0), max(hi - sp[1], 0), pad, pad))
        ref = torch.zeros((oh, e - b, k), dtype=torch.float64)
        for r in range(f):
            for q in range(f):
                ref += cols[r:r + (oh - 1) * stride + 1:stride, q:q + (e - b - 1) * stride + 1:stride] @ wd[r, q]
        assert bool(((y[:, b:e].double().cpu() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all()), b
