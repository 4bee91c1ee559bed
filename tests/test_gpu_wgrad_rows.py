"""Weight gradient of pointwise layers at the edges of the kernel's shapes: filters that fill no tile of each shape, fewer
positions than one round, a last round that some groups of waves do not take part in, strides, odd grids, several splits.
Reference: float64 sums of the GPU's own bf16 inputs; bound: 2e-6 of the norm (fp32 sums of at most 10^5 exact products)."""
import pytest

pytestmark = pytest.mark.gpu

# n, extents, c, k, stride
CASES = [
    (1, (3, 5), 64, 64, 1), (2, (33, 47), 56, 48, 1), (5, (40, 41), 64, 128, 1), (1, (64, 64), 128, 72, 1),
    (3, (31, 37), 128, 128, 1), (2, (50, 61), 256, 64, 1), (2, (29, 64), 64, 256, 1), (1, (20, 21), 328, 200, 1),
    (3, (17, 15), 64, 128, 2), (1, (9, 10, 11), 72, 136, 2), (2, (22, 23), 256, 512, 3), (40, (7, 7), 512, 256, 1),
]


@pytest.mark.parametrize("n,sp,c,k,stride", CASES)
def test_weight_and_bias_gradient(n, sp, c, k, stride):
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    osp = tuple((e - 1) // stride + 1 for e in sp)
    x = torch.randn((n,) + sp + (c,), generator=g, device="cuda").to(torch.bfloat16)
    dy = (torch.randn((n,) + osp + (k,), generator=g, device="cuda") + 0.5).to(torch.bfloat16)
    d = L.conv_desc(n, sp, c, k, (1,) * len(sp), stride, 0, 0)
    ws = torch.full((L.conv_workspace_bytes(d, A.CONV_WGRAD_BIAS),), 255, dtype=torch.uint8, device="cuda")
    dw, db, dw2 = torch.full((c, k), float("nan"), device="cuda"), torch.full((k,), float("nan"), device="cuda"), torch.full((c, k), float("nan"), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    L.conv_wgrad_bias(d, x.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), ws.data_ptr(), s)
    L.conv_wgrad(d, x.data_ptr(), dy.data_ptr(), dw2.data_ptr(), ws.data_ptr(), s)
    torch.cuda.synchronize()
    xs = x[(slice(None),) + (slice(None, None, stride),) * len(sp)].double().reshape(-1, c)
    dys = dy.double().reshape(-1, k)
    ref, refb = xs.t() @ dys, dys.sum(dim=0)
    assert float((dw.double() - ref).norm() / ref.norm()) <= 2e-6
    assert float((db.double() - refb).norm() / refb.norm()) <= 2e-6
    assert torch.equal(dw, dw2)
