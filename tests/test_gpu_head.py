"""Weight gradient of class heads (pointwise, at most 8 outputs): fewer rows than lanes, rows that leave a remainder behind the
four taken at a time, one to 32 channel vectors.  Reference: float64 sums; bound: 2e-6 of the norm (fp32 sums of exact products)."""
import pytest

pytestmark = pytest.mark.gpu

CASES = [(1, (1, 1), 8, 8), (1, (5, 3), 256, 4), (1, (61, 67), 16, 8), (1, (37, 41), 64, 4), (3, (113, 97), 8, 2), (2, (9, 31, 33), 32, 3),
         (1, (40, 41, 43), 32, 8), (1, (33, 64, 65), 128, 4), (2, (50, 61), 64, 5), (1, (33, 35), 8, 1)]


@pytest.mark.parametrize("n,sp,c,k", CASES)
def test_weight_gradient(n, sp, c, k):
    import torch
    import paper_1807_02037_amd as L
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    x = torch.randn((n,) + sp + (c,), generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn((n,) + sp + (k,), generator=g, device="cuda").to(torch.bfloat16)
    d = L.conv_desc(n, sp, c, k, (1,) * len(sp), 1, 0, 0)
    ws = torch.full((L.conv_workspace_bytes(d, L.abi.CONV_WGRAD),), 255, dtype=torch.uint8, device="cuda")
    dw = torch.full((c, k), float("nan"), device="cuda")
    L.conv_wgrad(d, x.data_ptr(), dy.data_ptr(), dw.data_ptr(), ws.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ref = x.double().reshape(-1, c).t() @ dy.double().reshape(-1, k)
    assert float((dw.double() - ref).norm() / ref.norm()) <= 2e-6
