"""Tensors that start anywhere in a caller's buffer: activations and gradients one element (2 bytes) past a vector boundary take
kernels that load through registers, and a bias gradient needs no more than a float's alignment.  Reference: the same call on
aligned tensors, whose kernels may add in another order: fp32 sums of a few hundred exact products each (2^-14 of the value
and of the root mean square), and for bf16 results one rounding each (2^-7 of the value together)."""
import pytest

pytestmark = pytest.mark.gpu

# n, extents, c, k, filter, stride, pad: pointwise, strided, few and many columns; 3x3 and 3x3x3; first layer; head
CASES = [(2, (19, 21), 64, 136, 1, 1, 0), (2, (19, 21), 128, 64, 1, 2, 0), (1, (9, 7, 8), 64, 64, 1, 1, 0), (2, (15, 14), 64, 72, 3, 1, 1),
         (1, (9, 10, 11), 24, 40, 3, 1, 1), (1, (9, 70), 3, 16, 3, 1, 1), (1, (17, 18), 32, 8, 1, 1, 0)]


@pytest.mark.parametrize("shift", [1, 4])
@pytest.mark.parametrize("n,sp,c,k,filt,stride,pad", CASES)
def test_tensors_between_vector_boundaries(n, sp, c, k, filt, stride, pad, shift):
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    nd = len(sp)
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    osp = tuple((e + 2 * pad - filt) // stride + 1 for e in sp)
    d = L.conv_desc(n, sp, c, k, (filt,) * nd, stride, pad, 0)
    s = torch.cuda.current_stream().cuda_stream
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
    base = {"x": rnd(n, *sp, c), "dy": rnd(n, *osp, k), "add": rnd(n, *sp, c), "mask": rnd(n, *sp, c)}
    w = rnd(*(filt,) * nd, c, k)
    ws = torch.empty(max(L.conv_workspace_bytes(d, q) for q in range(4)), dtype=torch.uint8, device="cuda")

    def run(off):
        def place(t, o=off):
            buf = torch.full((t.numel() + 16,), 7.0, dtype=t.dtype, device="cuda")
            buf[o:o + t.numel()] = t.reshape(-1)
            return buf, buf.data_ptr() + o * t.element_size()
        (x, px), (dy, pdy), (_, padd), (_, pmask) = keep = [place(base[q]) for q in ("x", "dy", "add", "mask")]
        (y, py), (dx, pdx) = place(torch.full_like(base["dy"], float("nan"))), place(torch.full_like(base["x"], float("nan")))
        dw = torch.full((filt ** nd * c * k,), float("nan"), device="cuda")
        db, pdb = place(torch.full((k,), float("nan"), device="cuda"), 1 if off else 0)
        L.conv_fwd(d, px, w.data_ptr(), None, None, None, py, ws.data_ptr(), s)
        L.conv_dgrad(d, pdy, w.data_ptr(), None, padd, pmask, pdx, ws.data_ptr(), s)
        L.conv_wgrad_bias(d, px, pdy, dw.data_ptr(), pdb, ws.data_ptr(), s)
        torch.cuda.synchronize()
        for buf, count in ((y, base["dy"].numel()), (dx, base["x"].numel())):
            assert bool((buf[:off] == 7).all()) and bool((buf[off + count:] == 7).all())
        o = 1 if off else 0
        assert bool((db[:o] == 7).all()) and bool((db[o + k:] == 7).all())
        cut = lambda buf, like: buf[off:off + like.numel()].double().reshape(like.shape)
        return cut(y, base["dy"]), cut(dx, base["x"]), dw.double(), db[o:o + k].double()

    for name, got, ref, bf16 in zip(("y", "dx", "dw", "db"), run(shift), run(0), (True, True, False, False)):
        rms = float(ref.square().mean().sqrt())
        assert bool(((got - ref).abs() <= (2.0 ** -7 * ref.abs() if bf16 else 0) + 2.0 ** -14 * (ref.abs() + rms)).all()), name


@pytest.mark.parametrize("shift", [1, 2, 4])
@pytest.mark.parametrize("n,sp,c,k", [(3, (45, 37), 72, 40), (60, (14, 14), 264, 256), (2, (23, 21), 264, 136), (1, (13, 13, 12), 96, 144), (9, (88, 88), 72, 24)])
def test_filter_between_vector_boundaries(n, sp, c, k, shift):
    """A 3x3 or 3x3x3 filter that starts between 16-byte boundaries: the forward pass takes the kernel that it takes otherwise, the same bits."""
    import torch
    import paper_1807_02037_amd as L
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    filt = (3,) * len(sp)
    x = torch.randn((n,) + sp + (c,), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randn(filt + (c, k), generator=g, device="cuda").to(torch.bfloat16)
    moved = torch.empty(w.numel() + 8, dtype=torch.bfloat16, device="cuda")[shift:shift + w.numel()].copy_(w.reshape(-1))
    d = L.conv_desc(n, sp, c, k, filt, 1, 1, 0)
    ws = torch.empty(L.conv_workspace_bytes(d, L.abi.CONV_FWD), dtype=torch.uint8, device="cuda")
    out = []
    for t in (w, moved):
        y = torch.full((n,) + sp + (k,), float("nan"), dtype=torch.bfloat16, device="cuda")
        L.conv_fwd(d, x.data_ptr(), t.data_ptr(), None, None, None, y.data_ptr(), ws.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        out.append(y)
    assert bool(torch.isfinite(out[0]).all()) and torch.equal(out[0], out[1])
