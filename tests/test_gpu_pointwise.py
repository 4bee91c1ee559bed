"""Pointwise layers (1x1, any stride) at the edges of the kernel's tiles and of its choice between them: positions that
fill no tile, output channels beyond the last column tile, reductions that end inside a stage of 64 channels, grids with
odd extents under a stride, enough and too few tiles for the wider shapes.  Reference: the same sums in float64 on the
GPU's own bf16 inputs.  Bound per element: 2^-8 of the value (one rounding of the result, half of it, and the rounding
of the scaled filter where there is a scale) plus 2^-8 of the root mean square for sums that cancel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# n, extents, c, k, stride
CASES = [
    (1, (5, 7), 32, 32, 1),            # one partial tile, half a stage
    (2, (9, 13), 40, 72, 1),           # ragged in positions, channels and reduction
    (1, (64, 65), 64, 64, 1),          # exactly one stage, 64 columns
    (3, (75, 150), 72, 64, 1),         # 264 tiles of 128 x 64, one position over
    (2, (91, 90), 96, 136, 1),         # 128 x 128 and 64 x 128 tiles, 8 columns over
    (1, (128, 129), 200, 256, 1),      # 128 x 128 tiles (forward), partial last stage
    (1, (33, 31), 520, 104, 1),        # long reduction, few tiles: 64 x 64
    (4, (15, 17), 64, 128, 2),         # odd extents under a stride
    (1, (64, 130), 128, 96, 2),
    (1, (7, 6, 9), 48, 40, 2),         # 3-D, strided
    (1, (10, 11), 32, 64, 3),
    (2, (5, 6, 7), 64, 200, 1),
    (2, (15, 17), 320, 328, 2),        # data gradient here and not in the general kernel: large filter
    (1, (9, 8, 7), 264, 512, 2),
    (1, (20, 22), 512, 256, 3),
    (9, (57, 55), 128, 256, 2),        # and many products: 128 x 128 / 64 x 128 tiles
    (8, (66, 71), 64, 392, 2),         # 128 x 64 tiles
    # strided data gradients whose work-groups also write the positions between the strides, and sizes beyond which they do not
    (1, (57, 59), 152, 360, 2),        # odd extents: the last positions have no neighbours
    (3, (60, 58), 72, 520, 2),
    (1, (15, 13, 11), 256, 400, 2),    # seven positions to each row
    (2, (40, 1), 256, 400, 2),         # one extent without neighbours
    (1, (25, 26), 320, 328, 3),        # nine positions: a launch of their own
    (2, (15, 16), 1032, 1024, 2),
    (32, (56, 57), 296, 72, 2),        # beyond the caches, rows in whole lines and not
    (32, (56, 57), 320, 72, 2),
    # long reductions on 256 x 128 tiles: one column of them with a partial last stage, and whole lines from memory
    (1, (313, 314), 600, 104, 1), (1, (313, 314), 104, 776, 1), (1, (207, 208), 1024, 232, 1), (1, (207, 208), 232, 1024, 1),
    (2, (256, 258), 160, 64, 2),       # 128 x 64 tiles for 160 columns, under a stride
    # long reductions on other tiles; 153 to 192 columns; masked, 384 channels
    (1, (181, 182), 600, 264, 1), (1, (181, 181), 576, 136, 1), (1, (130, 253), 264, 776, 1), (1, (181, 182), 72, 160, 1), (1, (181, 182), 192, 40, 1),
    (2, (256, 258), 64, 168, 2), (1, (181, 183), 136, 384, 1),
]


def close(got, ref):
    got, ref = got.double(), ref
    rms = float(ref.square().mean().sqrt())
    err = (got - ref).abs()
    lim = 2.0 ** -8 * (ref.abs() + rms)
    assert bool((err <= lim).all()), float((err / lim).max())


@pytest.mark.parametrize("terms", ["all", "none", "mask"])
@pytest.mark.parametrize("n,sp,c,k,stride", CASES)
def test_forward_and_data_gradient(n, sp, c, k, stride, terms):
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    g = torch.Generator(device="cuda")
    g.manual_seed(c * 1000 + k)

    def rnd(shape, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)

    osp = tuple((e - 1) // stride + 1 for e in sp)
    x, w, dy = rnd((n,) + sp + (c,)), rnd((c, k), c ** -0.5), rnd((n,) + osp + (k,))
    scale, shift = (1 + 0.1 * torch.randn(k, generator=g, device="cuda"), torch.randn(k, generator=g, device="cuda")) if terms == "all" else (None, None)
    res, addend = (rnd(dy.shape), rnd(x.shape)) if terms == "all" else (None, None)
    mask = rnd(x.shape) if terms != "none" else None
    d = L.conv_desc(n, sp, c, k, (1,) * len(sp), stride, 0, A.F_RELU if terms == "all" else 0)
    ws = torch.empty(max(L.conv_workspace_bytes(d, A.CONV_FWD), L.conv_workspace_bytes(d, A.CONV_DGRAD), 256), dtype=torch.uint8, device="cuda")
    y, dx = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
    s = torch.cuda.current_stream().cuda_stream
    p = lambda t: None if t is None else t.data_ptr()
    L.conv_fwd(d, p(x), p(w), p(scale), p(shift), p(res), p(y), p(ws), s)
    L.conv_dgrad(d, p(dy), p(w), p(scale), p(addend), p(mask), p(dx), p(ws), s)
    torch.cuda.synchronize()
    grid = (slice(None),) + (slice(None, None, stride),) * len(sp)
    ref = (x[grid].double().reshape(-1, c) @ w.double()).reshape(dy.shape)
    if scale is not None:
        ref = torch.relu(ref * scale.double() + shift.double() + res.double())
    close(y, ref)
    ws64 = w.double() if scale is None else (w.float() * scale).to(torch.bfloat16).double()
    ref = torch.zeros(x.shape, dtype=torch.float64, device="cuda")
    ref[grid] = (dy.double().reshape(-1, k) @ ws64.t()).reshape(ref[grid].shape)
    if addend is not None:
        ref = ref + addend.double()
    if mask is not None:
        ref = ref * (mask > 0)
    close(dx, ref)


@pytest.mark.parametrize("c,k", [(40, 72), (104, 136)])
def test_positions_do_not_leak_into_each_other(c, k):
    """A reduction that ends inside a stage reads past the end of its row: what lies there must not count, NaN included."""
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    x = torch.ones((1, 8, 20, c), dtype=torch.bfloat16, device="cuda")
    x[0, 3, 5] = float("nan")
    x[0, 6, 1] = float("inf")
    dy = torch.ones((1, 8, 20, k), dtype=torch.bfloat16, device="cuda")
    dy[0, 2, 2] = float("nan")
    w = torch.ones((c, k), dtype=torch.bfloat16, device="cuda")
    d = L.conv_desc(1, (8, 20), c, k, (1, 1), 1, 0, 0)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    s = torch.cuda.current_stream().cuda_stream
    L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, y.data_ptr(), ws.data_ptr(), s)
    L.conv_dgrad(d, dy.data_ptr(), w.data_ptr(), None, None, None, dx.data_ptr(), ws.data_ptr(), s)
    torch.cuda.synchronize()
    want = torch.full_like(y, float(c))
    want[0, 3, 5] = float("nan")
    want[0, 6, 1] = float("inf")
    assert np.array_equal(y.float().cpu().numpy(), want.float().cpu().numpy(), equal_nan=True)
    want = torch.full_like(dx, float(k))
    want[0, 2, 2] = float("nan")
    assert np.array_equal(dx.float().cpu().numpy(), want.float().cpu().numpy(), equal_nan=True)


# n, extents, c, k, stride, direction, mask, tile: each rule of launch_pw_shape on both of its sides
TILES = [
    # 256 x 128: whole lines from memory; partial lines, less than 88 MB, columns that do not fill their tiles, wide data gradients beside them
    (256, (14, 14), 1024, 256, 1, "fwd", 0, "256, 128, 4, 2, 3"), (256, (14, 14), 256, 1024, 1, "dgrad", 1, "256, 128, 4, 2, 3"),
    (256, (14, 14), 1032, 256, 1, "fwd", 0, "128, 128, 2, 2"), (200, (14, 14), 1024, 256, 1, "fwd", 0, "128, 128, 2, 2"), (256, (14, 14), 896, 256, 1, "fwd", 0, "128, 128, 2, 2"),
    (256, (14, 14), 1024, 136, 1, "fwd", 0, "128, 128, 2, 2"), (256, (14, 14), 520, 1024, 1, "dgrad", 1, "128, 128, 2, 2"),
    (221, (7, 7), 656, 752, 1, "fwd", 0, "128, 128, 2, 2"), (28, (35, 35), 224, 784, 1, "dgrad", 1, "128, 128, 2, 2"),
    # one column of them, the last round three quarters full and not
    (1, (256, 384), 600, 128, 1, "fwd", 0, "256, 128, 4, 2, 3"), (1, (256, 383), 600, 128, 1, "fwd", 0, "128, 128, 2, 2"),
    (1, (256, 384), 104, 776, 1, "dgrad", 0, "256, 128, 4, 2, 3"), (1, (256, 383), 104, 776, 1, "dgrad", 0, "128, 128, 2, 2"),
    # 160 and 192 columns, short reductions, little for the epilogue: 128 x 64
    (64, (28, 28), 256, 160, 1, "fwd", 0, "128, 64, 2, 2"), (64, (28, 28), 264, 160, 1, "fwd", 0, "128, 128, 2, 2"), (64, (28, 28), 64, 168, 1, "fwd", 0, "128, 128, 2, 2"),
    (64, (28, 28), 192, 40, 1, "dgrad", 1, "128, 64, 2, 2"), (128, (28, 28), 192, 40, 1, "dgrad", 1, "64, 128, 2, 2"), (128, (28, 28), 160, 40, 1, "dgrad", 1, "128, 64, 2, 2"),
    (64, (28, 28), 168, 64, 1, "dgrad", 0, "128, 128, 2, 2"), (41, (28, 28), 160, 64, 1, "dgrad", 0, "128, 128, 2, 2"), (64, (48, 48), 64, 160, 2, "fwd", 0, "128, 64, 2, 2"),
    (64, (48, 48), 160, 64, 2, "dgrad", 1, "128, 64, 2, 2"), (64, (48, 48), 168, 64, 2, "dgrad", 1, "64, 128, 2, 2"),
    # masked, 384 to 512 channels: 128 x 128 where the last round is three quarters full, 64 x 128 where it is not, for less, and under a stride
    (32, (28, 28), 256, 384, 1, "dgrad", 1, "128, 128, 2, 2"), (31, (28, 28), 256, 384, 1, "dgrad", 1, "64, 128, 2, 2"), (32, (28, 28), 256, 376, 1, "dgrad", 1, "64, 128, 2, 2"),
    (31, (23, 23), 464, 400, 1, "dgrad", 1, "64, 128, 2, 2"), (31, (23, 23), 464, 400, 1, "dgrad", 0, "128, 128, 2, 2"), (31, (23, 23), 464, 520, 1, "dgrad", 1, "128, 128, 2, 2"),
    (32, (55, 55), 256, 384, 2, "dgrad", 1, "64, 128, 2, 2"),
]


@pytest.mark.parametrize("n,sp,c,k,stride,direction,mask,tile", TILES)
def test_tile_of_a_layer(n, sp, c, k, stride, direction, mask, tile):
    import torch
    from helpers import kernel_names
    import paper_1807_02037_amd as L
    osp = tuple((e - 1) // stride + 1 for e in sp)
    x, dy = (torch.zeros((n,) + v, dtype=torch.bfloat16, device="cuda") for v in (sp + (c,), osp + (k,)))
    w, ws = torch.zeros((c, k), dtype=torch.bfloat16, device="cuda"), torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    d = L.conv_desc(n, sp, c, k, (1,) * len(sp), stride, 0, 0)
    assert ws.numel() >= max(L.conv_workspace_bytes(d, q) for q in (L.abi.CONV_FWD, L.abi.CONV_DGRAD))
    s = torch.cuda.current_stream().cuda_stream
    if direction == "fwd":
        names = kernel_names(lambda: L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, dy.data_ptr(), ws.data_ptr(), s))
    else:
        dx = torch.empty_like(x)
        names = kernel_names(lambda: L.conv_dgrad(d, dy.data_ptr(), w.data_ptr(), None, None, x.data_ptr() if mask else None, dx.data_ptr(), ws.data_ptr(), s))
    assert any("PwTile<%s" % tile in v for v in names), names
