"""Stride-1 3x3 and 3x3x3 convolutions that keep the extents, at the edges of the tiles of consecutive positions: fewer positions
than one tile, a last tile with few rows, images that begin inside a tile, channel counts that fill no block or tile, one and
two groups of waves, rows too wide for the widest tile.  Reference: float64 over the GPU's own bf16 inputs; bound: bf16
rounding of the result plus fp32 sums.  The two parameter gradients of the same layers: 2e-6 of the norm."""
import pytest

pytestmark = pytest.mark.gpu

# n, extents, c, k
CASES = [
    (1, (1, 1), 8, 8), (1, (3, 2), 40, 24), (3, (5, 7), 264, 72), (2, (9, 120), 16, 40), (2, (9, 121), 16, 40), (5, (13, 88), 24, 200),
    (70, (14, 14), 136, 256), (131, (23, 21), 40, 32), (9, (7, 7), 264, 264), (1, (40, 87), 96, 96),
    (1, (1, 1, 1), 8, 8), (2, (2, 1, 3), 88, 48), (1, (5, 6, 7), 96, 24), (3, (3, 11, 13), 40, 104), (1, (33, 31, 30), 72, 64),
    (2, (3, 4, 87), 24, 16), (2, (3, 4, 88), 24, 16), (1, (41, 40, 39), 8, 40),
    # tiles of 256 positions, the last one partly filled: 256 x 64 up to rows of 87, 256 x 32 up to 119 (narrow outputs, or any
    # where 256 x 64 does not fit); rows of 88, 119, 120 and 121 beside them
    (9, (87, 87), 40, 72), (13, (77, 71), 72, 64), (9, (88, 88), 72, 64), (13, (89, 119), 40, 32), (10, (99, 119), 24, 72), (9, (75, 120), 40, 32),
    (9, (75, 120), 200, 72), (8, (76, 121), 40, 64), (1, (40, 43, 41), 40, 32), (1, (42, 40, 41), 40, 72), (2, (20, 41, 87), 24, 72),
    # between one and two of the 64 x 64 tiles for a compute unit, long reduction: 128 x 64; one at most: two groups
    (3, (45, 37), 256, 256), (2, (23, 21), 264, 136),
    # rings of filter rows: 256 x 64 with three up to rows of 39 and two beyond, 128 x 64 with four up to 55, three up to 103, two beyond and
    # for one or two blocks of the reduction in the plane
    (22, (40, 39), 24, 72), (22, (39, 40), 72, 72), (9, (43, 55), 24, 72), (9, (43, 56), 72, 72), (4, (53, 103), 24, 72), (4, (53, 104), 72, 72),
    (1, (27, 28, 29), 24, 72), (1, (33, 32, 33), 40, 72),
    (9, (43, 55), 8, 40), (22, (40, 39), 8, 72),
    # the reduction of a tile split among its waves: tiles of 32 and of 64 positions, fewer units than waves, partial units, columns beyond the last
    # tile, and the shapes beside the rule
    (1, (56, 56), 64, 72), (1, (30, 31), 104, 184), (1, (6, 7, 8), 128, 64), (1, (10, 10, 10), 48, 56), (3, (7, 7), 512, 320), (1, (3, 3, 87), 64, 64), (1, (1, 120), 64, 128),
    (1, (16, 16, 17), 256, 232), (1, (13, 14, 15), 104, 256), (32, (7, 7), 520, 512), (9, (20, 20), 64, 136), (1, (25, 25, 26), 64, 64), (1, (20, 20, 20), 128, 96),
    # weight gradient of a volume, patches of a work-group: eight, nine, and a last one with fewer; a ring of four: nine, ten, twenty
    (1, (64, 64, 64), 32, 32), (1, (65, 64, 64), 32, 32), (1, (64, 33, 47), 40, 72), (2, (21, 35, 30), 72, 104),
    (1, (36, 64, 64), 64, 32), (1, (40, 64, 32), 64, 64), (1, (37, 63, 62), 56, 40),
]


@pytest.mark.parametrize("n,sp,c,k", CASES)
def test_all_directions(n, sp, c, k):
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    nd = len(sp)
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k + n)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
    filt = (3,) * nd
    x, dy, addend = rnd(n, *sp, c), rnd(n, *sp, k), rnd(n, *sp, c)
    w = (rnd(*filt, c, k).float() / (c * 3 ** nd) ** 0.5).to(torch.bfloat16)
    d = L.conv_desc(n, sp, c, k, filt, 1, 1, 0)
    s = torch.cuda.current_stream().cuda_stream
    y, dx = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
    dw, db = torch.full(filt + (c, k), float("nan"), device="cuda"), torch.full((k,), float("nan"), device="cuda")
    ws = torch.full((max(L.conv_workspace_bytes(d, q) for q in (A.CONV_FWD, A.CONV_DGRAD, A.CONV_WGRAD_BIAS)) + 256,), 255, dtype=torch.uint8,
                    device="cuda")
    L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, y.data_ptr(), ws.data_ptr(), s)
    L.conv_dgrad(d, dy.data_ptr(), w.data_ptr(), None, addend.data_ptr(), None, dx.data_ptr(), ws.data_ptr(), s)
    L.conv_wgrad_bias(d, x.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), ws.data_ptr(), s)
    torch.cuda.synchronize()

    # tap by tap over a padded copy, float64 on the device
    pad = [0, 0] + [1, 1] * nd
    xp, dyp = torch.nn.functional.pad(x.double(), pad), torch.nn.functional.pad(dy.double(), pad)
    wd, dyd = w.double(), dy.double().reshape(-1, k)
    ry, rdx, rdw = torch.zeros_like(dyd), addend.double().reshape(-1, c), torch.zeros_like(dw, dtype=torch.float64)
    ay, adx = ry.clone(), rdx.abs()
    for tap in torch.cartesian_prod(*[torch.arange(3)] * nd).tolist():
        cut = (slice(None),) + tuple(slice(t, t + e) for t, e in zip(tap, sp))
        back = (slice(None),) + tuple(slice(2 - t, 2 - t + e) for t, e in zip(tap, sp))
        xt, dt, wt = xp[cut].reshape(-1, c), dyp[back].reshape(-1, k), wd[tuple(tap)]
        ry += xt @ wt
        ay += xt.abs() @ wt.abs()
        rdx += dt @ wt.t()
        adx += dt.abs() @ wt.abs().t()
        rdw[tuple(tap)] = xt.t() @ dyd
    # one bf16 rounding (2^-9), and fp32 sums of exact products: 2^-18 of the sum of magnitudes covers 27 * 264 terms in any order
    for got, ref, mag in ((y, ry, ay), (dx, rdx, adx)):
        assert bool(((got.double().reshape(ref.shape) - ref).abs() <= ref.abs() * 2.0 ** -8 + mag * 2.0 ** -18).all())
    assert float((dw.double() - rdw).norm() / rdw.norm().clamp_min(1e-30)) <= 2e-6
    assert float((db.double() - dyd.sum(0)).norm() / dyd.sum(0).norm()) <= 2e-6


# n, extents, c, k, direction, part of the kernel's name
KERNELS = [
    # tiles of 128 x 64, one and two blocks of the reduction in the plane: a ring of two filter rows; from three blocks on four, three where four do not fit, two beyond; 256 x 64
    (9, (43, 55), 24, 72, "fwd", "FlatTile<128, 64, 2, 2, 6, 2,"), (9, (43, 55), 40, 72, "fwd", "FlatTile<128, 64, 2, 2, 6, 2,"),
    (9, (43, 55), 72, 72, "fwd", "FlatTile<128, 64, 2, 2, 4, 4,"), (9, (43, 56), 40, 72, "fwd", "FlatTile<128, 64, 2, 2, 6, 2,"),
    (9, (43, 56), 72, 72, "dgrad", "FlatTile<128, 64, 2, 2, 6, 3,"), (4, (53, 104), 72, 72, "fwd", "FlatTile<128, 64, 2, 2, 6, 2,"), (1, (27, 28, 29), 24, 72, "fwd", "FlatTile<128, 64, 2, 2, 4, 4,"),
    (22, (39, 39), 24, 72, "fwd", "FlatTile<256, 64, 4, 1, 6, 3,"), (22, (40, 40), 72, 72, "fwd", "FlatTile<256, 64, 4, 1, 8, 2,"),
    # the split reduction: tiles of 32 positions, of 64, and the layers beside it
    (2, (20, 21), 120, 136, "fwd", "SplitTile<1>"), (1, (56, 56), 64, 72, "fwd", "conv_flat_kernel"), (1, (30, 31), 104, 184, "dgrad", "SplitTile<1>"),
    (2, (20, 21), 136, 120, "dgrad", "conv_flat_kernel"), (2, (20, 21), 136, 160, "dgrad", "conv_flat_kernel"), (1, (6, 7, 8), 56, 40, "fwd", "SplitTile<1>"),
    (1, (15, 16, 16), 256, 232, "fwd", "SplitTile<2>"), (1, (15, 16, 16), 256, 232, "dgrad", "SplitTile<2>"), (32, (7, 7), 512, 520, "dgrad", "SplitTile<2>"),
    (32, (7, 7), 520, 512, "fwd", "conv_flat_kernel"), (1, (16, 16, 17), 256, 232, "fwd", "conv_flat_kernel"),
    # the weight gradient's ring: from 20 MB on, from 32 MB with few input channels, more than eight patches a work-group, more than one tile
    (1, (36, 64, 64), 64, 32, "wgrad", "wgrad_patch_ring_kernel"), (1, (32, 64, 64), 64, 32, "wgrad", "wgrad_patch_group_kernel"), (1, (40, 64, 32), 64, 64, "wgrad", "wgrad_patch_ring_kernel"),
    (1, (39, 64, 31), 64, 64, "wgrad", "wgrad_patch_group_kernel"), (1, (64, 64, 64), 40, 64, "wgrad", "wgrad_patch_ring_kernel"), (1, (36, 64, 64), 40, 64, "wgrad", "wgrad_patch_group_kernel"),
    (1, (64, 64, 80), 32, 32, "wgrad", "wgrad_patch_group_kernel"), (1, (22, 22, 22), 128, 152, "wgrad", "wgrad_patch_group_kernel"),
]


def pointers(n, sp, c, k, make):
    """x, dy, w, and outputs of all directions as this file's layers have them; workspace; descriptor."""
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    filt = (3,) * len(sp)
    x, dy, w = make(n, *sp, c), make(n, *sp, k), make(*filt, c, k)
    d = L.conv_desc(n, sp, c, k, filt, 1, 1, 0)
    ws = torch.empty(max(L.conv_workspace_bytes(d, q) for q in (A.CONV_FWD, A.CONV_DGRAD, A.CONV_WGRAD_BIAS)) + 256, dtype=torch.uint8, device="cuda")
    return x, dy, w, torch.full_like(dy, float("nan")), torch.full_like(x, float("nan")), ws, d


@pytest.mark.parametrize("n,sp,c,k,direction,part", KERNELS)
def test_kernel_of_a_layer(n, sp, c, k, direction, part):
    """Each rule of the choice between the kernels on both of its sides, by the kernel's name."""
    import torch
    from helpers import kernel_names
    import paper_1807_02037_amd as L
    x, dy, w, y, dx, ws, d = pointers(n, sp, c, k, lambda *shape: torch.zeros(shape, dtype=torch.bfloat16, device="cuda"))
    dw, db = torch.empty((3,) * len(sp) + (c, k), device="cuda"), torch.empty((k,), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    call = {"fwd": lambda: L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, y.data_ptr(), ws.data_ptr(), s),
            "dgrad": lambda: L.conv_dgrad(d, dy.data_ptr(), w.data_ptr(), None, None, None, dx.data_ptr(), ws.data_ptr(), s),
            "wgrad": lambda: L.conv_wgrad_bias(d, x.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), ws.data_ptr(), s)}[direction]
    names = kernel_names(call)
    assert any(part in v for v in names), names


# n, extents, c, k: the split reduction with every term of the epilogues.  Tiles of 64 positions in both directions with several chunks and a
# partial last one of either reduction; in the plane for the data gradient; tiles of 32
SPLIT = [(1, (15, 16, 16), 256, 232), (1, (15, 16, 16), 232, 256), (32, (7, 7), 512, 520), (2, (20, 21), 120, 168), (1, (9, 10, 11), 192, 72)]


@pytest.mark.parametrize("n,sp,c,k", SPLIT)
def test_split_reduction_epilogues(n, sp, c, k):
    import torch
    import paper_1807_02037_amd as L
    A = L.abi
    nd = len(sp)
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
    x, dy, w, y, dx, ws, _ = pointers(n, sp, c, k, rnd)
    w = (w.float() / (c * 3 ** nd) ** 0.5).to(torch.bfloat16)
    res, addend, mask = rnd(*dy.shape), rnd(*x.shape), rnd(*x.shape)
    scale, shift = 1 + 0.1 * torch.randn(k, generator=g, device="cuda"), torch.randn(k, generator=g, device="cuda")
    d = L.conv_desc(n, sp, c, k, (3,) * nd, 1, 1, A.F_RELU | A.F_AFFINE | A.F_RES)
    ws = torch.empty(max(L.conv_workspace_bytes(d, q) for q in (A.CONV_FWD, A.CONV_DGRAD)) + 256, dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    L.conv_fwd(d, x.data_ptr(), w.data_ptr(), scale.data_ptr(), shift.data_ptr(), res.data_ptr(), y.data_ptr(), ws.data_ptr(), s)
    L.conv_dgrad(d, dy.data_ptr(), w.data_ptr(), scale.data_ptr(), addend.data_ptr(), mask.data_ptr(), dx.data_ptr(), ws.data_ptr(), s)
    torch.cuda.synchronize()
    pad = [0, 0] + [1, 1] * nd
    xp, dyp = torch.nn.functional.pad(x.double(), pad), torch.nn.functional.pad(dy.double(), pad)
    wd, wsd = w.double(), (w.float() * scale).to(torch.bfloat16).double()
    ry, rdx = torch.zeros_like(dy, dtype=torch.float64).reshape(-1, k), torch.zeros_like(x, dtype=torch.float64).reshape(-1, c)
    ay, adx = ry.clone(), rdx.clone()
    for tap in torch.cartesian_prod(*[torch.arange(3)] * nd).tolist():
        xt = xp[(slice(None),) + tuple(slice(t, t + e) for t, e in zip(tap, sp))].reshape(-1, c)
        dt = dyp[(slice(None),) + tuple(slice(2 - t, 2 - t + e) for t, e in zip(tap, sp))].reshape(-1, k)
        ry += xt @ wd[tuple(tap)]
        ay += xt.abs() @ wd[tuple(tap)].abs()
        rdx += dt @ wsd[tuple(tap)].t()
        adx += dt.abs() @ wsd[tuple(tap)].abs().t()
    ry, ay = ry * scale.double() + shift.double() + res.double().reshape(-1, k), ay * scale.double()
    rdx = (rdx + addend.double().reshape(-1, c)) * (mask.double().reshape(-1, c) > 0)
    # one bf16 rounding, fp32 sums of up to 27 * 256 exact products (2^-18 of their magnitudes) and the terms added in fp32
    for got, ref, mag in ((y, ry.clamp_min(0), ay + ry.abs() + 8), (dx, rdx, adx + 8)):
        assert bool(((got.double().reshape(ref.shape) - ref).abs() <= ref.abs() * 2.0 ** -8 + mag * 2.0 ** -18).all())


@pytest.mark.parametrize("n,sp,c,k", [(1, (15, 16, 16), 256, 232), (1, (9, 10, 11), 192, 72), (2, (20, 21), 120, 168), (32, (7, 7), 512, 520), (3, (45, 37), 72, 40)])
def test_infinities_and_nan_stay_in_their_windows(n, sp, c, k):
    """Tiles are runs of positions: a tap beyond the edge of an image reads a pixel of another row or image and has to replace it by zeros, infinities and NaN included."""
    import torch
    import paper_1807_02037_amd as L
    nd = len(sp)
    x, dy, w, y, dx, ws, d = pointers(n, sp, c, k, lambda *shape: torch.ones(shape, dtype=torch.bfloat16, device="cuda"))
    w *= 2.0 ** -4
    values = (float("nan"), float("inf"), float("-inf"))
    first, last, side = (0,) + (0,) * nd, (n - 1,) + tuple(e - 1 for e in sp), (n // 2, sp[0] // 2) + (0,) * (nd - 2) + (sp[-1] - 1,)
    for at, v in zip((first, side, last), values):
        x[at + (c // 2,)] = v
        dy[at + (k - 1,)] = v
    s = torch.cuda.current_stream().cuda_stream
    L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, y.data_ptr(), ws.data_ptr(), s)
    L.conv_dgrad(d, dy.data_ptr(), w.data_ptr(), None, None, None, dx.data_ptr(), ws.data_ptr(), s)
    torch.cuda.synchronize()
    for t, out, red in ((x, y, c), (dy, dx, k)):
        # ones everywhere: a finite output is a sixteenth of the taps inside times the channels, in bf16; others are the sum of what their window holds
        pos = t.double().sum(-1)
        special = torch.where(torch.isfinite(pos), torch.zeros_like(pos), pos)
        inside = torch.nn.functional.pad(torch.ones_like(pos), [1, 1] * nd)
        sp_p = torch.nn.functional.pad(special, [1, 1] * nd)
        taps = torch.cartesian_prod(*[torch.arange(3)] * nd).tolist()
        cut = lambda a, tap: a[(slice(None),) + tuple(slice(q, q + e) for q, e in zip(tap, sp))]
        want = sum(cut(inside, tap) for tap in taps) * red / 16 + sum(cut(sp_p, tap) for tap in taps)
        want = want.to(torch.bfloat16).unsqueeze(-1).expand_as(out)
        assert bool(((out == want) | (out.isnan() & want.isnan())).all())
