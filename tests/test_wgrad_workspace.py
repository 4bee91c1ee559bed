"""Workspace of the weight gradients: the partial filters and column sums that the kernel of a geometry writes fit the bytes that
lms_conv_workspace_bytes returns.  On the host from the library's own sizes, over random geometries of every kernel; on the GPU
with a guard region behind the exact size."""
import ctypes
import random

import pytest

import paper_1807_02037_amd as L

A = L.abi


def ints(v):
    return (ctypes.c_int * 3)(*v)


def host(name, ret, *args):
    f = getattr(ctypes.CDLL(A.lib()._name), name)     # functions of the kernel files, by their C++ names
    f.restype = ret
    return f(*args)


class RunPlan(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int) for f in ("kt", "ctiles", "ktiles", "splits", "q_per_split")] + [("q", ctypes.c_longlong)]


class StemGradPlan(ctypes.Structure):
    _fields_ = [(f, ctypes.c_void_p) for f in ("X", "DY", "part", "cs_part")] + [(f, ctypes.c_int) for f in (
        "cx", "ky", "H", "W", "OH", "OW", "filt", "stride", "pad_h", "pad_w", "run", "lead", "span", "th", "tw", "gpr", "rows", "gw", "groups", "tiles_h",
        "tiles_w", "tiles", "tiles_per_split", "splits")] + [(f, ctypes.c_uint) for f in ("gw_magic", "pix_magic", "span_magic")]


def aligned_splits(n, sp, c, k, filt, stride, pad):
    """Splits of the two kernels that only take tensors on 16-byte boundaries, before the others are asked; 0: neither takes it."""
    if len(sp) == 3:
        return 0
    osp = [(e + 2 * pad - f) // stride + 1 for e, f in zip(sp, filt)]
    a3, o3, f3, s3, p3 = ints((1,) + sp), ints([1] + osp), ints((1,) + tuple(filt)), ints((1, stride, stride)), ints((0, pad, pad))
    i32, i64 = ctypes.c_int, ctypes.c_longlong
    patch = host("_ZN3lms20wgrad_patch_eligibleEiiPKiS1_", ctypes.c_bool, i32(c), i32(k), f3, s3)
    if host("_ZN3lms20wgrad_small_eligibleEiiPKiS1_S1_", ctypes.c_bool, i32(c), i32(k), a3, f3, s3) and (osp[1] >= 64 or not patch):
        p = StemGradPlan()
        took = host("_ZN3lms15wgrad_stem_planERNS_12StemGradPlanExiiPKiS3_S3_S3_S3_", ctypes.c_bool, ctypes.byref(p), i64(n * osp[0] * osp[1]), i32(c), i32(k), a3, o3, f3, s3, p3)
        if took:
            assert 1 <= p.splits <= 256 and p.tiles_per_split * p.splits >= p.tiles > p.tiles_per_split * (p.splits - 1)
            assert p.groups <= 3 * 512 and p.rows * p.gw == p.groups and p.th * p.gpr * 16 <= 256 and p.tiles_w * p.tw >= p.OW and p.tiles_h * p.th >= p.OH
        return p.splits if took else 0
    if not patch or filt != (3, 3) or stride != 1:
        return 0
    r = host("_ZN3lms14wgrad_run_planExPKiS1_S1_S1_ii", RunPlan, i64(n), a3, o3, f3, p3, i32(c), i32(k))
    if r.splits:
        assert (r.splits - 1) * r.q_per_split < r.q <= r.splits * r.q_per_split and r.q_per_split % 32 == 0 and r.q == n * (sp[0] + 1) * (sp[1] + 1)
    return r.splits


def written(n, sp, c, k, filt, stride, pad):
    """Splits of the kernel that the launch takes, in its order of choice (the general kernel: at least one), for tensors on any boundary."""
    ext = lambda v: (1,) * (3 - len(v)) + tuple(v)
    nd = len(sp)
    osp = ext([(e + 2 * pad - f) // stride + 1 for e, f in zip(sp, filt)])
    rows, i32, i64 = n * osp[0] * osp[1] * osp[2], ctypes.c_int, ctypes.c_longlong
    f3, s3, p3 = ints(ext(filt)), ints(ext([stride] * nd)), ints((0,) * (3 - nd) + (pad,) * nd)
    a3, o3 = ints(ext(sp)), ints(osp)
    taps = f3[0] * f3[1] * f3[2]
    if taps == 1 and stride == 1 and pad == 0 and k <= 8 and c % 8 == 0 and c <= 256 and (c & (c - 1)) == 0:
        return max(1, min(1024, rows // (256 // (c // 8) * 8)))
    patch = host("_ZN3lms20wgrad_patch_eligibleEiiPKiS1_", ctypes.c_bool, i32(c), i32(k), f3, s3)
    if host("_ZN3lms20wgrad_small_eligibleEiiPKiS1_S1_", ctypes.c_bool, i32(c), i32(k), a3, f3, s3) and (osp[2] >= 64 or not patch):
        return host("_ZN3lms18wgrad_small_splitsExPKi", i32, i64(rows), o3)
    if host("_ZN3lms19wgrad_rows_eligibleEiiPKiS1_S1_S1_", ctypes.c_bool, i32(c), i32(k), a3, f3, s3, p3):
        return host("_ZN3lms17wgrad_rows_splitsExii", i32, i64(rows), i32(c), i32(k))
    if patch:
        return host("_ZN3lms18wgrad_patch_splitsExPKiS1_S1_S1_ii", i32, i64(n), a3, o3, f3, p3, i32(c), i32(k))
    return 1


def test_partials_fit_the_workspace():
    rng, taken = random.Random(5), dict(stem=0, run=0, other=0)
    for _ in range(20000):
        nd = rng.choice((2, 2, 3))
        filt = (rng.choice((1, 3, 3, 7 if nd == 2 else 2)),) * nd
        stride, pad = rng.choice((1, 1, 2)), rng.choice((0, filt[0] // 2))
        sp = tuple(rng.randint(max(1, filt[0] - 2 * pad), 230 if nd == 2 else 100) for _ in range(nd))
        c = rng.choice((1, 2, 3, 4, 8, rng.randint(1, 80), 8 * rng.randint(1, 64)))
        k = rng.choice((1, 8, 32, 64, rng.randint(1, 80), 8 * rng.randint(1, 64)))
        n = rng.randint(1, 9)
        d = L.conv_desc(n, sp, c, k, filt, stride, pad, 0)
        wide = aligned_splits(n, sp, c, k, filt, stride, pad)
        taken["stem" if wide and c <= 4 else "run" if wide else "other"] += 1
        splits = max(wide, written(n, sp, c, k, filt, stride, pad))
        per = c * k * filt[0] ** nd
        what = (n, sp, c, k, filt, stride, pad, splits)
        assert splits * per * 4 <= L.conv_workspace_bytes(d, A.CONV_WGRAD), what
        assert splits * (per + k) * 4 <= L.conv_workspace_bytes(d, A.CONV_WGRAD_BIAS) or (filt[0] == 1 and k <= 8), what
    assert min(taken.values()) >= 50, taken


@pytest.mark.parametrize("n,sp,c,k", [(64, (56, 56), 64, 64), (8, (14, 14), 256, 256), (50, (7, 7), 64, 128), (51, (8, 7), 64, 64), (300, (7, 7), 128, 128), (3, (20, 30), 136, 72)])
def test_patches_of_unaligned_tensors_fill_the_compute_units(n, sp, c, k):
    """3x3 layers whose tensors start between 16-byte boundaries take patches of 8 x 16 positions, two images of at most 8 x 7 to a patch, and a
    work-group per compute unit where there are as many patches: their number of partial filters."""
    patches = (n + 1) // 2 if sp[0] <= 8 and sp[1] <= 7 else n * -(-sp[0] // 8) * -(-sp[1] // 16)
    tiles = -(-c // 64) * -(-k // 64)
    per = -(-patches // min(patches, -(-256 // tiles)))
    ext, one = ints((1,) + sp), ints((1, 3, 3))
    got = host("_ZN3lms18wgrad_patch_splitsExPKiS1_S1_S1_ii", ctypes.c_int, ctypes.c_longlong(n), ext, ext, one, ints((0, 1, 1)), ctypes.c_int(c), ctypes.c_int(k))
    assert got == -(-patches // per)


# first layers whose rows are and are not shorter than a segment, and one geometry of every other kernel; n, extents, c, k, filter, stride, pad
GUARDED = [
    (1, (80, 80, 80), 1, 32, 3, 1, 1), (8, (100, 100), 1, 32, 3, 1, 1), (2, (224, 224), 3, 64, 3, 1, 1), (1, (40, 40, 72), 1, 32, 3, 1, 1),
    (2, (40, 40), 3, 16, 3, 1, 1), (1, (9, 70), 4, 8, 3, 1, 0), (1, (66, 90), 3, 64, 7, 2, 3), (3, (33, 31), 3, 24, 5, 1, 2),
    (2, (20, 21), 64, 72, 1, 1, 0), (1, (33, 35), 16, 8, 1, 1, 0), (2, (17, 19), 64, 64, 1, 2, 0), (1, (15, 14), 64, 80, 3, 1, 1),
    (1, (9, 10, 11), 24, 40, 3, 1, 1), (2, (15, 15), 32, 64, 3, 2, 1), (1, (12, 13), 20, 12, 3, 1, 1), (3, (7, 7), 64, 64, 3, 1, 1),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,sp,c,k,filt,stride,pad", GUARDED)
def test_nothing_behind_the_workspace_is_written(n, sp, c, k, filt, stride, pad):
    import torch
    nd = len(sp)
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    osp = tuple((e + 2 * pad - filt) // stride + 1 for e in sp)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
    x, dy, w = rnd(n, *sp, c), rnd(n, *osp, k), rnd(*(filt,) * nd, c, k)
    d = L.conv_desc(n, sp, c, k, (filt,) * nd, stride, pad, 0)
    s = torch.cuda.current_stream().cuda_stream
    scale = torch.ones(k, device="cuda")
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    dw, dw2, db = torch.full((filt ** nd, c, k), float("nan"), device="cuda"), torch.empty((filt ** nd, c, k), device="cuda"), torch.empty(k, device="cuda")
    calls = ((A.CONV_WGRAD, lambda ws: L.conv_wgrad(d, x.data_ptr(), dy.data_ptr(), dw2.data_ptr(), ws, s)),
             (A.CONV_WGRAD_BIAS, lambda ws: L.conv_wgrad_bias(d, x.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), ws, s)),
             (A.CONV_FWD, lambda ws: L.conv_fwd(d, x.data_ptr(), w.data_ptr(), None, None, None, y.data_ptr(), ws, s)),
             (A.CONV_DGRAD, lambda ws: L.conv_dgrad(d, dy.data_ptr(), w.data_ptr(), scale.data_ptr(), None, None, dx.data_ptr(), ws, s)))
    for which, call in calls:
        need = L.conv_workspace_bytes(d, which)
        buf = torch.full((need + (8 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
        call(buf.data_ptr())
        torch.cuda.synchronize()
        assert bool((buf[need:] == 0xA5).all()), which
    # float64, tap by tap
    xp = torch.nn.functional.pad(x.double(), [0, 0] + [pad, pad] * nd)
    dyd = dy.double().reshape(-1, k)
    for t, tap in enumerate(torch.cartesian_prod(*[torch.arange(filt)] * nd).reshape(-1, nd).tolist()):
        cut = (slice(None),) + tuple(slice(a, a + (o - 1) * stride + 1, stride) for a, o in zip(tap, osp))
        ref = xp[cut].reshape(-1, c).t() @ dyd
        # fp32 sums of exact products: 1e-6 of the norm of the sums of magnitudes
        mag = float((xp[cut].reshape(-1, c).abs().t() @ dyd.abs()).norm())
        assert float((dw[t].double() - ref).norm()) <= 1e-6 * mag, tap
    assert torch.equal(dw, dw2)
    assert float((db.double() - dyd.sum(0)).norm()) <= 1e-6 * float(dyd.abs().sum(0).norm())
