"""Max pooling and its gradient at the edges of the kernels' tiles: maps of one row, column or pixel, extents around a tile of 16,
odd and even, channel counts that fill no group of 64, windows of 1 or 2 per axis, values with many ties, infinities and
NaN (passed over: a window of nothing else names nobody, or its first element without overlap).  Reference: the window walked in
row-major order, strictly greater wins; forward exact, gradient one bf16 rounding of a sum of at most four terms (2^-8, and 2^-22
of the terms' magnitudes for the order of fp32 sums)."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class Geom(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int64)] + [(f, ctypes.c_int * 3) for f in ("in_sp", "out_sp", "filt", "stride", "pad")] + [("c", ctypes.c_int), ("k", ctypes.c_int)]


def reference(x, dy, win, stride, pad, mask, overlap):
    n, d, h, w, c = x.shape
    osp = dy.shape[1:4]
    best = np.full(dy.shape, -np.inf, np.float32)
    arg = np.full(dy.shape, -1 if overlap else 0, np.int64)
    taps = [(a, b, e) for a in range(win[0]) for b in range(win[1]) for e in range(win[2])]
    at = []
    for t, tap in enumerate(taps):
        idx = [np.arange(o) * s + k - p for o, s, k, p in zip(osp, stride, tap, pad)]
        ok = np.ones(osp, bool)
        for i, (ix, e) in enumerate(zip(idx, x.shape[1:4])):
            sh = [1, 1, 1]
            sh[i] = -1
            ok &= ((ix >= 0) & (ix < e)).reshape(sh)
        grid = np.ix_(*[np.clip(ix, 0, e - 1) for ix, e in zip(idx, x.shape[1:4])])
        at.append((idx, ok))
        v = np.where(ok[None, ..., None], x[(slice(None),) + grid], -np.inf)
        better = v > best
        best = np.where(better, v, best)
        arg = np.where(better, t, arg)
    dx, mag = np.zeros(x.shape, np.float64), np.zeros(x.shape, np.float64)
    for t, (idx, ok) in enumerate(at):
        part = np.where((arg == t) & ok[None, ..., None], dy, 0.0)
        grid = np.ix_(*[np.clip(ix, 0, e - 1) for ix, e in zip(idx, x.shape[1:4])])
        for a in range(n):
            np.add.at(dx[a], grid, part[a])
            np.add.at(mag[a], grid, np.abs(part[a]))
    if mask:
        dx = np.where(x > 0, dx, 0.0)
    return best, dx, mag


# n, extents, c, window, stride, padding
CASES = [
    (2, (1, 1, 1), 8, 3, 2, 1), (2, (1, 1, 7), 16, 3, 2, 1), (1, (1, 9, 1), 8, 3, 2, 1), (2, (1, 16, 16), 72, 3, 2, 1), (1, (1, 17, 15), 64, 3, 2, 1),
    (1, (1, 33, 48), 24, 3, 2, 1), (2, (1, 31, 34), 136, 3, 2, 1), (3, (1, 56, 56), 64, 3, 2, 1),
    (2, (1, 6, 10), 8, 2, 2, 0), (1, (4, 6, 8), 24, 2, 2, 0), (2, (2, 2, 2), 16, 2, 2, 0), (3, (16, 16, 16), 40, 2, 2, 0),
]


@pytest.mark.parametrize("n,sp,c,win,stride,pad", CASES)
@pytest.mark.parametrize("mask", [0, 1])
def test_forward_and_gradient(n, sp, c, win, stride, pad, mask):
    import torch
    import paper_1807_02037_amd as L
    flat = win == 3 or sp[0] == 1
    ext = lambda v, d: [d if flat else v, v, v]
    w3, s3, p3 = ext(win, 1), ext(stride, 1), ext(pad, 0)
    osp = [(e + 2 * p - w) // s + 1 for e, w, s, p in zip(sp, w3, s3, p3)]
    rng = np.random.default_rng(c + sp[1])
    x = rng.integers(-2, 3, (n,) + sp + (c,)).astype(np.float32)
    x[(x == 0) & (rng.random(x.shape) < 0.5)] = -0.0             # equal to 0: the first of them is the maximum
    spots = rng.random(x.shape)
    x[spots < 0.04] = np.nan
    x[(spots > 0.04) & (spots < 0.08)] = -np.inf
    x[spots > 0.99] = np.inf
    x[0, ..., 0] = np.nan
    x[0, ..., 1] = -np.inf
    dev = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    xd = dev(x)
    dyd = dev(rng.standard_normal([n] + osp + [c]).astype(np.float32))
    y, dx = torch.empty_like(dyd), torch.full_like(xd, 7.0)
    g = Geom(n, *[(ctypes.c_int * 3)(*v) for v in (sp, osp, w3, s3, p3)], c, c)
    lib, st = ctypes.CDLL(L.abi.lib()._name), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    assert lib._ZN3lms11maxpool_fwdERKNS_8ConvGeomEPKvPvP12ihipStream_t(ctypes.byref(g), ptr(xd), ptr(y), st) == 0
    assert lib._ZN3lms11maxpool_bwdERKNS_8ConvGeomEPKvS4_iPvP12ihipStream_t(ctypes.byref(g), ptr(dyd), ptr(xd), mask, ptr(dx), st) == 0
    torch.cuda.synchronize()
    best, ref, mag = reference(x, dyd.float().cpu().numpy(), w3, s3, p3, mask, win == 3)
    assert np.array_equal(y.float().cpu().numpy(), best)
    assert np.array_equal(np.signbit(y.float().cpu().numpy()), np.signbit(best))
    assert (np.abs(dx.float().cpu().numpy() - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -22 * mag).all()
