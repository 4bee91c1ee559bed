"""Global average pooling and its gradient at the edges of the work split (channel vectors that fill no work-group,
channel counts that are no multiple of 8, one position, more positions than row lanes, small images that share a work-group, batches
beyond one launch), node by node against the oracle on the GPU's own inputs.  Tolerance: one bf16 rounding (2^-8 of the
value) and fp32 sums far below it."""
import numpy as np
import pytest

import workloads as W
from node_oracle import eval_node

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,size,width", [(2, 32, 16), (1, 1, 8), (3, 7, 72), (2, 9, 20), (1, 23, 3), (5, 6, 520), (70, 5, 264), (1, 67, 10)])
def test_gap_forward_and_gradient(batch, size, width):
    import paper_1807_02037_amd as L
    from paper_1807_02037_amd.session import Session
    A = L.abi
    spec = W.tiny_chain(batch=batch, size=size, cin=8, width=width, depth=1)
    s = Session(spec, W.make_tensors(spec, affine="random"), flags=A.X_KEEP_ALL)
    s.step()
    seen = 0
    for info in s.infos:
        if info.op not in (A.OP_GAP, A.OP_GAP_BWD):
            continue
        seen += 1
        x = [s.node_value(i) for i in s.g.node_inputs(info.id)]
        got = s.node_value(info.id)
        want = eval_node(info, s.g.node_attr(info.id), x, tuple(info.dims[i] for i in range(info.ndim)))
        assert np.abs(got - want).max() <= 2.0 ** -8 * np.abs(want).max() + 1e-30, info.name
    assert seen == 2


def _call(name, *args):
    """gap_fwd / gap_bwd of the kernel files, by their C++ names: shapes that no network of a test's size reaches."""
    import ctypes
    import torch
    import paper_1807_02037_amd as L
    f = getattr(ctypes.CDLL(L.abi.lib()._name), name)
    conv = lambda a: ctypes.c_void_p(None if a is None else a.data_ptr()) if a is None or torch.is_tensor(a) else a
    assert f(*map(conv, args), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()


def _gap(n, positions, c, x, y, dx, mask):
    import ctypes
    i64, i32 = ctypes.c_int64, ctypes.c_int
    _call("_ZN3lms7gap_fwdElliPKvPvP12ihipStream_t", i64(n), i64(positions), i32(c), x, y)
    _call("_ZN3lms7gap_bwdElliPKvS1_PvP12ihipStream_t", i64(n), i64(positions), i32(c), y, mask, dx)


# images sharing a work-group in every number (row lanes 1 to 256 over 1, 2 or 4 waves), batches that fill no work-group, one
# and several vectors a row; last: pointers that allow no vectors
@pytest.mark.parametrize("n,positions,c,shift", [
    (1, 1, 8, 0), (777, 1, 2048, 0), (5001, 1, 16, 0), (5003, 4, 16, 0), (4099, 2, 10, 0), (3001, 5, 72, 0), (2500, 9, 24, 0), (9001, 16, 24, 0),
    (3000, 33, 8, 0), (2100, 70, 16, 0), (2050, 300, 32, 0), (5, 700, 40, 0), (2, 3000, 3, 0), (3001, 7, 130, 0), (301, 20, 64, 1), (2500, 3, 32, 1)])
def test_gap_of_any_batch(n, positions, c, shift):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n + c)
    new = lambda count: torch.full((count + shift,), float("nan"), dtype=torch.bfloat16, device="cuda")[shift:]
    x, mask, y, dx = new(n * positions * c), new(n * positions * c), new(n * c), new(n * positions * c)
    x.copy_(torch.randn(x.shape, generator=g, device="cuda"))
    mask.copy_(torch.randn(x.shape, generator=g, device="cuda"))
    _gap(n, positions, c, x, y, dx, mask)
    ref = x.double().reshape(n, positions, c).mean(1)
    mag = x.double().abs().reshape(n, positions, c).mean(1)
    # bf16 has 8 significant bits: nearest rounding moves a value by at most 2^-8 of itself; fp32 sums of at most 3000 terms
    assert bool(((y.double().reshape(n, c) - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -16 * mag).all())
    ref = (y.float().reshape(n, 1, c) / positions).to(torch.bfloat16) * (mask.reshape(n, positions, c) > 0)
    assert torch.equal(dx.reshape(ref.shape), ref)


# more positions than 31 bits count; more images than one launch of the pooling and of its gradient takes
@pytest.mark.parametrize("n,positions,c", [(1, (1 << 31) + 8, 1), ((1 << 19) + 3, 1, 4095), ((1 << 31) // 3 + 7, 1, 3)])
def test_gap_beyond_one_launch(n, positions, c):
    import torch
    if positions == 1:
        x = torch.arange(251, dtype=torch.float32, device="cuda").to(torch.bfloat16).repeat(n * c // 251 + 1)[: n * c]
    else:                             # ones: the lanes' fp32 sums, 2^23 each, are exact
        x = torch.ones(n * positions * c, dtype=torch.bfloat16, device="cuda")
    y, dx = torch.empty(n * c, dtype=torch.bfloat16, device="cuda"), torch.full_like(x, float("nan"))
    _gap(n, positions, c, x, y, dx, None)
    if positions == 1:
        assert torch.equal(y, x) and torch.equal(dx, x)
    else:
        assert float(y) == 1.0 and bool((dx == torch.full((), 1.0 / positions).to(torch.bfloat16).item()).all())
