"""Global average pooling and its gradient at the edges of the work split (channel vectors that fill no work-group,
channel counts that are no multiple of 8, one position, more positions than row lanes), node by node against the
oracle on the GPU's own inputs.  Tolerance: one bf16 rounding (2^-8 of the value) and fp32 sums far below it."""
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
