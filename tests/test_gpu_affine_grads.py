"""Filter and scale gradient of affine layers out of one pass over the raw filter gradient: channel counts below and above one
work-group's columns, with and without whole groups of four, fewer and more rows than are in flight, the filter size from which a
work-group takes whole lines.  The filter gradient is one product per element, the same bits; the scale gradient against float64:
fp32 sums of n products, each addition off by at most 2^-24 of the partial sum, which 4 accumulators, the shuffles and the waves
keep to chains of at most n / 32 + 40 additions in every variant."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# input channels, output channels, filter extent
LAYERS = [(8, 4, 1), (8, 6, 1), (16, 8, 1), (64, 40, 1), (8, 256, 3), (72, 24, 3), (255, 20, 1), (257, 64, 1), (128, 36, 3), (512, 128, 3),
          (1032, 64, 1), (512, 512, 3), (1024, 2048, 1)]


@pytest.mark.parametrize("c,k,filt", LAYERS)
def test_scale_and_filter_gradient(c, k, filt):
    import torch
    import paper_1807_02037_amd as L
    from paper_1807_02037_amd.session import Session
    layer = {"name": "y", "op": "conv", "in": "x", "filt": (filt, filt), "cout": k, "stride": 1, "pad": filt // 2, "relu": False,
             "res": None, "affine": True, "bias": False}
    spec = {"name": "affine_layer", "cfg": 0, "ndim": 2, "input": ("x", (2, 5, 5, c)), "layers": [layer],
            "loss": {"op": "mse", "in": "y", "target": "t"}}
    s = Session(spec, W.make_tensors(spec, affine="random"), flags=L.abi.X_KEEP_ALL, lr=0.0)
    s.step()
    raw = s.node_tensor(next(i.id for i in s.infos if i.name.decode() == "y/dw_raw")).reshape(-1, k)
    w, scale, dw, dscale = s.dev["y.w"], s.dev["y.scale"], s.dev["grad/y.w"].reshape(-1, k), s.dev["grad/y.scale"]
    assert torch.equal(dw, raw * scale)
    terms = raw.double() * w.reshape(-1, k).double()
    chain = terms.shape[0] / 32 + 40
    assert bool(((dscale.double() - terms.sum(0)).abs() <= chain * 2.0 ** -24 * terms.abs().sum(0) + 1e-30).all())
