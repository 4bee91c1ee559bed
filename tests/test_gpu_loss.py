"""Loss and gradient out of one pass: squared error with and without full 16-byte vectors, below and above one vector per thread and
work-group, softmax cross-entropy with few classes on fewer and more rows than the grid has threads, and with many classes.  The loss
against float64 from the operands the step kept (fp32 sums of positive terms: 1e-5), the gradient against the same arithmetic in fp32
(one rounding to bf16: 2^-8 of the element; the exponentials of the device are good to 1e-6)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SPECS = {
    "mse_scalar": lambda: W.tiny_chain(batch=3, size=9, width=16),
    "mse_small": lambda: W.bottleneck_stage(batch=1, size=5),
    "mse_large": lambda: W.bottleneck_stage(batch=7, size=56),
    "ce_few": lambda: W.unet3d(batch=1, size=8, base=8, levels=2),
    "ce_rows": lambda: W.unet3d(batch=1, size=72, base=8, levels=2),
    "ce_wide": lambda: W.resnet50(batch=3, size=64, stage_blocks=(1, 1), base=32),
}


@pytest.mark.parametrize("name", sorted(SPECS))
def test_loss_and_gradient(name):
    import torch
    import paper_1807_02037_amd as L
    from paper_1807_02037_amd.session import Session
    spec = SPECS[name]()
    s = Session(spec, W.make_tensors(spec), flags=L.abi.X_KEEP_ALL, lr=0.0)
    for _ in range(2):
        loss, _ = s.step()
    spec_loss = spec["loss"]
    y = s.node_tensor(s.ids[spec_loss["in"]]).float()
    t = s.dev[spec_loss["target"]]
    grad = [i for i in s.infos if i.name.decode().startswith("loss/grad")]
    assert len(grad) == 1
    dy = s.node_tensor(grad[0].id).float().reshape(y.shape)
    relu = any(layer["name"] == spec_loss["in"] and layer.get("relu") for layer in spec["layers"])
    if spec_loss["op"] == "mse":
        ref = float(((y.double() - t.double()) ** 2).mean())
        g = torch.tensor(2.0 / y.numel(), dtype=torch.float32, device="cuda") * (y - t.float())
    else:
        lp = torch.log_softmax(y.double(), dim=-1).reshape(-1, y.shape[-1])
        lab = t.reshape(-1).long()
        ref = float(-lp[torch.arange(lab.numel(), device="cuda"), lab].mean())
        g = ((lp.exp() - torch.nn.functional.one_hot(lab, y.shape[-1])) / lab.numel()).float().reshape(y.shape)
    if relu:
        g = torch.where(y > 0, g, torch.zeros_like(g))
    assert abs(loss - ref) <= 1e-5 * abs(ref)
    # without keep-all the gradient may be written over y while the same pass sums the loss: the same bits of the loss and of every
    # parameter gradient
    packed = Session(spec, W.make_tensors(spec), lr=0.0)
    loss2, _ = packed.step()
    assert loss2 == loss
    kept, bits = s.grad_bits(), packed.grad_bits()
    assert kept.keys() == bits.keys() and all(np.array_equal(kept[k], bits[k]) for k in kept)
    assert np.isfinite(loss) and bool(((dy - g).abs() <= 2.0 ** -8 * g.abs() + 1e-6 / y.numel()).all())
