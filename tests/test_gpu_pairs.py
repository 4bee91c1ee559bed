"""Operations that the executor computes together with a neighbour (a loss with its gradient, the filter gradient of an affine
layer with its scale gradient) in graphs built by hand, where they may be and where something between them forbids it."""
import pytest

pytestmark = pytest.mark.gpu


GUARD = 1 << 20          # bytes behind the arena that the executor was given


class Built:
    """A graph whose variables and results are all bound to tensors of the caller."""

    def __init__(self, flags=0):
        import paper_1807_02037_amd as L
        self.L, self.A, self.g, self.flags = L, L.abi, L.Graph(), flags
        self.dev, self.ex = {}, None

    def var(self, name, tensor, kind):
        import torch
        dtype = {torch.bfloat16: self.A.BF16, torch.float32: self.A.F32, torch.int32: self.A.I32}[tensor.dtype]
        node = self.g.add_variable(name, dtype, tuple(tensor.shape), kind)
        self.dev[node] = tensor
        return node

    def op(self, name, op, inputs, phase=None, out=None, **attr):
        node = self.g.add_op(name, op, inputs, self.A.BWD if phase is None else phase, **attr)
        if out is not None:
            self.g.set_external(node)
            self.dev[node] = out
        return node

    def step(self):
        import torch
        if self.ex is None:
            need = self.g.memory_need()[1]
            self.arena = torch.full((need + GUARD,), 0xa5, dtype=torch.uint8, device="cuda")
            self.need = need
            self.streams = [torch.cuda.Stream() for _ in range(3)]
            torch.cuda.synchronize()
            self.pool = self.L.api.PinnedPool(1 << 20)
            self.ex = self.L.Executor(self.g, self.arena.data_ptr(), need, self.pool.ptr, 1 << 20, *[s.cuda_stream for s in self.streams], self.flags)
            for node, t in self.dev.items():
                self.ex.bind(node, t.data_ptr())
        out = self.ex.step()
        torch.cuda.synchronize()
        assert bool((self.arena[self.need:] == 0xa5).all())
        return out


def rnd(seed, shape, dtype=None):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(dtype or torch.bfloat16)


@pytest.mark.parametrize("first", ["scale", "dot"])
@pytest.mark.parametrize("update", [None, "filter", "scale"])
def test_affine_gradients_read_the_updated_variable(first, update):
    """An operation created after an update reads the updated value, also where the update is held back (everything bound)."""
    import torch
    rows, k, lr = 96, 40, 0.5
    f32 = torch.float32
    b = Built()
    A = b.A
    raw, w, scale = rnd(1, (1, 1, rows, k), f32), rnd(2, (1, 1, rows, k)), rnd(3, (k,), f32)
    vraw, vw, vs = b.var("raw", raw, A.VAR_CONST), b.var("w", w, A.VAR_PARAM), b.var("s", scale, A.VAR_PARAM)
    if update:
        var, t = (vw, w) if update == "filter" else (vs, scale)
        grad = rnd(4, tuple(t.shape), f32)
        ref = (t.float() - lr * grad).to(t.dtype)
        u = b.op("upd", A.OP_SGD, [var, b.var("g", grad, A.VAR_CONST)], phase=A.UPD, out=t, lr=lr)
        b.g.add_update_edge(u, var)
    dw, ds = torch.full_like(raw, float("nan")), torch.full_like(scale, float("nan"))
    ops = [("dw", A.OP_SCALE_COLS, [vraw, vs], dw), ("ds", A.OP_DOT_COLS, [vraw, vw], ds)]
    for name, op, inputs, out in (ops if first == "scale" else ops[::-1]):
        b.op(name, op, inputs, out=out)
    _, st = b.step()
    torch.cuda.synchronize()
    if update:
        assert float((t.float() - ref.float()).abs().max()) <= 2.0 ** -7 * float(ref.float().abs().max())
    assert torch.equal(dw, raw * scale)
    terms = raw.double() * w.double()
    assert bool(((ds.double() - terms.sum((0, 1, 2))).abs() <= 1e-5 * terms.abs().sum((0, 1, 2))).all())
    if not update:
        assert st.n_kernels == 1


@pytest.mark.parametrize("kind", ["mse", "ce"])
@pytest.mark.parametrize("update", [None, "before", "between"])
def test_loss_reads_what_it_was_created_on(kind, update):
    """A target (or the logits) updated between the loss and its gradient: the loss is of the old values, the gradient of the new ones."""
    import torch
    n, c, lr = 300, 16, 0.5
    f32 = torch.float32
    b = Built()
    A = b.A
    y = rnd(5, (n, c))
    t = rnd(6, (n, c)) if kind == "mse" else torch.arange(n, dtype=torch.int32, device="cuda") % c
    vy, vt = b.var("y", y, A.VAR_PARAM), b.var("t", t, A.VAR_TARGET)
    grad = rnd(7, (n, c), f32)
    old = y.clone()
    upd = None

    def add_update():
        u = b.op("upd", A.OP_SGD, [vy, b.var("g", grad, A.VAR_CONST)], phase=A.UPD, out=y, lr=lr)
        b.g.add_update_edge(u, vy)

    if update == "before":
        add_update()
    b.op("loss", A.OP_MSE if kind == "mse" else A.OP_SOFTMAX_CE, [vy, vt], phase=A.FWD)
    if update == "between":
        add_update()
    dy = torch.full_like(y, float("nan"))
    b.op("dy", A.OP_MSE_GRAD if kind == "mse" else A.OP_SOFTMAX_CE_GRAD, [vy, vt], out=dy)
    loss, st = b.step()
    torch.cuda.synchronize()
    new = (old.float() - lr * grad).to(torch.bfloat16) if update else old
    assert float((y.float() - new.float()).abs().max()) <= 2.0 ** -7 * float(new.float().abs().max())
    at_loss = (old if update == "between" else y).double()
    if kind == "mse":
        ref, g = float(((at_loss - t.double()) ** 2).mean()), 2.0 / y.numel() * (y.double() - t.double())
    else:
        lab = t.long()
        ref = float(torch.nn.functional.cross_entropy(at_loss, lab))
        g = (torch.softmax(y.double(), -1) - torch.nn.functional.one_hot(lab, c)) / n
    assert abs(loss - ref) <= 1e-5 * abs(ref)
    assert bool(((dy.double() - g).abs() <= 2.0 ** -8 * g.abs() + 1e-6 / n).all())
    assert st.n_kernels == (2 if update is None else 3 if update == "before" else 4), st.n_kernels


@pytest.mark.parametrize("kind,n,c", [("mse", 300, 16), ("mse", 7, 9), ("mse", 50000, 128), ("ce", 300, 16), ("ce", 300000, 4), ("ce", 70, 1000), ("ce", 5000, 65)])
def test_loss_has_the_same_bits_apart(kind, n, c):
    """The same loss and gradient with a control edge between them, which keeps them apart, and without; the arena holds what the plan
    asks for and nothing else is written."""
    import torch
    got = []
    for apart in (False, True):
        b = Built()
        A = b.A
        y = rnd(8, (n, c))
        t = rnd(9, (n, c)) if kind == "mse" else torch.arange(n, dtype=torch.int32, device="cuda") % c
        vy, vt = b.var("y", y, A.VAR_PARAM), b.var("t", t, A.VAR_TARGET)
        loss = b.op("loss", A.OP_MSE if kind == "mse" else A.OP_SOFTMAX_CE, [vy, vt], phase=A.FWD)
        dy = torch.full_like(y, float("nan"))
        grad = b.op("dy", A.OP_MSE_GRAD if kind == "mse" else A.OP_SOFTMAX_CE_GRAD, [vy, vt], out=dy)
        if apart:
            b.g.add_control_edge(loss, grad)
        value, st = b.step()
        assert st.n_kernels == (3 if apart else 2)
        got.append((value, dy))
    assert got[0][0] == got[1][0]
    assert torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("kind,n,c", [("mse", 300, 16), ("mse", 50000, 128), ("ce", 300, 16), ("ce", 300000, 4), ("ce", 70, 1000), ("ce", 2000, 129), ("ce", 5000, 65)])
def test_gradient_over_the_tensor_it_comes_from(kind, n, c):
    """The gradient bound to the memory of y (or z): the loss of the same pass has the bits it has with a tensor of its own."""
    import torch
    got = []
    for in_place in (False, True):
        b = Built()
        A = b.A
        y = rnd(8, (n, c))
        t = rnd(9, (n, c)) if kind == "mse" else torch.arange(n, dtype=torch.int32, device="cuda") * 7 % c
        vy, vt = b.var("y", y, A.VAR_PARAM), b.var("t", t, A.VAR_TARGET)
        b.op("loss", A.OP_MSE if kind == "mse" else A.OP_SOFTMAX_CE, [vy, vt], phase=A.FWD)
        dy = y if in_place else torch.full_like(y, float("nan"))
        b.op("dy", A.OP_MSE_GRAD if kind == "mse" else A.OP_SOFTMAX_CE_GRAD, [vy, vt], out=dy)
        value, st = b.step()
        assert st.n_kernels == 2
        got.append((value, dy.clone()))
    assert got[0][0] == got[1][0]
    assert torch.equal(got[0][1], got[1][1])


def test_executor_allocates_no_device_memory():
    """A head of 72 classes over a million positions keeps one partial sum a position: 4 MB, which come out of the arena."""
    import torch

    def build(rows):
        b = Built()
        A = b.A
        z, t = rnd(10, (rows, 72)), torch.zeros(rows, dtype=torch.int32, device="cuda")
        vz, vt = b.var("z", z, A.VAR_PARAM), b.var("t", t, A.VAR_TARGET)
        b.op("loss", A.OP_SOFTMAX_CE, [vz, vt], phase=A.FWD)
        b.op("dz", A.OP_SOFTMAX_CE_GRAD, [vz, vt], out=torch.empty_like(z))
        return b

    build(16).step()                                            # code objects are loaded
    b = build(1 << 20)
    need = b.g.memory_need()[1]
    assert need >= 4 << 20
    arena, pool = torch.empty(need, dtype=torch.uint8, device="cuda"), b.L.api.PinnedPool(256)
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    b.ex = b.L.Executor(b.g, arena.data_ptr(), need, pool.ptr, 256, *[s.cuda_stream for s in streams], 0)
    for node, t in b.dev.items():
        b.ex.bind(node, t.data_ptr())
    loss, st = b.ex.step()
    assert before - torch.cuda.mem_get_info()[0] < 3 << 20
    assert st.n_kernels == 2 and abs(loss - 4.28) < 1.0


@pytest.mark.parametrize("kind", ["mse", "ce"])
def test_mask_other_than_the_tensor_itself(kind):
    import torch
    n, c = 333, 24
    b = Built()
    A = b.A
    y, mask = rnd(11, (n, c)), rnd(12, (n, c))
    t = rnd(13, (n, c)) if kind == "mse" else torch.arange(n, dtype=torch.int32, device="cuda") % c
    vy, vt, vm = b.var("y", y, A.VAR_PARAM), b.var("t", t, A.VAR_TARGET), b.var("m", mask, A.VAR_CONST)
    b.op("loss", A.OP_MSE if kind == "mse" else A.OP_SOFTMAX_CE, [vy, vt], phase=A.FWD)
    dy = torch.full_like(y, float("nan"))
    b.op("dy", A.OP_MSE_GRAD if kind == "mse" else A.OP_SOFTMAX_CE_GRAD, [vy, vt, vm], out=dy, flags=A.F_MASK)
    loss, st = b.step()
    yd = y.double()
    if kind == "mse":
        ref, g = float(((yd - t.double()) ** 2).mean()), 2.0 / y.numel() * (yd - t.double())
    else:
        ref = float(torch.nn.functional.cross_entropy(yd, t.long()))
        g = (torch.softmax(yd, -1) - torch.nn.functional.one_hot(t.long(), c)) / n
    g = torch.where(mask > 0, g, torch.zeros_like(g))
    assert st.n_kernels == 2 and abs(loss - ref) <= 1e-5 * abs(ref)
    assert bool(((dy.double() - g).abs() <= 2.0 ** -8 * g.abs() + 1e-6 / n).all())


@pytest.mark.parametrize("first", ["scale", "dot"])
@pytest.mark.parametrize("why", ["second in the arena", "another raw gradient", "control edge"])
def test_affine_gradients_that_run_apart(first, why):
    """The second result in the arena (its block is not there when the first runs), two raw gradients, an operation in between that the
    second waits for: two launches, the same values."""
    import torch
    rows, k, f32 = 80, 24, torch.float32
    b = Built()
    A = b.A
    raw, w, scale = rnd(14, (1, 1, rows, k), f32), rnd(15, (1, 1, rows, k)), rnd(16, (k,), f32)
    vraw, vw, vs = b.var("raw", raw, A.VAR_CONST), b.var("w", w, A.VAR_PARAM), b.var("s", scale, A.VAR_PARAM)
    raw2 = rnd(17, tuple(raw.shape), f32) if why == "another raw gradient" else raw
    vraw2 = b.var("raw2", raw2, A.VAR_CONST) if why == "another raw gradient" else vraw
    outs = {"scale": torch.full_like(raw, float("nan")), "dot": torch.full_like(scale, float("nan"))}
    order = ["scale", "dot"] if first == "scale" else ["dot", "scale"]
    nodes = []
    for i, q in enumerate(order):
        src = vraw if i == 0 else vraw2
        if i == 1 and why == "control edge":
            other = b.op("between", A.OP_SCALE_COLS, [vraw, vs], out=torch.empty_like(raw))
        nodes.append(b.op(q, A.OP_SCALE_COLS if q == "scale" else A.OP_DOT_COLS, [src, vs if q == "scale" else vw],
                          out=None if i == 1 and why == "second in the arena" else outs[q]))
    if why == "control edge":
        b.g.add_control_edge(other, nodes[1])
    _, st = b.step()
    if why == "second in the arena":
        off = b.ex.tensor_ptr(nodes[1]) - b.arena.data_ptr()
        outs[order[1]] = b.arena[off:off + outs[order[1]].numel() * 4].view(f32).view(outs[order[1]].shape)
    by = {order[0]: raw, order[1]: raw2}
    assert torch.equal(outs["scale"], by["scale"] * scale)
    terms = by["dot"].double() * w.double()
    assert bool(((outs["dot"].double() - terms.sum((0, 1, 2))).abs() <= 1e-5 * terms.abs().sum((0, 1, 2))).all())
    if why != "control edge":
        assert st.n_kernels == 2
