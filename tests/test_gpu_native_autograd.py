"""The differentiable call as a node of torch's C++ autograd (csrc/torch_marshal.cpp, layer()) against the Python Function
that it stands for: values bit for bit, and the same answer -- a result or an error -- for every form of argument, every
combination of wanted gradients and every mode that looks into an autograd function."""
import pytest
import torch

from paper_2603_08343_amd import binding
from paper_2603_08343_amd.autograd import WhtAffine, WhtAffineFunction, wht_affine

pytestmark = pytest.mark.gpu

D = 256


def _tensors(shape=(3, 5, D), dtype=torch.bfloat16, seed=3):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x, r, dy = (torch.empty(*shape, device="cuda", dtype=dtype).normal_(generator=g) for _ in range(3))
    a = torch.empty(shape[-1], device="cuda").uniform_(0.5, 1.5, generator=g)
    b = torch.empty(shape[-1], device="cuda").normal_(generator=g)
    return x, r, dy, a, b


def _flat(out):
    out = out if isinstance(out, (tuple, list)) else (out,)
    return [t if not isinstance(t, torch.Tensor) else (t.dtype, tuple(t.shape), t.requires_grad, t._base is None, t.detach().float().cpu())
            for t in out]


def _outcome(call):
    try:
        out = _flat(call())
        torch.cuda.synchronize()
        return out
    except Exception as e:                                    # compared, not hidden
        text = str(e)
        for node in ("torch::autograd::CppNode<WhtAffineFunction>", "WhtAffineFunctionBackward"):
            text = text.replace(node, "node")
        return type(e), text


def _same(call, monkeypatch, label):
    """call() builds everything it needs: it runs once on each path."""
    print(f"[autograd] {label}", flush=True)
    native = _outcome(call)

    class NoLayer:
        forward, backward = staticmethod(binding._native().forward), staticmethod(binding._native().backward)
        layer = staticmethod(lambda *args: None)

    with monkeypatch.context() as m:
        m.setattr(binding, "_native_module", NoLayer)
        general = _outcome(call)
    if isinstance(general, tuple):
        assert native == general, label
        return
    assert len(native) == len(general), label
    for n, g in zip(native, general):
        if isinstance(n, tuple) and isinstance(n[-1], torch.Tensor):
            assert n[:4] == g[:4] and torch.equal(n[4].nan_to_num(7.0), g[4].nan_to_num(7.0)), label
        else:
            assert n == g, label


def _train(shape=(3, 5, D), dtype=torch.bfloat16, needs=(True, True, True, True), use_resid=True, form=lambda t: t, grad=None):
    x, r, dy, a, b = _tensors(shape, dtype)
    for t, need in zip((x, a, b, r), needs):
        t.requires_grad_(need)
    y = wht_affine(form(x), a, b, form(r) if use_resid else None)
    wanted = [t for t, need in zip((x, a, b, r if use_resid else None), needs) if need and t is not None]
    if not wanted:
        return y
    return (y, *torch.autograd.grad(y, wanted, dy.view(y.shape) if grad is None else grad(dy, y)))


def test_plain_calls_are_taken_and_the_others_declined():
    x, r, dy, a, b = _tensors()
    wht_affine(x, a, b)
    layer = binding._native_module.layer
    p = torch.nn.Parameter(a.clone())
    assert layer(x, p, b, None) is not None and layer(x.clone().requires_grad_(True), p, b, r) is not None
    assert layer(x[0, 0], p, b, None).shape == (D,) and layer(x.float(), p, b, None) is not None
    for args in ((x.transpose(0, 1), p, b, None), (x.cpu(), p, b, None), (x.half(), p, b, None), (x, p[:-4], b, None), (x[:0], p, b, None),
                 (x, p, b, r.float()), (x, p, b, r.view(15, D)), (x, p, b.bfloat16(), None), (None, p, b, None)):
        assert layer(*args) is None
    with torch.autograd.forward_ad.dual_level():
        assert layer(x, p, b, None) is None


@pytest.mark.parametrize("shape,dtype", [((D,), torch.bfloat16), ((7, D), torch.float32), ((1, 1, 1, D), torch.bfloat16), ((3, 67, 768), torch.bfloat16),
                                         ((2, 4099, 64), torch.float32)])
def test_shapes_and_types(shape, dtype, monkeypatch):
    for use_resid in (False, True):
        _same(lambda: _train(shape, dtype, use_resid=use_resid), monkeypatch, f"{shape} {dtype} resid={use_resid}")


def test_every_combination_of_gradients(monkeypatch):
    for bits in range(16):
        needs = tuple(bool(bits >> i & 1) for i in range(4))
        _same(lambda: _train(needs=needs), monkeypatch, f"needs={needs}")
        _same(lambda: _train(needs=needs, use_resid=False), monkeypatch, f"needs={needs}, no residual")


def test_forms_of_input_and_gradient(monkeypatch):
    forms = {"transposed": lambda t: t.transpose(0, 1), "strided": lambda t: torch.cat((t, t), -1)[..., :D], "float": lambda t: t.float(),
             "half": lambda t: t.half(), "cpu": lambda t: t.cpu(), "narrow": lambda t: t[..., :24].contiguous(), "no rows": lambda t: t[:0],
             "shifted": lambda t: torch.cat((t.new_zeros(4), t.reshape(-1)))[4:].view(t.shape), "parameter": torch.nn.Parameter,
             "flat": lambda t: t.reshape(-1, D)}
    for name, form in forms.items():
        # a parameter or a slice is not what the gradient is asked for: values only
        _same(lambda: _train(needs=(False,) * 4, form=form), monkeypatch, f"form {name}")
    for name in ("transposed", "strided", "flat"):
        _same(lambda: _train(form=forms[name], grad=lambda dy, y: torch.ones_like(y)), monkeypatch, f"gradient through {name}")
    _same(lambda: _train(grad=lambda dy, y: dy[:, :1].expand_as(y)), monkeypatch, "expanded gradient")
    _same(lambda: _train(grad=lambda dy, y: dy.transpose(0, 1).contiguous().transpose(0, 1)), monkeypatch, "transposed gradient")
    _same(lambda: _train(grad=lambda dy, y: dy.float()), monkeypatch, "float32 gradient of a bfloat16 result")
    _same(lambda: _train(grad=lambda dy, y: torch.cat((dy.new_zeros(4), dy.reshape(-1)))[4:].view(dy.shape)), monkeypatch, "misaligned gradient")


def test_graph_semantics(monkeypatch):
    def double_backward():
        x, r, dy, a, b = _tensors()
        x.requires_grad_(True), r.requires_grad_(True), a.requires_grad_(True), dy.requires_grad_(True)
        y = wht_affine(x, a, b, r)
        g = torch.autograd.grad(y, (x, a, r), dy, create_graph=True)
        return (*g, *torch.autograd.grad(g[2].sum(), (dy,), allow_unused=True))

    def twice(retain):
        x, r, dy, a, b = _tensors()
        x.requires_grad_(True)
        y = wht_affine(x, a, b)
        return (*torch.autograd.grad(y, x, dy, retain_graph=retain), *torch.autograd.grad(y, x, dy))

    def saved_then_changed():
        x, r, dy, a, b = _tensors()
        a.requires_grad_(True)
        y = wht_affine(x, a, b)
        x.add_(1.0)
        return torch.autograd.grad(y, a, dy)

    def result_changed(kind):
        x, r, dy, a, b = _tensors()
        a.requires_grad_(True)
        y = wht_affine(x, a, b)
        if kind == "add":
            y.add_(1.0)
        elif kind == "row":
            y[0].zero_()
        return (y, *torch.autograd.grad(y, a, dy))

    def part():
        x, r, dy, a, b = _tensors()
        for t in (x, a, b):
            t.requires_grad_(True)
        y = wht_affine(x, a, b)
        return (*torch.autograd.grad(y, b, dy, retain_graph=True), *torch.autograd.grad(y, x, dy, retain_graph=True), *torch.autograd.grad(y, a, dy))

    _same(double_backward, monkeypatch, "double backward")
    _same(lambda: twice(True), monkeypatch, "retained graph")
    _same(lambda: twice(False), monkeypatch, "freed graph")
    _same(saved_then_changed, monkeypatch, "saved input changed in place")
    for kind in ("none", "add", "row"):
        _same(lambda: result_changed(kind), monkeypatch, f"result changed in place: {kind}")
    _same(part, monkeypatch, "one gradient at a time")


def test_modes_hooks_and_transforms(monkeypatch):
    x, r, dy, a, b = _tensors()

    def under(ctx):
        with ctx:
            return _train()

    def hooks():
        seen = []
        with torch.autograd.graph.saved_tensors_hooks(lambda t: seen.append((tuple(t.shape), t.dtype)) or t.cpu(), lambda t: t.cuda()):
            out = _train()
        return (*out, tuple(seen))

    def checkpointed():
        x, r, dy, a, b = _tensors()
        x.requires_grad_(True), a.requires_grad_(True)
        y = torch.utils.checkpoint.checkpoint(lambda t: wht_affine(t, a, b), x, use_reentrant=False)
        return (y, *torch.autograd.grad(y, (x, a), dy))

    def forward_mode():
        with torch.autograd.forward_ad.dual_level():
            return wht_affine(torch.autograd.forward_ad.make_dual(x, dy), a, b)

    def no_grad():
        with torch.no_grad():
            return wht_affine(x, a.clone().requires_grad_(True), b, r)

    def inference():
        with torch.inference_mode():
            y = wht_affine(x, a, b, r)
            return y, y.is_inference()

    def inference_saved():
        with torch.inference_mode():
            t = x.clone()
        return wht_affine(t, a.clone().requires_grad_(True), b)

    def side_stream():
        side, fill = torch.cuda.Stream(), torch.empty(1 << 28, device="cuda")
        late = torch.zeros_like(x)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            fill.zero_()
            late.copy_(x)
            late.requires_grad_(True)
            y = wht_affine(late, a, b)
            out = (y, *torch.autograd.grad(y, late, dy))
        torch.cuda.synchronize()
        return out

    _same(hooks, monkeypatch, "saved tensor hooks")
    _same(checkpointed, monkeypatch, "checkpoint")
    _same(lambda: under(torch.autocast("cuda", dtype=torch.bfloat16)), monkeypatch, "autocast")
    _same(lambda: under(torch.autograd.detect_anomaly(check_nan=False)), monkeypatch, "anomaly mode")
    _same(lambda: under(torch.overrides.TorchFunctionMode()), monkeypatch, "function mode")
    _same(forward_mode, monkeypatch, "forward mode")
    _same(no_grad, monkeypatch, "no_grad")
    _same(inference, monkeypatch, "inference mode")
    _same(inference_saved, monkeypatch, "inference tensor to be saved")
    _same(side_stream, monkeypatch, "side stream")
    _same(lambda: torch.vmap(lambda t: wht_affine(t, a, b))(x), monkeypatch, "vmap")
    _same(lambda: torch.vmap(lambda s: wht_affine(x, a, b) * s)(torch.ones(2, device="cuda", dtype=x.dtype)), monkeypatch, "vmap, captured tensors")
    _same(lambda: torch.func.grad(lambda t: wht_affine(x, t, b).float().sum())(a), monkeypatch, "func.grad")
    _same(lambda: torch.func.jvp(lambda t: wht_affine(x, t, b), (a,), (b,)), monkeypatch, "func.jvp")


def test_module_and_threads():
    """Backward passes of several graphs at once: each on its own tensors, all equal to the Python Function's."""
    import concurrent.futures
    x, r, dy, a, b = _tensors((64, D))
    ref_y = WhtAffineFunction.apply(x, a.requires_grad_(True), b, r)
    ref = torch.autograd.grad(ref_y, a, dy)[0]
    layer = WhtAffine(D, device="cuda")
    with torch.no_grad():
        layer.alpha.copy_(a)
        layer.beta.copy_(b)

    def one(_):
        for _ in range(20):
            y = layer(x, r)
            g, = torch.autograd.grad(y, layer.alpha, dy)
            if not (torch.equal(y, ref_y) and torch.equal(g, ref)):
                return False
        return True

    with concurrent.futures.ThreadPoolExecutor(4) as pool:
        assert all(pool.map(one, range(8)))


def test_compiled_autograd_of_a_graph_built_eagerly():
    """The backward pass under torch's compiled autograd: it breaks its graph at the node, as it does inside the Python Function,
    and gets the gradients of the eager backward pass, bit for bit, on either path."""
    compiled_autograd = pytest.importorskip("torch._dynamo.compiled_autograd")
    x, _, dy, a, b = _tensors((7, 1024))

    def grads(call, compiled):
        leaves = [t.clone().requires_grad_(True) for t in (x, a, b)]
        y = call(leaves[0] * 2, leaves[1], leaves[2], None)
        if compiled:
            with compiled_autograd._enable(torch.compile(backend="eager")):
                y.backward(dy)
        else:
            y.backward(dy)
        return [t.grad for t in leaves]

    for name, call in (("node", wht_affine), ("Function", WhtAffineFunction.apply)):
        print(f"[autograd] compiled autograd, {name}", flush=True)
        assert all(torch.equal(p, q) for p, q in zip(grads(call, True), grads(call, False))), name
