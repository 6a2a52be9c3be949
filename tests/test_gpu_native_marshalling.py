"""The tensor calls' native marshalling (csrc/torch_marshal.cpp) against binding.py's own code: what the
one hands on, refuses or returns has to be what the other does, for every form of argument."""
import pytest
import torch

import paper_2603_08343_amd as wht
from paper_2603_08343_amd import binding

pytestmark = pytest.mark.gpu

N, D = 6, 256


class _Declines:
    """Stands in for the extension module: sends every call to binding.py's code."""
    forward = backward = staticmethod(lambda *args: None)


def _args():
    g = torch.Generator(device="cuda").manual_seed(3)
    x, dy, r = (torch.empty(N, D, device="cuda", dtype=torch.bfloat16).normal_(generator=g) for _ in range(3))
    a = torch.empty(D, device="cuda").uniform_(0.5, 1.5, generator=g)
    b = torch.empty(D, device="cuda").normal_(generator=g)
    return x, dy, r, a, b


class _Sub(torch.Tensor):
    pass


def _io_forms(t):
    """(label, tensor) pairs: accepted and refused forms of an [N,d] argument."""
    wide = torch.zeros(N, 2 * D, device="cuda", dtype=t.dtype)
    yield "plain", t
    yield "subclass", t.as_subclass(_Sub)
    yield "parameter", torch.nn.Parameter(t.clone())
    yield "requires grad", t.clone().requires_grad_(True)
    yield "shifted by 8 bytes", torch.zeros(N * D + 4, device="cuda", dtype=t.dtype)[4:].view(N, D)
    yield "row stride", wide[:, :D]
    yield "transposed", t.t().contiguous().t()
    yield "one dimension", t.reshape(-1)
    yield "three dimensions", t.view(1, N, D)
    yield "no rows", t[:0]
    yield "narrow", t[:, :24].contiguous()
    yield "half", t.half()
    yield "float32", t.float()
    yield "cpu", t.cpu()
    yield "numpy", t.float().cpu().numpy()
    yield "none", None


def _outcome(call):
    try:
        out = call()
        torch.cuda.synchronize()
    except Exception as e:                                    # compared, not hidden
        return type(e), str(e)
    out = out if isinstance(out, tuple) else (out,)
    return [None if t is None else (t.dtype, tuple(t.shape), t.requires_grad, t.detach().float().cpu()) for t in out]


def _same(call, monkeypatch, label):
    native = _outcome(call)
    with monkeypatch.context() as m:
        m.setattr(binding, "_native_module", _Declines)
        general = _outcome(call)
    if isinstance(general, tuple):
        assert native == general, label
        return
    assert len(native) == len(general), label
    for n, g in zip(native, general):
        assert (n is None) == (g is None), label
        if n is not None:
            assert n[:3] == g[:3] and torch.equal(n[3].nan_to_num(7.0), g[3].nan_to_num(7.0)), label


def test_plain_calls_are_taken():
    x, dy, r, a, b = _args()
    wht.wht_affine_forward(x, a, b)
    native = binding._native_module
    a_param = torch.nn.Parameter(a.clone())
    for t in (x, x.clone().requires_grad_(True), x.float()):
        assert native.forward(t, a_param, b, None, None, None, False, False) is not None
    assert native.forward(x, a, b, r, torch.empty_like(x), torch.empty(N, device="cuda"), True, True) is not None
    assert native.backward(dy, x, a, None, None, None, None, True, True, False) is not None
    assert native.backward(dy, None, a, None, None, None, None, True, False, False) is not None
    with torch.no_grad(), torch.autocast("cuda"):
        assert native.forward(x, a, b, None, None, None, False, False) is not None
    assert native.forward(x[:0], a, b, None, None, None, False, False) is None


def test_forward_calls(monkeypatch):
    x, dy, r, a, b = _args()
    wht.wht_affine_forward(x, a, b)
    for label, t in _io_forms(x):
        print(f"[marshal] forward {label}", flush=True)
        _same(lambda: wht.wht_affine_forward(t, a, b), monkeypatch, f"x {label}")
        _same(lambda: wht.wht_affine_forward_residual(x, a, b, t), monkeypatch, f"resid {label}")
        _same(lambda: wht.wht_affine_forward_residual_stats(t, a, b, r), monkeypatch, f"stats x {label}")
        if label != "none":
            out = t.clone() if isinstance(t, torch.Tensor) else t
            _same(lambda: wht.wht_affine_forward(x, a, b, y=out), monkeypatch, f"y {label}")
    for label, p in (("parameter", torch.nn.Parameter(a.clone())), ("bf16", a.bfloat16()), ("short", a[:-4]),
                     ("strided", torch.zeros(2 * D, device="cuda")[::2]), ("cpu", a.cpu()), ("column", a.view(D, 1)),
                     ("shifted", torch.zeros(D + 1, device="cuda")[1:]), ("none", None)):
        print(f"[marshal] alpha, beta, sumsq {label}", flush=True)
        _same(lambda: wht.wht_affine_forward(x, p, b), monkeypatch, f"alpha {label}")
        _same(lambda: wht.wht_affine_forward(x, a, p), monkeypatch, f"beta {label}")
    for label, q in (("given", torch.empty(N, device="cuda")), ("long", torch.empty(N + 1, device="cuda")),
                     ("bf16", torch.empty(N, device="cuda", dtype=torch.bfloat16)), ("none", None)):
        _same(lambda: wht.wht_affine_forward_residual_stats(x, a, b, r, sumsq=q), monkeypatch, f"sumsq {label}")
    y = torch.empty_like(x)
    assert wht.wht_affine_forward(x, a, b, y=y) is y


def test_backward_calls(monkeypatch):
    x, dy, r, a, b = _args()
    for label, t in _io_forms(dy):
        print(f"[marshal] backward {label}", flush=True)
        _same(lambda: wht.wht_affine_backward(t, x, a), monkeypatch, f"dy {label}")
        _same(lambda: wht.wht_affine_backward(dy, t, a), monkeypatch, f"x {label}")
        _same(lambda: wht.wht_affine_backward(dy, t, a, want_param_grads=False), monkeypatch, f"frozen x {label}")
        _same(lambda: wht.wht_affine_backward_static(dy, t, a), monkeypatch, f"static x {label}")
        if label != "none":
            out = t.clone() if isinstance(t, torch.Tensor) else t
            _same(lambda: wht.wht_affine_backward(dy, x, a, dx=out), monkeypatch, f"dx {label}")
    need = wht.wht_affine_backward_workspace_bytes(N, D, wht.DTYPE_BF16)
    for label, w in (("bytes", torch.empty(need, dtype=torch.uint8, device="cuda")), ("small", torch.empty(need - 16, dtype=torch.uint8, device="cuda")),
                     ("floats", torch.empty(need // 4, device="cuda")), ("cpu", torch.empty(need, dtype=torch.uint8))):
        _same(lambda: wht.wht_affine_backward(dy, x, a, workspace=w), monkeypatch, f"workspace {label}")
    for want in ((True, True), (True, False), (False, True), (False, False)):
        _same(lambda: wht.wht_affine_backward(dy, x, a, want_dx=want[0], want_param_grads=want[1]), monkeypatch, f"want {want}")
    dx, da, db = torch.empty_like(dy), torch.empty_like(a), torch.empty_like(a)
    out = wht.wht_affine_backward(dy, x, a, dx=dx, dalpha=da, dbeta=db)
    assert out[0] is dx and out[1] is da and out[2] is db


def test_streams_modes_and_wrapped_tensors(monkeypatch):
    x, dy, r, a, b = _args()
    ref = wht.wht_affine_forward(x, a, b)
    side = torch.cuda.Stream()
    # the current stream is the one the call goes to: there x gets its values only after a long fill, so a
    # call on any other stream would read zeros
    late, fill = torch.zeros_like(x), torch.empty(1 << 29, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        fill.zero_()
        fill.add_(1.0)
        late.copy_(x)
        y = wht.wht_affine_forward(late, a, b)
    torch.cuda.synchronize()
    assert torch.equal(y, ref) and torch.equal(wht.wht_affine_forward(x, a, b, stream=side), ref)
    # a batched tensor (vmap) has no address: refused by both
    _same(lambda: torch.vmap(lambda t: wht.wht_affine_forward(t, a, b))(x.view(1, N, D)), monkeypatch, "vmap")

    seen = []

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    with Mode():                                              # allocations stay visible to a function mode
        wht.wht_affine_forward(x, a, b)
    assert torch.empty_like in seen
