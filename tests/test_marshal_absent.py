"""A tree without the extension module _torch_marshal, or with one compiled for another torch: the tensor
calls warn once and take binding.py's own code, which needs the library alone."""
import sys
import types

import pytest
import torch

import paper_2603_08343_amd as wht
from paper_2603_08343_amd import binding

NAME = "paper_2603_08343_amd._torch_marshal"


def _other_torch():
    m = types.ModuleType(NAME)
    m.torch_version = "0.0.1"
    m.bind = lambda *args: pytest.fail("a module built for another torch must not be used")
    return m


@pytest.fixture(params=["absent", "built for another torch"])
def unusable(request, monkeypatch):
    module = None if request.param == "absent" else _other_torch()      # None: importing it raises
    monkeypatch.setitem(sys.modules, NAME, module)
    monkeypatch.delattr(wht, "_torch_marshal", raising=False)
    if module is not None:
        monkeypatch.setattr(wht, "_torch_marshal", module, raising=False)
    monkeypatch.setattr(binding, "_native_module", None)


def test_calls_are_declined_after_one_warning(unusable, monkeypatch, recwarn):
    monkeypatch.setattr(binding, "_torch_module", torch)                # as if a GPU had been seen
    for _ in range(2):
        native = binding._native()
        assert native.forward(*[None] * 8) is None and native.backward(*[None] * 10) is None
    assert [w.category for w in recwarn] == [RuntimeWarning]


@pytest.mark.gpu
def test_calls_give_the_same_results(unusable, monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(5)
    x, dy = (torch.empty(6, 256, device="cuda").normal_(generator=g) for _ in range(2))
    a, b = (torch.empty(256, device="cuda").uniform_(0.5, 1.5, generator=g) for _ in range(2))

    def calls():
        return (wht.wht_affine_forward(x, a, b), wht.wht_affine_forward_residual(x, a, b, dy),
                *wht.wht_affine_forward_residual_stats(x, a, b, dy), *wht.wht_affine_backward(dy, x, a),
                *wht.wht_affine_backward_static(dy, x, a))

    with pytest.warns(RuntimeWarning):
        general = calls()
    monkeypatch.undo()                                                  # the module as built
    assert all(torch.equal(p, q) for p, q in zip(general, calls()))
    assert binding._native_module is not binding._NoNative
