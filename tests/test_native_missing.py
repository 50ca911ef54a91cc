"""Without the torch extension the hot entry points go through ctypes, as all others do, and say so once."""
import sys
import warnings

import pytest

import paper_2210_03858_amd
from paper_2210_03858_amd import binding as B


@pytest.fixture
def no_extension(monkeypatch):
    monkeypatch.setattr(B, "_native", None)
    monkeypatch.delattr(paper_2210_03858_amd, "_bcq_torch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2210_03858_amd._bcq_torch", None)


def test_missing_extension_warns_once(no_extension):
    with pytest.warns(RuntimeWarning, match="_bcq_torch.so"):
        assert B._try_native("linear") is None
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert B._try_native("fwd_grouped") is None
    with pytest.raises(RuntimeError, match="_bcq_torch.so"):
        B.native()


@pytest.mark.gpu
@pytest.mark.filterwarnings("ignore:_bcq_torch")
def test_layer_without_extension(no_extension):
    import torch
    from paper_2210_03858_amd.autograd import BCQLinear
    layer = BCQLinear.from_weight(torch.randn((96, 256), device="cuda"), 2, q_train=1)
    x = torch.randn((40, 256), device="cuda").bfloat16().requires_grad_(True)
    wanted = (x, layer.alpha_train)
    y = layer(x)
    got = (y,) + torch.autograd.grad(y, wanted, torch.ones_like(y))
    B._native = None
    del sys.modules["paper_2210_03858_amd._bcq_torch"]
    assert B.native()
    y = layer(x)
    for a, b in zip(got, (y,) + torch.autograd.grad(y, wanted, torch.ones_like(y))):
        assert torch.equal(a, b)
