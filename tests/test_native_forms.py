"""Which calls the binding's native path takes itself and which it hands to the
general one: a change in what it reads of a tensor would otherwise go unseen,
since both paths give the same outputs."""
import copy
import ctypes
import pickle

import pytest
import torch

import paper_2312_00229_amd as wz
from paper_2312_00229_amd import _lib


class _Tagged(torch.Tensor):
    pass


def _calls(x, dtype=None):
    """Results of the three native calls on x (a gradient of the output's size, outputs of fresh tensors)."""
    address, struct = _lib.lib().address, wz.Params().c()
    p = ctypes.addressof(struct)
    shape = (*x.shape[:-2], 2 * x.shape[-2], 2 * x.shape[-1])
    y = torch.empty(shape, dtype=x.dtype, device=x.device)
    g = torch.ones(shape, device=x.device)
    return (wz._native.zoom2x(address["weno_zoom2x"], p, x, dtype),
            wz._native.zoom2x_(address["weno_zoom2x"], p, x, y),
            wz._native.zoom2x_backward(address["weno_zoom2x_backward"], p, x, g, torch.empty_like(x)))


def test_host_tensors_are_handed_on():
    assert wz._native is not None, "build the package: _native.so is missing"
    for x in (torch.zeros(3, 8, 8), torch.zeros(3, 8, 8, dtype=torch.uint8), torch.nn.Parameter(torch.zeros(8, 8))):
        assert _calls(x) == (None, None, None)


@pytest.mark.gpu
def test_plain_tensors_are_taken(gpu):
    base = torch.rand((2, 3, 20, 24), device="cuda")
    for x in (base[0, 0], base[0], base, base[..., ::2], base[0, 0].t()):
        out, rc, rc_backward = _calls(x)
        assert torch.is_tensor(out) and rc == 0 and rc_backward == 0
    out, rc, rc_backward = _calls((255 * base).byte())
    assert torch.is_tensor(out) and rc == 0 and rc_backward == _lib.WENO_EDTYPE
    assert _calls(base, torch.uint8)[0].dtype == torch.uint8


@pytest.mark.gpu
def test_other_forms_are_handed_on(gpu):
    base = torch.rand((2, 3, 20, 24), device="cuda")
    for x in (base.as_subclass(_Tagged), torch.nn.Parameter(base), base.double()):
        assert _calls(x) == (None, None, None)
    # interleaved channels: an output of their own layout, allocated by the general path
    out, rc, _ = _calls(base.contiguous(memory_format=torch.channels_last))
    assert out is None and rc == 0
    assert _calls(base, torch.float64)[0] is None


@pytest.mark.parametrize("again", [copy.copy, copy.deepcopy, lambda p: pickle.loads(pickle.dumps(p)),
                                   lambda p: _lib.WenoParams(p.beta, p.k_eps, p.h, p.nbw, p.boundary)])
def test_parameters_are_read_where_they_are(monkeypatch, again):
    # a parameter struct of the caller's own, copied, sent between processes or built by hand
    class Own(wz.Params):
        def c(self):
            return struct

    struct = again(wz.Params(beta=1.5).c())
    seen = []

    class Recorder:
        zoom2x = zoom2x_ = zoom2x_backward = staticmethod(lambda fn, params, *a: seen.append(params) or 0)

    monkeypatch.setattr(wz, "_native", Recorder)
    x, y = torch.zeros(4, 4), torch.zeros(8, 8)
    wz.zoom2x(x, Own())
    wz.zoom2x_(x, y, Own())
    wz.zoom2x_backward(x, y, Own())
    assert seen == 3 * [ctypes.addressof(struct)]
