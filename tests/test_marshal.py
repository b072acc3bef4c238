"""What the extension takes and refuses for the arguments of the library's calls (no GPU: the calls stop at their own checks or have nothing to do)."""
import ctypes

import pytest
import torch

import paper_2605_11537_amd as moe
from paper_2605_11537_amd import binding


class _OnDevice:
    """Answers as a device tensor does."""
    is_cuda = True

    def __init__(self, contiguous=True):
        self.contiguous = contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return 16


def _combine(y, x=None, T=0, d=8, dtype=0, residual=0, out=None, stream=0):
    return binding._c().moe_combine(y, x, None, None, T, d, dtype, residual, out, stream)


def test_what_a_tensor_may_be():
    assert _combine(None) == 0 and _combine(_OnDevice()) == 0            # an empty batch: nothing is looked at
    for bad in (torch.zeros(8), torch.nn.Parameter(torch.zeros(8)), _OnDevice(contiguous=False), torch.zeros(4, 4).t()):
        with pytest.raises(ValueError, match="device-resident contiguous"):
            _combine(bad)
    for no_tensor in (16, 0, 1.5, "x", [1], object()):                   # an address is none, nor is 0
        with pytest.raises(AttributeError):
            _combine(no_tensor)


def test_ints_and_the_stream():
    assert _combine(None, T=False, residual=True) == 0                   # a bool is an int
    assert _combine(None, T=2 ** 32) == 0 and _combine(None, stream=None) == 0       # taken to 32 bits, as by ctypes
    for bad in (1.0, "1", None, torch.tensor(1)):
        with pytest.raises(TypeError):
            _combine(None, d=bad)
    with pytest.raises(TypeError):
        _combine(None, stream=torch.zeros(1))
    with pytest.raises(TypeError):
        binding._c().moe_combine(None)
    with pytest.raises(TypeError):
        binding._c().moe_layer_forward(*[None] * 44)
    with pytest.raises(ValueError):
        binding._c().bind("no_such_call", 0)


def test_errors_are_the_library_s():
    assert _combine(None, T=1) == -1 and b"moe_combine: null pointer" in moe.lib().moe_last_error()
    w = binding.SruWeightsC(2, 100, 256, 128, 0, None, None, None, None, None, 0)
    assert binding._c().sru_predict(None, ctypes.addressof(w), 1, 8, 1, None, None, None, 0, 0) != 0
    assert b"n_in=100" in moe.lib().moe_last_error()


def test_every_call_is_bound():
    for n in binding.MARSHALLED:
        with pytest.raises(TypeError, match="arguments"):                # bound, and counted
            getattr(binding._c(), n)()
