"""What the extension takes and refuses for the arguments of the library's calls (no GPU: the calls stop at their own checks or have nothing to do)."""
import ctypes
import importlib

import numpy as np
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


class _Whole:
    """A whole number of no type that is known."""

    def __index__(self):
        return 8


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
    for whole in (np.int64(8), np.uint8(8), torch.tensor(8), _Whole()):  # as any whole number is
        assert _combine(None, d=whole) == 0
    for bad in (1.0, "1", None, np.float32(8), torch.tensor(8.0), torch.tensor([8, 8])):
        with pytest.raises(TypeError):
            _combine(None, d=bad)
    for no_address in (torch.zeros(1), np.int64(16), _Whole(), 1.5):
        with pytest.raises(TypeError):
            _combine(None, stream=no_address)
    with pytest.raises(TypeError):
        binding._c().moe_combine(None)
    with pytest.raises(TypeError):
        binding._c().moe_layer_forward(*[None] * 44)
    with pytest.raises(ValueError):
        binding._c().bind("no_such_call", 0)


INT_FIELDS = ("T", "n_plan", "top_k", "renormalize", "d", "F", "router_E", "E", "budget", "slot_capacity", "policy", "dtype", "router_layout",
              "weight_layout", "schedule", "residual")
SIZE_FIELDS = ("route_ws_bytes", "front_ws_bytes", "ffn_ws_bytes")


def _layer(**fields):
    """top_k = -1: the call stops at its first check, whose message names T and top_k."""
    values = {**dict.fromkeys(SIZE_FIELDS, 0), **dict.fromkeys(INT_FIELDS, 1), "top_k": -1, **fields}
    return binding._c().moe_layer_forward(*[None] * 25, *values.values(), 0)


@pytest.mark.parametrize("name", INT_FIELDS + SIZE_FIELDS)
def test_the_fields_of_a_layer_keep_their_value(name):
    """A field takes any whole number that fits it, and none that would become another one."""
    size = name in SIZE_FIELDS
    lowest, highest = (0, 2 ** 64 - 1) if size else (-2 ** 31, 2 ** 31 - 1)
    for bad in (lowest - 1, highest + 1, 2 ** 32 + 4 if not size else 2 ** 64 + 4, 2 ** 70, -2 ** 70):
        with pytest.raises(OverflowError):
            _layer(**{name: bad})
    for bad in (1.0, "1", None, np.float64(1), torch.tensor(1.0)):
        with pytest.raises(TypeError):
            _layer(**{name: bad})
    one = -1 if name == "top_k" else 1
    for fits in (one, np.int64(one), np.int16(one), torch.tensor(one)):
        assert _layer(**{name: fits}) == -1 and b"T=1 top_k=-1 out of range" in moe.lib().moe_last_error()
    if name != "top_k":
        assert _layer(**{name: highest}) == -1 and _layer(**{name: lowest}) == -1
    else:
        assert _layer(top_k=lowest) == -1 and b"top_k=-2147483648 " in moe.lib().moe_last_error()
    assert _layer(T=np.int64(2 ** 31 - 1)) == -1 and b"T=2147483647 " in moe.lib().moe_last_error()


def test_errors_are_the_library_s():
    assert _combine(None, T=1) == -1 and b"moe_combine: null pointer" in moe.lib().moe_last_error()
    w = binding.SruWeightsC(2, 100, 256, 128, 0, None, None, None, None, None, 0)
    assert binding._c().sru_predict(None, ctypes.addressof(w), 1, 8, 1, None, None, None, 0, 0) != 0
    assert b"n_in=100" in moe.lib().moe_last_error()


def test_every_call_is_bound():
    for n in binding.MARSHALLED:
        with pytest.raises(TypeError, match="arguments"):                # bound, and counted
            getattr(binding._c(), n)()


@pytest.fixture
def unloaded(monkeypatch):
    """The binding as in a process that has not loaded the library."""
    moe.lib()
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_calls", None)


@pytest.mark.parametrize("other", ["torch", "python", "none"])
def test_an_extension_of_another_torch_or_python_is_refused(unloaded, monkeypatch, other):
    """It reads torch's objects by the layout that its headers gave them."""
    if other == "torch":
        monkeypatch.setattr(torch.version, "git_version", "0" * 40)
    elif other == "python":
        monkeypatch.setattr("sys.hexversion", 0x030900F0)
    else:
        monkeypatch.delattr(importlib.import_module("paper_2605_11537_amd._marshal"), "built_for", raising=False)
    with pytest.raises(RuntimeError, match="rebuild"):
        moe.lib()
    assert binding._lib is None and binding._calls is None
    monkeypatch.undo()
    assert moe.lib() is not None
