"""What the binding asks of the machine it runs on: libmesa.so and ctypes.  The native marshalling is an extension of one
Python version that looks up two functions of a torch with devices; where it cannot be had, every call takes the general path."""
import pytest
import torch

from paper_2111_11124_amd import _ffi


@pytest.fixture()
def fresh(monkeypatch):
    monkeypatch.setattr(_ffi, "_lib", None)
    monkeypatch.setattr(_ffi, "_fast", None)
    return monkeypatch


def _usable():
    assert _ffi.workspace_bytes(_ffi.OP_UPDATE_RUNNING_PARAMS, 4, 3, 64) > 0        # a size query needs no device
    assert _ffi.conv2d_dw_q_workspace_bytes(_ffi.Conv2d(2, 3, 8, 8, 4, 3, 3, 1, 1, 1, 1, 1, 1)) > 0
    a, q = torch.ones(1), torch.zeros(64, dtype=torch.int8)
    with pytest.raises(ValueError, match="device tensors"):                         # and a call is judged as ever
        _ffi.mesa_quantize_headwise(torch.zeros(64), (1, 1, 64), a, a, q)


def test_the_extension_of_this_python_is_the_one_that_is_loaded(fresh):
    assert _ffi._FAST_PATH.exists() and _ffi._FAST_PATH.name not in ("_marshal.so", "_marshal.abi3.so")
    assert not isinstance(_ffi._load_fast(), _ffi._General)
    _usable()


def test_without_the_extension(fresh, tmp_path):
    fresh.setattr(_ffi, "_FAST_PATH", tmp_path / "_marshal.so")
    _usable()
    assert isinstance(_ffi._fast, _ffi._General)


def test_with_an_extension_that_cannot_be_loaded(fresh, tmp_path):
    (tmp_path / "_marshal.so").write_bytes(b"of another machine")
    fresh.setattr(_ffi, "_FAST_PATH", tmp_path / "_marshal.so")
    _usable()
    assert isinstance(_ffi._fast, _ffi._General)


@pytest.mark.parametrize("name", ["_cuda_getDevice", "_cuda_getCurrentRawStream"])
def test_on_a_torch_without_device_functions(fresh, name):
    fresh.delattr(torch._C, name, raising=False)
    _usable()
    assert isinstance(_ffi._fast, _ffi._General)
