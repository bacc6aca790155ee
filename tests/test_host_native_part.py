"""The binding's native part (_host_calls.so) is a shorter way to the library and may be missing.  No GPU: the calls
here are refused by the general path's own checks, which shows that it took them."""
import ctypes
import sys

import pytest
import torch

import paper_2512_10411_amd
from paper_2512_10411_amd import binding


@pytest.fixture
def first_call(monkeypatch):
    """The binding as before its first call with tensors, restored afterwards."""
    monkeypatch.setattr(binding, "torch", None)
    monkeypatch.setattr(binding, "_host", None)


def refused_by_the_general_path():
    x = torch.zeros(1, 2, 8, 128, dtype=torch.bfloat16)
    lens = torch.tensor([8], dtype=torch.int32)
    for call in (lambda: binding.swaa_attn_fwd(x, x, x, 4, 0), lambda: binding.swaa_attn_fwd_fa_decode(x, x, x, 4, 0, 2),
                 lambda: binding.swaa_attn_decode(x, x, x, 4, 0), lambda: binding.swaa_attn_decode_ex(x, x, x, 4, 0, seq_lens=lens),
                 lambda: binding.swaa_attn_fwd_ex(x, x, x, 4, 0)):
        with pytest.raises(ValueError, match="GPU"):
            call()
    assert binding._host is binding._NoHostCalls


def test_the_library_alone_is_enough(first_call, monkeypatch, tmp_path, recwarn):
    monkeypatch.setattr(binding, "HOST_CALLS_PATH", str(tmp_path / "_host_calls.so"))
    refused_by_the_general_path()
    assert not recwarn.list


def test_a_missing_library_is_reported_behind_a_calls_own_mistakes(first_call, monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "libswaa.so"))
    monkeypatch.setattr(binding, "_lib", None)
    refused_by_the_general_path()


def test_a_native_part_that_does_not_load_is_left_out(first_call, monkeypatch):
    monkeypatch.delattr(paper_2512_10411_amd, "_host_calls", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2512_10411_amd._host_calls", None)  # (as if built against another torch)
    with pytest.warns(RuntimeWarning, match="paper_2512_10411_amd.build"):
        refused_by_the_general_path()


def test_the_native_part_that_is_built_is_bound(first_call, recwarn):
    assert binding._torch() is torch
    assert binding._host.__name__ == "paper_2512_10411_amd._host_calls"
    assert not recwarn.list


@pytest.mark.parametrize("other", ["forward arguments", "decode arguments", "library", "torch"])
def test_a_native_part_compiled_for_another_layout_or_torch_is_left_out(first_call, monkeypatch, other):
    for name, block in (("forward arguments", "SwaaFwdArgs"), ("decode arguments", "SwaaDecodeArgs")):
        if other == name:  # (a field more than the native part knows of)
            old = getattr(binding, block)
            monkeypatch.setattr(binding, block, type(block, (ctypes.Structure,), {"_fields_": old._fields_ + [("more", ctypes.c_void_p)]}))
    if other == "library":
        lib = binding.load_library()
        version = lib.swaa_version()
        monkeypatch.setattr(lib, "swaa_version", lambda: version + 1)
    if other == "torch":
        monkeypatch.setattr(torch, "__version__", "1.13.1")
    with pytest.warns(RuntimeWarning, match="compiled for"):
        binding._torch()
    assert binding._host is binding._NoHostCalls


def test_an_older_native_part_is_left_out(first_call, monkeypatch):
    def bind(*args):
        raise TypeError("bind takes six addresses and two functions")
    binding._torch()
    monkeypatch.setattr(binding._host, "bind", bind)
    monkeypatch.setattr(binding, "torch", None)
    with pytest.warns(RuntimeWarning, match="paper_2512_10411_amd.build"):
        refused_by_the_general_path()
