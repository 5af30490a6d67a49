"""Argument marshalling of the extension module behind the binding (no GPU: the calls are refused on the host)."""
import ctypes
import sys

import numpy as np
import pytest
import torch

import paper_2402_06262_amd as roco
from paper_2402_06262_amd import binding

EINVAL, EWORKSPACE = -1, -3
P = roco.RocoParams(4, 64, 128, 16, roco.ROCO_F32)


def _decode(params=P, q=0x1000, ws=0x1000, workspace_bytes=0, stream=0, **kw):
    a = dict(k_new=0x1000, v_new=0x1000, qpos=0x1000, K_cache=0x1000, V_cache=0x1000, stats=0x1000, pos=0x1000, n_used=0x1000,
             next_slot=0x1000, out=0x1000, evicted_slot=None, evicted_pos=None)
    a.update(kw)
    roco.roco_decode_step(params, q, workspace=ws, workspace_bytes=workspace_bytes, stream=stream, **a)


def _code(call, *a, **k):
    with pytest.raises(roco.RocoError) as e:
        call(*a, **k)
    return e.value.code


def test_addresses_none_and_sizes_reach_the_library():
    assert _code(_decode) == EWORKSPACE                      # everything valid but the workspace's size
    assert _code(_decode, q=None) == EINVAL
    assert _code(_decode, q=0x1001) == EINVAL                # misaligned
    assert _code(_decode, workspace_bytes=np.int64(5)) == EWORKSPACE
    assert _code(_decode, params=roco.RocoParams(0, 64, 128, 16, roco.ROCO_F32)) == EINVAL
    need = roco.decode_workspace_bytes(P)
    assert _code(_decode, workspace_bytes=need - 1, ws=torch.empty(need, dtype=torch.uint8)) in (EWORKSPACE, EINVAL)


def test_a_tensor_is_its_address_and_its_bytes():
    small = torch.empty(64, dtype=torch.float32)
    assert _code(_decode, q=small, ws=small, workspace_bytes=None) == EWORKSPACE
    assert _code(_decode, q=small, ws=torch.nn.Parameter(small), workspace_bytes=None) == EWORKSPACE
    assert _code(_decode, q=small.view(torch.uint8)[1:17], ws=small, workspace_bytes=None) == EINVAL  # its storage offset counts

    class Sub(torch.Tensor):
        pass

    assert _code(_decode, q=small.as_subclass(Sub), ws=small, workspace_bytes=None) == EWORKSPACE


def test_what_is_refused_stays_refused():
    with pytest.raises(ValueError, match="contiguous"):
        _decode(q=torch.empty(8, 8).t())
    with pytest.raises(AttributeError):
        _decode(q="address")
    with pytest.raises(AttributeError):
        _decode(workspace_bytes=None)                        # an address has no size
    with pytest.raises(TypeError):
        _decode(params=7)
    with pytest.raises(TypeError):
        roco.roco_decode_step(P, 1)


@pytest.mark.parametrize("call,n", [("roco_encode_block", 1), ("roco_decode_step_gqa", 1), ("roco_encode_block_gqa", 2)])
def test_steps_of_many(call, n):
    fn = getattr(roco, call)
    args = [0x1000] * 14
    assert _code(fn, P, *[4] * n, *args, workspace_bytes=0, stream=0) == EWORKSPACE
    assert _code(fn, P, *[0] * n, *args, workspace_bytes=0, stream=0) == EINVAL
    assert _code(fn, P, *[np.int32(4)] * n, *args[:-1], torch.empty(16), stream=0) in (EINVAL, EWORKSPACE)


def test_prompts_and_the_static_step():
    a = [0x1000] * 8
    assert _code(roco.roco_prefill_compress, P, *[0x1000] * 4, 64, *a, workspace_bytes=0, stream=0) == EWORKSPACE
    assert _code(roco.roco_prefill_compress, P, *[0x1000] * 4, 0, *a, workspace_bytes=0, stream=0) == EINVAL
    assert _code(roco.roco_prefill_compress_gqa, P, 2, *[0x1000] * 4, 64, *a, workspace_bytes=0, stream=0) == EWORKSPACE
    assert _code(roco.roco_prefill_compress_lse, P, 2, *[0x1000] * 4, 64, *a, workspace_bytes=0, stream=0) == EWORKSPACE
    assert _code(roco.roco_prefill_compress_lse, P, 2, *[0x1000] * 4, 64, None, *a[1:], workspace_bytes=0, stream=0) == EINVAL
    assert _code(roco.roco_decode_step_static, P, *[0x1000] * 10, None, None, None, stream=0) == EINVAL  # no output


def test_the_extension_follows_the_loaded_library(monkeypatch):
    before = binding._calls()
    monkeypatch.setattr(binding, "_lib", None)
    assert binding._calls() is before and binding._native_lib is binding._lib is roco.load_library()
    assert ctypes.sizeof(roco.RocoParams) == 44


@pytest.mark.parametrize("check", [test_addresses_none_and_sizes_reach_the_library, test_a_tensor_is_its_address_and_its_bytes,
                                   test_what_is_refused_stays_refused, test_prompts_and_the_static_step])
def test_a_tree_without_the_extension(monkeypatch, check):
    """Only the library is built: the same calls by ctypes alone."""
    monkeypatch.setattr(binding, "_NATIVE_NAME", "_not_built")
    monkeypatch.setattr(binding, "_native_lib", None)
    monkeypatch.setattr(binding, "_marshal", None, raising=False)
    check()
    assert isinstance(binding._marshal, binding._PlainCalls)


@pytest.mark.parametrize("call,n", [("roco_encode_block", 1), ("roco_decode_step_gqa", 1), ("roco_encode_block_gqa", 2)])
def test_steps_of_many_without_the_extension(monkeypatch, call, n):
    monkeypatch.setattr(binding, "_native_lib", None)
    monkeypatch.setattr(binding, "_marshal", None, raising=False)
    monkeypatch.setitem(sys.modules, "torch", None)  # plain addresses need no PyTorch
    args = [0x1000] * 14
    assert _code(getattr(roco, call), P, *[4] * n, *args, workspace_bytes=0, stream=0) == EWORKSPACE
    assert _code(getattr(roco, call), P, *[0] * n, *args, workspace_bytes=0, stream=0) == EINVAL
    assert isinstance(binding._marshal, binding._PlainCalls)


class _MoreParams(roco.RocoParams):
    _fields_ = [("layer", ctypes.c_int32)]


def test_parameters_are_the_structure_or_one_derived_from_it():
    assert _code(_decode, params=_MoreParams(4, 64, 128, 16, roco.ROCO_F32)) == EWORKSPACE
    for other in (bytes(44), bytearray(44), np.zeros(11, np.int32), (ctypes.c_int32 * 11)(), ctypes.pointer(P), None):
        with pytest.raises(TypeError):
            _decode(params=other)


def test_integers_have_the_width_of_their_arguments():
    """Beyond it they wrap, as in a C call: a size from 2^63 on is a size, 2^32 + 64 tokens are 64."""
    assert _code(_decode, q=None, workspace_bytes=2 ** 64 - 1) == EINVAL
    assert _code(_decode, q=None, workspace_bytes=-1) == EINVAL
    assert _code(_decode, workspace_bytes=2 ** 64) == EWORKSPACE
    assert _code(roco.roco_prefill_compress, P, *[0x1000] * 4, 2 ** 72 + 64, *[0x1000] * 8, workspace_bytes=0, stream=0) == EWORKSPACE

    class Sized:
        nbytes = np.int64(5)

        def is_contiguous(self):
            return True

        def data_ptr(self):
            return 0x1000

    assert _code(_decode, ws=Sized(), workspace_bytes=None) == EWORKSPACE
