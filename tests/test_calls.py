"""The native entry points of the binding refuse arguments as the binding promises: TypeError for anything but a device
tensor of the right type, ValueError for shapes and freed handles.  Runs without a GPU: every case ends before a launch."""
import types

import pytest
import torch

import paper_2508_15601_amd as tm
from paper_2508_15601_amd import binding


def half(*shape):
    return torch.zeros(shape, dtype=torch.float16)


PACKED = types.SimpleNamespace(_h=0, K=256, N=32)
GROUP = types.SimpleNamespace(_h=0, K=256, N=32, experts=[None, None])
CACHE = types.SimpleNamespace(_h=0, batch=2, kv_heads=4)
OFF = torch.zeros(3, dtype=torch.int32)


@pytest.mark.parametrize("call, error", [
    (lambda: tm.tm_gemm_w4a16([0.0], PACKED, half(1, 32)), TypeError),
    (lambda: tm.tm_gemm_w4a16(half(1, 256), PACKED, half(1, 32)), TypeError),          # host tensors
    (lambda: tm.tm_gemm_w4a16(half(256), PACKED, half(1, 32)), ValueError),
    (lambda: tm.tm_gemm_w4a16(half(1, 128), PACKED, half(1, 32)), ValueError),
    (lambda: tm.tm_gemm_w4a16(half(2, 256), PACKED, half(1, 32)), ValueError),
    (lambda: tm.tm_gemm_w4a16_static(half(2, 256), PACKED, half(2, 16)), ValueError),
    (lambda: tm.tm_gemm_w4a16_ws(half(2, 256), PACKED, half(1, 32), None), ValueError),
    (lambda: tm.tm_gemm_w4a16_ex(half(2, 256), PACKED, half(2, 32), act=1), ValueError),
    (lambda: tm.tm_gemm_w4a16_ex(half(2, 256), PACKED, half(2, 32), bias=half(16)), ValueError),
    (lambda: tm.tm_gemm_w4a16_ex(half(2, 256), PACKED, half(2, 32), residual=half(1, 32)), ValueError),
    (lambda: tm.tm_gemm_w4a16_grouped(half(2, 256), GROUP, OFF[:2], half(2, 32)), ValueError),
    (lambda: tm.tm_gemm_w4a16_grouped_act(half(2, 256), GROUP, OFF, half(2, 32)), ValueError),
    (lambda: tm.tm_kv_append(CACHE, half(2, 1, 4, 64), half(2, 1, 4, 64), OFF[:2]), ValueError),
    (lambda: tm.tm_kv_append(CACHE, half(2, 1, 4, 128), half(2, 1, 4, 128), OFF), ValueError),
    (lambda: tm.tm_kv_append(CACHE, half(2, 1, 4, 128), half(2, 1, 4, 128), OFF[:2]), ValueError),      # freed cache
    (lambda: tm.tm_attn_decode(half(2, 8, 128), CACHE, OFF[:2], half(2, 4, 128), 1.0), ValueError),
    (lambda: tm.tm_attn_prefill(half(2, 8, 128), CACHE, OFF[:2], half(2, 8, 128), 1.0), ValueError),
])
def test_arguments_are_refused(call, error):
    with pytest.raises(error):
        call()


@pytest.mark.parametrize("batch, positions, counts", [(1, 2, None), (2, 1, None), (2, 2, 1), (1, 1, 1), (0, 2, 2)])
def test_prompt_attention_refuses_fewer_sequences_than_the_cache_has(batch, positions, counts):
    q, at = half(batch, 3, 8, 128), torch.zeros(positions, dtype=torch.int32)
    with pytest.raises(ValueError, match="sequences"):
        tm.tm_attn_prefill(q, CACHE, at, half(batch, 3, 8, 128), 1.0,
                           counts=None if counts is None else torch.zeros(counts, dtype=torch.int32))


@pytest.mark.parametrize("empty", [lambda: tm.tm_gemm_w4a16(half(0, 256), PACKED, half(0, 32)),
                                   lambda: tm.tm_gemm_w4a16_ex(half(0, 256), PACKED, half(0, 32))])
def test_no_rows_is_a_no_op_that_returns_the_output(empty):
    assert tuple(empty().shape) == (0, 32)


class Whole:
    """Converts with int() and has no __index__."""

    def __int__(self):
        return 1


@pytest.mark.parametrize("number", [1, 1.0, True, Whole(), "1", torch.tensor(1)])
def test_numbers_are_taken_as_int_and_float_take_them(number):
    """act, max_len and scale: the call gets past its conversions, to the freed handle."""
    wide, narrow = half(2, 256), half(2, 16)
    assert tm.tm_gemm_w4a16_ex(half(0, 256), PACKED, half(0, 16), act=number).shape == (0, 16)
    assert tm.tm_gemm_w4a16_grouped_act(half(0, 256), GROUP, OFF, half(0, 16), act=number).shape == (0, 16)
    with pytest.raises(TypeError, match="device tensor"):
        tm.tm_gemm_w4a16_ex(wide, PACKED, narrow, act=number)
    with pytest.raises(TypeError, match="device tensor"):
        tm.tm_attn_decode(half(2, 8, 128), CACHE, OFF[:2], half(2, 8, 128), 1.0, max_len=number)


@pytest.mark.parametrize("bad, error", [(None, TypeError), ("x", ValueError), ([1], TypeError)])
def test_what_int_refuses_is_refused(bad, error):
    with pytest.raises(error):
        tm.tm_gemm_w4a16_ex(half(2, 256), PACKED, half(2, 16), act=bad)


@pytest.mark.parametrize("path", ["_LIB_PATH", "_CALLS_PATH"])
def test_a_missing_build_is_named_with_the_way_to_make_it(path, tmp_path, monkeypatch):
    tm.load_library()
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, path, str(tmp_path / "not_built.so"))
    with pytest.raises(ImportError, match="not_built.so is missing: run .*build"):
        tm.load_library()


@pytest.mark.gpu
def test_a_wrong_dtype_is_named():
    with pytest.raises(TypeError, match="X must have dtype torch.float16, got torch.float32"):
        tm.tm_gemm_w4a16(torch.zeros(1, 256, device="cuda"), PACKED, half(1, 32).cuda())
