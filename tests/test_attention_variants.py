"""Which workgroup shape an attention call takes (host arithmetic, no GPU): the
GPU tests' calls must reach every shape the kernel is built in."""
import ctypes

import pytest

pytest.importorskip("torch")
from test_gpu_kernels import ATT_VARIANT_CASES


def variant(bclib, B, H, Tq, Tk, d):
    v = [ctypes.c_int(-1) for _ in range(3)]
    rc = bclib.lib().bc_attention_variant(B, H, Tq, Tk, d, *(ctypes.byref(x) for x in v))
    assert rc == bclib.OK
    return tuple(x.value for x in v)


def test_gpu_cases_take_the_shapes_they_name(bclib):
    for want, shape in ATT_VARIANT_CASES:
        assert variant(bclib, *shape) == want, shape


def test_every_choice_is_among_the_gpu_cases(bclib):
    """Over a spread of calls the choice gives no shape that the cases lack."""
    named = {(v, s[4]) for v, s in ATT_VARIANT_CASES}
    got = set()
    for d in (32, 64, 72, 128):
        for bh in (1, 5, 16, 24, 48, 96, 256, 1000):
            for Tq in (1, 64, 65, 129, 256, 500, 1025, 2050, 4096, 14566):
                for Tk in (1, 256, 257, 14566):
                    got.add((variant(bclib, 1, bh, Tq, Tk, d), d))
    assert got == named


def test_bad_shapes_are_refused(bclib):
    v = [ctypes.c_int() for _ in range(3)]
    refs = [ctypes.byref(x) for x in v]
    assert bclib.lib().bc_attention_variant(1, 1, 8, 8, 40, *refs) != bclib.OK
    assert bclib.lib().bc_attention_variant(1, 1, 0, 8, 64, *refs) != bclib.OK
    assert bclib.lib().bc_attention_variant(1, 1, 8, 8, 64, None, None, None) != bclib.OK
