"""How steps are dealt to the fused kernel (host code of the library, no GPU)."""
import ctypes

import pytest

from paper_1911_03225_amd import fdm


def _trial(order, steps):
    f = fdm.load_library().fdm_debug_fused_trial   # (exported for this test)
    f.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]
    f.restype = ctypes.c_int32
    launches, singles = ctypes.c_int32(), ctypes.c_int32()
    n = f(order, steps, ctypes.byref(launches), ctypes.byref(singles))
    return n, launches.value, singles.value


@pytest.mark.parametrize("order", [1, 2, 3])
def test_a_fused_trial_times_fused_launches_alone(order):
    """What the autotuner reports as the fused schedule's time holds no steps
    of the stage kernels, however few steps were asked for."""
    per = 2 if order == 1 else 1
    for asked in list(range(1, 41)) + [2 ** 31 - 4 if order == 1 else 2 ** 31 - 2]:
        n, launches, singles = _trial(order, asked)
        assert singles == 0 and launches >= 2 and launches % 2 == 0, asked
        assert launches * per == n and asked <= n < asked + 4
    n, launches, singles = _trial(order, 2 ** 31 - 1)   # (nothing above it)
    assert n == 2 ** 31 - 1 and launches * per + singles == n
