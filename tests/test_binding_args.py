"""Arguments of the wrappers that pass integers straight to the C entry points:
what is no integer or None is refused before the call."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("bad", ["abc", b"abc", (ctypes.c_char * 8)(), ctypes.byref(ctypes.c_int(1)),
                                 ctypes.c_void_p(8), ctypes.c_char_p(b"x"), 1.5, np.int64(8), [8]])
def test_refused(bad):
    import paper_1203_4938_amd as dp
    for at in (0, 1, 2, 4, 5):
        a = [0, 0, 0, dp.FFT_FORWARD, 0, 0]
        a[at] = bad
        with pytest.raises(TypeError):
            dp.fft_exec(*a)
    for at in (0, 1, 2, 4, 5, 6):
        a = [0, 0, 0, 0, 0, 0, 0]
        a[at] = bad
        with pytest.raises(TypeError):
            dp.fft_conv_exec(*a)


def test_accepted():
    import paper_1203_4938_amd as dp
    for v in (0, None, False, 2 ** 64, -2 ** 64):  # all NULL
        assert dp.fft_exec(v, v, v, dp.FFT_FORWARD, v, v) == dp.FFT_E_INVALID
        assert dp.fft_conv_exec(v, v, v, 0, v, v, v) == dp.FFT_E_INVALID
