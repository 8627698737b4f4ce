"""Transforms over the sizes where the plan's tile widths change, whole ranges
and inner ones, both directions, against numpy's FFT in float64."""
import numpy as np
import pytest

import workloads
from parity import C64, C128, assert_parity

pytestmark = pytest.mark.gpu


def fourier(a, n, start, length, inverse):
    v = a.reshape(2 ** (n - start - length), 2 ** length, 2 ** start)
    f = np.fft.fft if inverse else np.fft.ifft
    return f(v, axis=1, norm="ortho").reshape(-1)


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", [9, 10, 12, 13, 16, 17, 18, 19, 20, 21, 22, 23])
@pytest.mark.parametrize("shape", ["whole", "above", "inside", "top"])
def test_ranges(qs_lib, dtype, n, shape):
    start, length = {"whole": (0, n), "above": (3, n - 3), "inside": (1, n - 2),
                     "top": (n // 2, n - n // 2)}[shape]
    a = workloads.gaussian_state(n, n)
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.qft(start, length)
        want = fourier(a, n, start, length, False)
        assert_parity(st.amplitudes(), want, dtype, f"{shape} n={n}")
        st.qft(start, length)
        st.qft(start, length, inverse=True)  # the range is stored bit-reversed here
        assert_parity(st.amplitudes(), want, dtype, f"{shape} n={n} there and back")
