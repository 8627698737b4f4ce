"""Transforms of one to three qubits anywhere in small states (the narrowest
strided passes), both directions, against numpy's FFT in float64."""
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
@pytest.mark.parametrize("n", [10, 11, 12])
@pytest.mark.parametrize("length", [1, 2, 3])
def test_narrow_ranges(qs_lib, dtype, n, length):
    a = workloads.gaussian_state(n, n)
    for start in range(n - length + 1):
        with qs_lib.State(n, dtype) as st:
            st.set_amplitudes(a)
            st.qft(start, length)
            want = fourier(a, n, start, length, False)
            assert_parity(st.amplitudes(), want, dtype, f"{start}+{length} of {n}")
            st.qft(start, length)
            st.qft(start, length, inverse=True)
            assert_parity(st.amplitudes(), want, dtype, f"{start}+{length} of {n} there and back")
