"""Complex64 circuits of many equal gates: the casts of their matrices to FP32 do
not add up in the state's norm. The bound is sqrt(gates) roundings of 2^-24, as
of errors at random; equal casts (1.7e-8 off for each Hadamard) grow with the
number of gates."""
import math

import numpy as np
import pytest

import workloads
from parity import C64

pytestmark = pytest.mark.gpu


def fourier_circuit(n, times):
    out = []
    for _ in range(times):
        for j in range(n - 1, -1, -1):
            out.append(("h", j))
            out += [("cp", m, j, math.pi / 2 ** (j - m)) for m in range(j - 1, -1, -1)]
    return out


@pytest.mark.parametrize("n,times", [(6, 24), (10, 12), (12, 12), (15, 8)])
@pytest.mark.parametrize("batched", [False, True])
def test_norm_of_repeated_fourier_circuits(qs_lib, n, times, batched):
    # (amplitudes without structure first: those of a transformed basis state
    # round back to powers of two)
    gates = workloads.random_circuit(n, 2, n) + fourier_circuit(n, times)
    c = qs_lib.Circuit(n).add_gates(gates)
    if batched:
        b = qs_lib.Batch([n], C64)
        b.run([c])
        got = b.amplitudes(0).astype(np.complex128)
        b.free()
    else:
        with qs_lib.State(n, C64) as st:
            st.set_amplitudes(workloads.gaussian_state(n, n).astype(np.complex64))
            st.run(c)
            got = st.amplitudes().astype(np.complex128)
    c.free()
    assert abs(np.linalg.norm(got) - 1.0) <= math.sqrt(len(gates)) * 2.0 ** -24
