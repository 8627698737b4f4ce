"""Blocks whose matrix rides in the kernel arguments, and blocks on states below
a matrix-core tile, from states of only the block's qubits up, against the
dense oracle; dense and factorized states."""
import numpy as np
import pytest

import workloads
from oracle import dense
from parity import C64, C128, assert_parity

pytestmark = pytest.mark.gpu


def haar(dim, seed):
    rng = np.random.default_rng(seed)
    q, r = np.linalg.qr(rng.standard_normal((dim, dim)) + 1j * rng.standard_normal((dim, dim)))
    return q * (np.diag(r) / abs(np.diag(r)))


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("n", [3, 8, 13, 17])
def test_argument_blocks(qs_lib, n, k, dtype):
    a = workloads.gaussian_state(n, n)
    rng = np.random.default_rng(n + k)
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        for i in range(4):
            bits = [int(x) for x in rng.choice(n, size=k, replace=False)]
            m = haar(2 ** k, 10 * i + k)
            st.apply_fused(bits, m)
            a = dense.apply_matrix(a, n, bits, m)
            m[:] = 0.0  # the matrix is the caller's again once the call returns
        assert_parity(st.amplitudes(), a, dtype, f"k={k} n={n}")
    if n <= 13:
        st = qs_lib.State(n, dtype, factorized=True)
        want = np.zeros(2 ** n, dtype=np.complex128)
        want[0] = 1.0
        for i in range(4):
            bits = [int(x) for x in rng.choice(n, size=k, replace=False)]
            m = haar(2 ** k, 40 * i + k)
            st.apply_fused(bits, m)
            want = dense.apply_matrix(want, n, bits, m)
        dn = qs_lib.State(n, dtype)
        st.expand_into(dn)
        assert_parity(dn.amplitudes(), want, dtype, f"factorized k={k} n={n}")
        st.free()
        dn.free()


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("k", [4, 5, 6])
@pytest.mark.parametrize("n", [6, 7, 9, 10, 11, 12])
def test_blocks_on_small_states(qs_lib, n, k, dtype):
    a = workloads.gaussian_state(n, n)
    rng = np.random.default_rng(n + k)
    with qs_lib.State(n, dtype) as st:
        for i in range(6):
            bits = [int(x) for x in rng.choice(n, size=k, replace=False)]
            m = haar(2 ** k, 10 * i + k)
            st.set_amplitudes(a)
            st.apply_fused(bits, m)
            assert_parity(st.amplitudes(), dense.apply_matrix(a, n, bits, m), dtype, f"{bits}")


@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("n", [3, 9, 14])
def test_blocks_on_bit_zero(qs_lib, n, k):
    """complex64 blocks that hold bit 0, at every row of the matrix: the sweeps
    of pairs, applied by themselves and as the blocks of a circuit."""
    a = workloads.gaussian_state(n, n)
    rng = np.random.default_rng(n * k)
    for row in range(k):
        bits = [1 + int(x) for x in rng.choice(n - 1, size=k - 1, replace=False)]
        bits.insert(row, 0)
        m = haar(2 ** k, 7 * row + k)
        want = dense.apply_matrix(a, n, bits, m)
        with qs_lib.State(n, C64) as st:
            st.set_amplitudes(a)
            st.apply_fused(bits, m)
            assert_parity(st.amplitudes(), want, C64, f"{bits}")
            st.set_amplitudes(a)
            c = qs_lib.Circuit(n).add_gates([("mat", tuple(bits), m)])
            c.plan(3)
            st.run(c)
            assert_parity(st.amplitudes(), want, C64, f"circuit {bits}")
            c.free()
