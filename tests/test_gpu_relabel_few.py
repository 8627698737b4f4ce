"""Relabellings of a few bits, read back by exchanges or by sweeps according to
their number, their bits and the state's size. Exact: amplitudes only move."""
import numpy as np
import pytest

from parity import C64, C128

pytestmark = pytest.mark.gpu

SWAPS = {  # label exchanges, and the launches of the readout below and from 20 qubits
    "pair": (lambda n: [(1, n - 2)], 1, 1),
    "two pairs": (lambda n: [(0, n - 1), (2, n - 3)], 1, 1),
    "two high pairs": (lambda n: [(n - 1, n - 2), (n - 3, n - 4)], 2, 2),
    "low cycle of three": (lambda n: [(0, 1), (1, 2)], 2, 2),
    "mixed cycle of three": (lambda n: [(0, n // 2), (n // 2, n - 1)], 2, 2),
    "high cycle of three": (lambda n: [(n - 1, n - 2), (n - 2, n - 3)], 2, 2),
    "cycle of four": (lambda n: [(0, 1), (1, n - 2), (n - 2, n - 1)], 3, 2),
    "cycle of three and pair": (lambda n: [(0, 1), (1, n - 2), (3, n - 1)], 3, 2),
    "two cycles of three": (lambda n: [(0, n - 1), (n - 1, n // 2), (1, n - 2), (n - 2, n // 2 + 1)], 4, 2),
    "cycle of six": (lambda n: [(i, i + 1) for i in range(5)], 2, 2),
}


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", [13, 19, 20, 21])
@pytest.mark.parametrize("name", list(SWAPS))
def test_few_bits(qs_lib, dtype, n, name):
    make, below, from20 = SWAPS[name]
    swaps = make(n)
    a = np.arange(2 ** n, dtype=np.float32).astype(np.complex64 if dtype == C64 else np.complex128)
    want, lab = a, list(range(n))
    for x, y in swaps:
        lab[x], lab[y] = lab[y], lab[x]
    idx = np.arange(2 ** n)
    src = np.zeros_like(idx)
    for q in range(n):
        src |= ((idx >> q) & 1) << lab[q]
    want = a[src]
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        for x, y in swaps:
            st.apply_swap(x, y)
        st.profile_start()
        got = st.amplitudes(a.dtype)
        stats = st.profile_stop()
        np.testing.assert_array_equal(got, want)
        assert stats["bitswap"]["launches"] == (below if n < 20 else from20)
