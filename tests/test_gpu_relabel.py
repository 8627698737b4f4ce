"""Readouts behind a relabelling: the amplitudes move to qubit order in at most
two sweeps, whatever the permutation. Exact: amplitudes only move."""
import numpy as np
import pytest

import workloads
from parity import C64, C128

pytestmark = pytest.mark.gpu


def permuted(a, n, perm):
    """a read with qubit q of the result at bit perm[q] of the index of a."""
    x = np.arange(2 ** n)
    y = np.zeros_like(x)
    for q in range(n):
        y |= ((x >> q) & 1) << perm[q]
    return a[y]


def swaps_to(perm):
    """SWAPs (as label exchanges) that take the identity labelling to perm."""
    cur, out = list(range(len(perm))), []
    for q in range(len(perm)):
        k = cur.index(perm[q])
        if k != q:
            cur[q], cur[k] = cur[k], cur[q]
            out.append((q, k))
    return out


SHAPES = {
    "one pair": lambda n, g: [(0, n - 1)],
    "one low pair": lambda n, g: [(0, 1)],
    "high pairs": lambda n, g: [(n - 1, n - 2), (n - 3, n - 4)],
    "reversal": lambda n, g: [(i, n - 1 - i) for i in range(n // 2)],
    "three bits in a cycle": lambda n, g: [(0, n - 1), (0, 1)],
    "rotation": lambda n, g: [(0, i) for i in range(1, n)],
    "random": lambda n, g: swaps_to(list(g.permutation(n))),
    "random high": lambda n, g: [(n - n // 2 + a, n - n // 2 + b) for a, b in
                                 swaps_to(list(g.permutation(n // 2)))],
}


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", [4, 5, 9, 10, 11, 12, 15, 18])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_readout_in_qubit_order(qs_lib, dtype, n, shape):
    g = np.random.default_rng(n)
    a = workloads.gaussian_state(n, n).astype(np.complex64 if dtype == C64 else np.complex128)
    swaps = SHAPES[shape](n, g)
    perm = list(range(n))
    for x, y in swaps:
        perm[x], perm[y] = perm[y], perm[x]
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        for x, y in swaps:
            st.apply_swap(int(x), int(y))
        np.testing.assert_array_equal(st.amplitudes(a.dtype), permuted(a, n, perm))
        # the labels are the identity now: a second readout moves nothing
        np.testing.assert_array_equal(st.amplitudes(a.dtype), permuted(a, n, perm))
