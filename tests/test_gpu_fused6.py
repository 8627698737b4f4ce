"""6-qubit blocks on the matrix cores against the dense oracle, at the sizes
and bit positions where the tile changes."""
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


# A tile is 12 bits wide (complex64) or 11 (complex128): below that the vector
# kernel runs; 20 qubits give a workgroup several complex64 tiles.
@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n,bits", [
    (10, (9, 0, 3, 7, 1, 5)), (11, (5, 4, 3, 2, 1, 0)), (12, (6, 7, 8, 9, 10, 11)),
    (12, (3, 1, 11, 4, 0, 10)), (13, (0, 12, 2, 10, 4, 7)), (17, (16, 15, 14, 13, 12, 11)),
    (17, (0, 1, 2, 3, 4, 5)), (18, (1, 2, 3, 4, 5, 6)), (20, (19, 4, 0, 11, 6, 5)),
    (20, (7, 8, 9, 6, 18, 10)),
])
def test_block(qs_lib, n, bits, dtype):
    a = workloads.gaussian_state(n, n)
    m = haar(64, 3 * n + bits[0])
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.apply_fused(list(bits), m)
        # 64-term sums of a unitary's products: the bound of the 5-qubit blocks
        # (32 terms) holds for twice the terms, being far above sqrt(64) roundings
        assert_parity(st.amplitudes(), dense.apply_matrix(a, n, list(bits), m), dtype, f"{bits}")
