"""6-qubit matrix-core blocks where a workgroup takes several tiles, the next
one's loads on their way during the products: a tile has 12 bits in complex64
(512 workgroups at most) and 11 in complex128 (256). Against the dense oracle."""
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


@pytest.mark.parametrize("dtype,n,tiles", [(C64, 21, 1), (C64, 22, 2), (C64, 23, 4),
                                           (C128, 20, 2), (C128, 21, 4)])
@pytest.mark.parametrize("where", ["low", "high", "middle", "spread"])
def test_several_tiles(qs_lib, dtype, n, tiles, where):
    assert 2 ** n // (2 ** (12 if dtype == C64 else 11)) == tiles * (512 if dtype == C64 else 256)
    bits = {"low": (2, 0, 5, 1, 4, 3), "high": tuple(range(n - 6, n)),
            "middle": (11, 9, 10, 12, 8, 13), "spread": (0, n - 1, 3, n - 4, 6, 11)}[where]
    a = workloads.gaussian_state(n, n)
    m = haar(64, n + bits[0])
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.profile_start()
        st.apply_fused(list(bits), m)
        assert "fused6_mfma" in st.profile_stop()
        assert_parity(st.amplitudes(), dense.apply_matrix(a, n, list(bits), m), dtype, f"{bits}")
