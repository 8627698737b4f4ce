"""Factorized kets: the one-launch reset and the one-launch read of amplitudes,
for few and many subsystems and indices, against the expanded vector."""
import numpy as np
import pytest

from parity import C64, C128

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", [1, 9, 17, 63])
def test_basis_reset(qs_lib, n, dtype):
    st = qs_lib.State(n, dtype, factorized=True)
    for x in (0, 2 ** n - 1, 0x2AAAAAAAAAAAAAAA % 2 ** n):
        st.set_basis(x)
        got = st.gather([x, x ^ 1, x ^ 2 ** (n - 1)])
        assert got[0] == 1.0 and got[1] == 0.0 and got[2] == 0.0
        assert len(st.subsystems()) == n
    st.free()


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("pairs", [0, 3, 8])
def test_gather_is_the_product(qs_lib, pairs, dtype):
    """17 qubits in 17 - pairs subsystems (one to three rounds of loads of
    eight), read at 1, 256, 257 and 1000 indices."""
    n = 17
    rng = np.random.default_rng(pairs)
    st = qs_lib.State(n, dtype, factorized=True)
    for q in range(n):
        m = np.linalg.qr(rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2)))[0]
        st.apply_fused([q], m)
    for j in range(pairs):
        m = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))[0]
        st.apply_fused([16 - 2 * j, 15 - 2 * j], m)
    assert len(st.subsystems()) == n - pairs
    dn = qs_lib.State(n, dtype)
    st.expand_into(dn)
    want = dn.amplitudes()
    # 17 factors, each product rounded to the state's type in the expansion
    # only: 17 roundings of the amplitude there, a few per read entry here
    u = 6e-8 if dtype == C64 else 1.2e-16
    for m in (1, 256, 257, 1000):
        idx = rng.integers(0, 2 ** n, size=m)
        got = st.gather(idx)
        assert np.all(np.abs(got - want[idx]) <= 40 * u * np.abs(want).max())
    dn.free()
    st.free()
