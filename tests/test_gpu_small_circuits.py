"""Circuits on states smaller than a tile, run whole in one launch: every width
at and below the largest such state, in the identity labelling and behind a
relabelling, against the oracle."""
import numpy as np
import pytest

import workloads
from oracle import dense
from parity import C64, C128, assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", range(1, 13))
def test_every_width(qs_lib, dtype, n):
    if n == 1:
        gates = [("h", 0), ("u3", 0, 0.3, 0.4, 0.5)]
    else:
        gates = workloads.random_circuit(n, 5, n) + [("cx", 0, n - 1), ("cp", n - 1, 0, 0.3), ("h", 0)]
    a = workloads.gaussian_state(n, n)
    c = qs_lib.Circuit(n).add_gates(gates)
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.profile_start()
        st.run(c)
        whole = "circuit_lds" in st.profile_stop()
        assert whole == (n <= (11 if dtype == C64 else 10))
        want = dense.run_circuit(a, n, gates)
        assert_parity(st.amplitudes(), want, dtype, f"n={n}")
        if n > 2:  # bit-reversed labels, then a swap inside the circuit
            st.qft()
            c.add_gates([("swap", 0, n - 1), ("h", 1)])
            st.run(c)
            want = dense.run_circuit(dense.qft(want, n), n, gates + [("swap", 0, n - 1), ("h", 1)])
            assert_parity(st.amplitudes(), want, dtype, f"n={n} relabelled")
    c.free()


@pytest.mark.parametrize("dtype", [C64, C128])
def test_wider_gates_run_as_blocks(qs_lib, dtype):
    n = 9
    g = np.random.default_rng(2)
    q, _ = np.linalg.qr(g.standard_normal((8, 8)) + 1j * g.standard_normal((8, 8)))
    gates = workloads.random_circuit(n, 2, 1) + [("mat", [0, 4, 8], q)]
    c = qs_lib.Circuit(n).add_gates(gates)
    with qs_lib.State(n, dtype) as st:
        st.profile_start()
        st.run(c)
        assert "circuit_lds" not in st.profile_stop()
        want = dense.apply_matrix(dense.run_circuit(dense.zero_state(n), n, gates[:-1]), n, [0, 4, 8], q)
        assert_parity(st.amplitudes(), want, dtype)
    c.free()
