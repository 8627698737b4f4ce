"""How circuits run on states below a tile: deep ones on up to five qubits as
one matrix, many gates on few of more qubits as blocks, the others gate by gate
in LDS; each in the identity labelling and behind a relabelling, against the
oracle. Their tables do not depend on the labelling."""
import numpy as np
import pytest

import workloads
from oracle import dense
from parity import C64, C128, assert_parity

pytestmark = pytest.mark.gpu


def haar(d, g):
    q, r = np.linalg.qr(g.standard_normal((d, d)) + 1j * g.standard_normal((d, d)))
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


def on(qubits, count, g):
    return [("mat", [int(x) for x in g.choice(qubits, 2, replace=False)], haar(4, g))
            for _ in range(count)]


def check(qs_lib, n, dtype, gates, swaps, what):
    """Run twice, then behind a relabelling; the kernels of the first run."""
    a = workloads.gaussian_state(n, n)
    c = qs_lib.Circuit(n).add_gates(gates)
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.profile_start()
        st.run(c)
        names = set(st.profile_stop())
        for x, y in swaps:
            st.apply_swap(x, y)
        st.run(c)
        want = dense.run_circuit(a, n, gates)
        for x, y in swaps:
            want = dense.run_circuit(want, n, [("swap", x, y)])
        assert_parity(st.amplitudes(), dense.run_circuit(want, n, gates), dtype, what)
    c.free()
    return names


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
def test_deep_circuits_are_one_launch(qs_lib, dtype, n):
    g = np.random.default_rng(n)
    gates = ([("u3", 0, 0.1 * i, 0.2, 0.3) for i in range(20)] if n == 1
             else workloads.random_circuit(n, 25, n) + on(range(n), 5, g))
    swaps = [] if n == 1 else [(0, n - 1), (0, 1)]
    assert check(qs_lib, n, dtype, gates, swaps, f"n={n}") == {"circuit_lds"}


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", [6, 8, 10])
@pytest.mark.parametrize("width", [3, 4, 5])
def test_gates_on_few_qubits_are_blocks(qs_lib, dtype, n, width):
    g = np.random.default_rng(n + width)
    qubits = [int(x) for x in g.permutation(n)[:width]]
    names = check(qs_lib, n, dtype, on(qubits, 80, g), [(0, n - 1), (1, 2), (0, 3)], f"{n} {width}")
    assert names == {f"fused{width}"} or names == {f"fused{width}_mfma"}


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("n", [2, 6, 9, 10])
def test_every_labelling_uses_the_same_tables(qs_lib, dtype, n):
    """A circuit that moves the labels, run again and again: the library asks
    for device memory in the first run only."""
    import torch
    gates = workloads.random_circuit(n, 3, n) + [("swap", q, q + 1) for q in range(n - 1)]
    gates += workloads.random_circuit(n, 2, n + 1)
    a = workloads.gaussian_state(n, n)
    c = qs_lib.Circuit(n).add_gates(gates)
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.run(c)
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        for _ in range(n):
            st.run(c)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
        for _ in range(n + 1):
            a = dense.run_circuit(a, n, gates)
        assert_parity(st.amplitudes(), a, dtype, f"n={n}")
    c.free()


@pytest.mark.parametrize("dtype", [C64, C128])
def test_blocks_are_known_after_a_run(qs_lib, dtype):
    """A run on a state below a tile leaves the circuit planned in blocks."""
    n = 8
    gates = workloads.random_circuit(n, 4, 3)
    c, ref = qs_lib.Circuit(n).add_gates(gates), qs_lib.Circuit(n).add_gates(gates).plan(5)
    assert c.info()["blocks"] == -1
    with qs_lib.State(n, dtype) as st:
        st.run(c)
        assert c.info() == ref.info()
        assert c.block(0)[0] == ref.block(0)[0]
        st.run(c)
        want = dense.run_circuit(dense.zero_state(n), n, gates + gates)
        assert_parity(st.amplitudes(), want, dtype)
    c.free()
    ref.free()
