"""The planner is host code: a pass takes pair rounds or, where these would be
many more, dense (complex64) or sparse (complex128) ones, which hold every gate
that four bits allow."""
import numpy as np
import pytest

import workloads


@pytest.fixture(scope="module")
def qs():
    import paper_2304_14969_amd as m
    m.open_library()
    return m


def rounds(qs, n, gates, dtype):
    c = qs.Circuit(n)
    for qubits, m in gates:
        c.add_matrix(qubits, m)
    info = c.tile_info(dtype)
    c.free()
    return info["passes"], info["rounds"]


def on_few(first, width, count, g):
    m = np.linalg.qr(g.standard_normal((4, 4)) + 1j * g.standard_normal((4, 4)))[0]
    return [([first + int(x) for x in g.choice(width, 2, replace=False)], m) for _ in range(count)]


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("n", [12, 16, 20, 21, 26])
@pytest.mark.parametrize("high", [False, True])
def test_gates_on_four_qubits_are_one_round(qs, dtype, n, high):
    g = np.random.default_rng(n)
    first = n - 4 if high else 0
    assert rounds(qs, n, on_few(first, 4, 200, g), dtype) == (1, 1)
    assert rounds(qs, n, on_few(first, 3, 200, g), dtype) == (1, 1)


@pytest.mark.parametrize("n", [12, 16, 20, 24, 28])
def test_rings_take_dense_rounds(qs, n):
    """A ring of diagonal gates is a chain: pairs would take a round a gate in
    every pass, dense rounds take three gates of it where they have four bits."""
    d = np.diag(np.exp(1j * np.arange(4)))
    gates = [([q, (q + 1) % n], d) for _ in range(6) for q in range(n)]
    _, r = rounds(qs, n, gates, qs.C64)
    assert r <= 2 * len(gates) // 3


def test_random_layers_take_pair_rounds(qs):
    """Two random pairs seldom share four bits: dense rounds would be as many
    as pair rounds, at twice the time each."""
    n = 24
    gates = workloads.random_circuit(n, 8, 1)
    c = qs.Circuit(n).add_gates(gates)
    info = c.tile_info(qs.C64)
    two = sum(len(x) == 3 for x in gates)
    assert info["rounds"] >= two // 2  # at most two gates a round
    c.free()
