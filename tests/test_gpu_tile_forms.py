"""Circuits whose passes take pair rounds and dense or sparse ones side by side
(gates on a few qubits, then random layers, then a chain), and batches that take
one form for all their kets, against the oracle."""
import numpy as np
import pytest

import workloads
from oracle import dense
from parity import C64, C128, assert_parity

pytestmark = pytest.mark.gpu


def haar(d, g):
    q, r = np.linalg.qr(g.standard_normal((d, d)) + 1j * g.standard_normal((d, d)))
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


def few(n, g, qubits, count=20):
    return [("mat", [int(x) for x in g.choice(qubits, 2, replace=False)], haar(4, g))
            for _ in range(count)]


def layers(n, g, count=3):
    out = []
    for _ in range(count):
        p = g.permutation(n)
        out += [("mat", [int(q)], haar(2, g)) for q in range(n)]
        out += [("mat", [int(p[2 * i]), int(p[2 * i + 1])], haar(4, g)) for i in range(n // 2)]
    return out


KINDS = {
    "few": lambda n, g: few(n, g, [0, 1, n - 2, n - 1]),
    "few and layers": lambda n, g: few(n, g, [n - 4, n - 3, n - 2, n - 1]) + layers(n, g),
    "layers, few, chain": lambda n, g: layers(n, g) + few(n, g, [0, 2, n - 1]) +
        [("mat", [q, q + 1], haar(4, g)) for q in range(n - 1)],
    "singles among few": lambda n, g: [x for y in few(n, g, [1, 4, n - 3]) for x in
                                       (y, ("mat", [int(g.integers(n))], haar(2, g)))],
    "three qubits and layers": lambda n, g: layers(n, g) + [("mat", [0, n // 2, n - 1], haar(8, g))] +
        layers(n, g, 2),
}


def run_oracle(a, n, gates):
    for _, qubits, m in gates:
        a = dense.apply_matrix(a, n, qubits, m)
    return a


@pytest.mark.parametrize("dtype,n", [(C64, 12), (C64, 14), (C64, 17), (C128, 11), (C128, 13), (C128, 16)])
@pytest.mark.parametrize("kind", list(KINDS))
def test_forms_side_by_side(qs_lib, dtype, n, kind):
    gates = KINDS[kind](n, np.random.default_rng(n + len(kind)))
    a = workloads.gaussian_state(n, n)
    c = qs_lib.Circuit(n).add_gates(gates)
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.run(c)
        assert_parity(st.amplitudes(), run_oracle(a, n, gates), dtype, kind)
    c.free()


@pytest.mark.parametrize("kinds", [["few"] * 4, ["layers, few, chain", "few", "few and layers", "few"],
                                   ["three qubits and layers", "few", "few and layers", "few"]])
def test_batch_in_one_form(qs_lib, kinds):
    """The sum decides for the batch; a second batch of the same circuits with
    others beside them decides anew, and the first still runs as it did."""
    widths = [12, 14, 13, 7]
    g = np.random.default_rng(len(kinds[0]))
    lists = [KINDS[k](n, g) for k, n in zip(kinds, widths)]
    circs = [qs_lib.Circuit(n).add_gates(x) for n, x in zip(widths, lists)]
    more = [qs_lib.Circuit(15).add_gates(layers(15, g, 6)) for _ in range(3)]
    one = qs_lib.Batch(widths, C64)
    two = qs_lib.Batch(widths + [15] * 3, C64)
    for again in range(2):
        for b, cs in ((one, circs), (two, circs + more)):
            b.reset()
            b.run(cs)
            for i, (n, x) in enumerate(zip(widths, lists)):
                assert_parity(b.amplitudes(i), run_oracle(dense.zero_state(n), n, x), C64,
                              f"ket {i} {kinds[i]}")
    one.free()
    two.free()


@pytest.mark.parametrize("dtype,n", [(C64, 14), (C128, 13)])
@pytest.mark.parametrize("kind", ["few", "layers, few, chain"])
def test_streaming_and_plain_passes_agree(qs_lib, dtype, n, kind):
    """Bit for bit, in every form."""
    gates = KINDS[kind](n, np.random.default_rng(n))
    a = workloads.gaussian_state(n, n)
    c = qs_lib.Circuit(n).add_gates(gates)
    saved = qs_lib.tune_get("sweep.stream")
    got = []
    try:
        for stream in (1, 2):
            qs_lib.tune_set("sweep.stream", stream)
            with qs_lib.State(n, dtype) as st:
                st.set_amplitudes(a)
                st.run(c)
                got.append(st.amplitudes())
    finally:
        qs_lib.tune_set("sweep.stream", saved)
    np.testing.assert_array_equal(got[0], got[1])
    assert_parity(got[0], run_oracle(a, n, gates), dtype, kind)
    c.free()
