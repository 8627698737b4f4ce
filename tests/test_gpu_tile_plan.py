"""The tile-pass planner over gate lists of every width (one-qubit gates
merged into wider ones, wide gates as blocks between the passes), against the
oracle applying the gates one at a time."""
import numpy as np
import pytest

import workloads
from oracle import dense
from parity import C64, C128, assert_parity

pytestmark = pytest.mark.gpu


def haar(d, g):
    q, r = np.linalg.qr(g.standard_normal((d, d)) + 1j * g.standard_normal((d, d)))
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


def mixed(n, count, widths, g):
    out = []
    for _ in range(count):
        k = int(g.choice(widths))
        out.append(("mat", [int(x) for x in g.choice(n, k, replace=False)], haar(2 ** k, g)))
    return out


LISTS = {
    "one-qubit only": lambda n, g: mixed(n, 30, [1], g),
    "one gate": lambda n, g: mixed(n, 1, [2], g),
    "the same pair both ways": lambda n, g: [("mat", [3, 9], haar(4, g)), ("mat", [9, 3], haar(4, g)),
                                             ("mat", [9], haar(2, g)), ("mat", [3, 9], haar(4, g))],
    "one and two": lambda n, g: mixed(n, 60, [1, 1, 2], g),
    "up to four": lambda n, g: mixed(n, 40, [1, 2, 2, 3, 4], g),
    "up to six": lambda n, g: mixed(n, 30, [1, 1, 2, 2, 3, 4, 5, 6], g),
    "a wide gate alone": lambda n, g: mixed(n, 1, [6], g),
    "chain": lambda n, g: [("mat", [q, q + 1], haar(4, g)) for q in range(n - 1)],
}


@pytest.mark.parametrize("dtype,n", [(C64, 12), (C64, 15), (C128, 11), (C128, 14)])
@pytest.mark.parametrize("name", list(LISTS))
@pytest.mark.parametrize("mfma", [1, 0])
def test_gate_lists(qs_lib, dtype, n, name, mfma):
    if dtype == C128 and not mfma:
        pytest.skip("the switch is for complex64")
    g = np.random.default_rng(1000 * n + len(name))
    gates = LISTS[name](n, g)
    a = workloads.gaussian_state(n, n)
    want = a
    for _, qubits, m in gates:
        want = dense.apply_matrix(want, n, qubits, m)
    saved = qs_lib.tune_get("tile.mfma")
    qs_lib.tune_set("tile.mfma", mfma)
    try:
        c = qs_lib.Circuit(n).add_gates(gates)
        with qs_lib.State(n, dtype) as st:
            st.set_amplitudes(a)
            st.run(c)
            assert_parity(st.amplitudes(), want, dtype, name)
        c.free()
    finally:
        qs_lib.tune_set("tile.mfma", saved)


def test_batch_of_every_kind(qs_lib):
    """One batch whose kets run as passes of pair rounds, passes of dense
    rounds (gates of three and four qubits) and block launches (wider gates)."""
    n = [12, 13, 12, 14, 13, 12]
    names = ["one and two", "up to four", "up to six", "chain", "one-qubit only", "up to four"]
    g = np.random.default_rng(5)
    lists = [LISTS[k](w, g) for k, w in zip(names, n)]
    lists = [[x for x in gates if len(x[1]) < 6] for gates in lists]  # batched blocks: 5 qubits
    b = qs_lib.Batch(n, C64)
    b.run([qs_lib.Circuit(w).add_gates(x) for w, x in zip(n, lists)], 5)
    for i, (w, gates) in enumerate(zip(n, lists)):
        want = dense.zero_state(w)
        for _, qubits, m in gates:
            want = dense.apply_matrix(want, w, qubits, m)
        assert_parity(b.amplitudes(i), want, C64, f"ket {i} {names[i]}")
    b.free()
