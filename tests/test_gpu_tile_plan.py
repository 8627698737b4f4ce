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


@pytest.mark.parametrize("dtype", [C64, C128])
def test_batch_of_every_width(qs_lib, dtype):
    """Kets of 1 to 14 qubits in one arena: those smaller than a tile are one
    pass each, alone in their tile, and leave their neighbours alone."""
    import workloads as w
    widths = [3, 14, 1, 2, 11, 12, 5, 10, 13, 4, 6, 9, 7, 8, 1, 11]
    lists = [w.random_circuit(n, 4, 70 + i) if n > 1 else [("h", 0), ("u3", 0, 0.3, 0.1, 0.2)]
             for i, n in enumerate(widths)]
    circs = [qs_lib.Circuit(n).add_gates(x) for n, x in zip(widths, lists)]
    b = qs_lib.Batch(widths, dtype)
    for again in range(2):
        b.reset()
        b.run(circs)
        for i, (n, gates) in enumerate(zip(widths, lists)):
            assert_parity(b.amplitudes(i), dense.run_circuit(dense.zero_state(n), n, gates), dtype,
                          f"ket {i} n={n}")
    b.free()


def test_batch_leaves_the_blocks_of_its_width(qs_lib):
    """A circuit that a batch ran as tile passes answers for its blocks as if
    the batch had planned them, and runs as them when asked to."""
    n = 12
    gates = workloads.random_circuit(n, 4, 3)
    c = qs_lib.Circuit(n).add_gates(gates)
    assert c.info()["blocks"] == -1
    b = qs_lib.Batch([n], C64)
    b.run([c], 3)
    ref = qs_lib.Circuit(n).add_gates(gates).plan(3)
    assert c.info() == ref.info()
    assert c.block(0)[0] == ref.block(0)[0]
    b.reset()
    b.run([c], 3)
    want = dense.run_circuit(dense.zero_state(n), n, gates)
    assert_parity(b.amplitudes(0), want, C64)
    b.free()
    c.use_tiles(False)
    with qs_lib.State(n, C64) as st:
        st.run(c)
        assert_parity(st.amplitudes(), want, C64)
    c.add_gates([("h", 0)])
    assert c.info()["blocks"] == -1
