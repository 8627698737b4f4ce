"""Batches of kets that can only take pair rounds: where every long one has many
gates on few qubits they run as blocks, beside a ket of random layers as passes
with it. Against the oracle, with the launches of either form."""
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


@pytest.mark.parametrize("dtype,widths", [(C64, [4, 7, 9, 11]), (C128, [4, 7, 11, 13])])
@pytest.mark.parametrize("beside", [False, True])
def test_few_qubits(qs_lib, dtype, widths, beside):
    g = np.random.default_rng(len(widths) + beside)
    lists = [on([int(x) for x in g.permutation(n)[:3 if i == 0 else 4]], 60, g)
             for i, n in enumerate(widths)]
    widths = list(widths)
    if beside:  # one pass, as many rounds as the others
        widths.append(9)
        lists.append(workloads.random_circuit(9, 14, 5))
    circs = [qs_lib.Circuit(n).add_gates(x) for n, x in zip(widths, lists)]
    b = qs_lib.Batch(widths, dtype)
    for again in range(2):
        b.reset()
        b.run(circs, 4)
        # blocks on three and on four qubits, or one pass of every ket
        assert b.info()["launches"] == (1 if beside else 2)
        for i, (n, x) in enumerate(zip(widths, lists)):
            assert_parity(b.amplitudes(i), dense.run_circuit(dense.zero_state(n), n, x), dtype,
                          f"ket {i} n={n}")
    b.free()
    for c in circs:
        c.free()
