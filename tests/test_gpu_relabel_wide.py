"""A relabelled ket with more tiles than a launch has workgroups (31 qubits,
16 GiB): the exchange strides through them. Exact: amplitudes only move."""
import pytest

from parity import C64

pytestmark = pytest.mark.gpu


def test_reversal_strides_over_tiles(qs_lib):
    n = 31
    with qs_lib.State(n, C64) as a, qs_lib.State(n, C64) as b:
        for x in (1, (1 << 30) | 5, 0x2AAAAAAB, 0x7FFFFFFE):
            rev = int(format(x, f"0{n}b")[::-1], 2)
            a.set_basis(x)
            for i in range(n // 2):
                a.apply_swap(i, n - 1 - i)
            b.set_basis(rev)
            assert a.inner(b) == 1.0
