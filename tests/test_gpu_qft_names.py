"""Every pass of a transform has a name in profiles, whatever its width."""
import pytest

from parity import C64, C128

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n", [(C64, 5), (C64, 13), (C64, 21), (C64, 22), (C64, 23), (C64, 25),
                                     (C128, 13), (C128, 20), (C128, 22), (C128, 24)])
def test_passes_are_named(qs_lib, dtype, n):
    with qs_lib.State(n, dtype) as st:
        st.profile_start()
        st.qft()
        st.qft(inverse=True)
        stats = st.profile_stop()
    assert "" not in stats and "qft_lds" in stats
    assert all(name.startswith("qft_") for name in stats)
    if (dtype, n) == (C64, 22):
        assert "qft_col9" in stats
