"""The plans of small states are those of the default knobs: a knob of the pass
shapes that is set keeps the plan and the launches it always had."""
import numpy as np
import pytest

import workloads
from parity import C64, C128, assert_parity

pytestmark = pytest.mark.gpu

KNOBS = [("qft.threads", 256), ("qft.threads", 512), ("qft.round_bits", 5), ("qft.col_rows", 1),
         ("qft.col_rows", 2), ("qft.col_max", 7), ("qft.lds_bits", 12)]


def passes(qs_lib, n, dtype, a, want):
    with qs_lib.State(n, dtype) as st:
        st.set_amplitudes(a)
        st.profile_start()
        st.qft()
        stats = st.profile_stop()
        assert_parity(st.amplitudes(), want, dtype)
    return sum(s["launches"] for s in stats.values())


@pytest.mark.parametrize("dtype,n", [(C64, 13), (C64, 22), (C128, 14), (C128, 21)])
def test_a_set_knob_keeps_its_plan(qs_lib, dtype, n):
    a = workloads.gaussian_state(n, n)
    want = np.fft.ifft(a, norm="ortho")
    passes(qs_lib, n, dtype, a, want)
    for key, value in KNOBS:
        saved = qs_lib.tune_get(key)
        qs_lib.tune_set(key, value)
        try:
            count = passes(qs_lib, n, dtype, a, want)
        finally:
            qs_lib.tune_set(key, saved)
        # a contiguous tile of 12 bits, then strided passes of 8 (or 7)
        per = 7 if key == "qft.col_max" else 8
        assert count == 1 + -(-(n - 12) // per), (key, value)
