"""Vectors that leave the device: in the caller's order, and no concern of an error
that another call of the thread has left behind (the copy makes no use of it).
"""
import numpy as np
import pytest

from paper_2510_12011_amd import inputs

pytestmark = pytest.mark.gpu


def test_an_error_of_another_call_is_left_alone():
    from paper_2510_12011_amd import _lib as L, sim
    spec = inputs.small_box()
    s = sim.from_spec(spec)
    s.run(20)
    state, times = s.get_state(), s.times()
    print("[case] error left", flush=True)
    for get in (s.get_state, s.times):
        assert L.lib().hipSetDevice(99) != 0     # no such device: an error for the caller
        got = get()
        assert L.lib().hipGetLastError() != 0    # still there
        ref = state if isinstance(got, dict) else times
        for k in (ref if isinstance(ref, dict) else range(2)):
            assert np.array_equal(got[k], ref[k])
