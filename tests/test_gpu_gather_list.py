"""The gather's list of particles taken from global memory: unsorted particles, whose
blocks list all of theirs at once, at lists of one entry, one below and one above the
length from which neighbouring entries go to a wavefront, and with a last block that is
not full.  Whole steps against the oracle in fixed-iteration mode, at 1e-12 of the
velocity, displacement, current and field scales (the bar of the whole-step parity
tests)."""
import pytest

from tests.test_gpu_parity import both, compare_states, gpu  # noqa: F401
from tests.test_gpu_scatter import plasma

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np_,r,vth", [
    (1, 2, 1.5),
    (32767, 2, 0.05), (32769, 2, 0.05),  # four lanes in both kernels
    (40961, 1, 0.5), (40961, 2, 0.5), (40961, 3, 0.5),
    (65537, 2, 1.5),
])
def test_unsorted_step_parity(np_, r, vth):
    wl = plasma((16, 16, 16), np_, r, vth, seed=np_ + r)
    g, o = both(wl, tol=0.0, pmax=1, sort_interval=-1)
    for step in range(2):
        g.picard_step()
        o.step()
        compare_states(wl, g, o, f"unsorted {np_} r={r} step {step}")
