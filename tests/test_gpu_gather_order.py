"""The gather's order of particles in blocks of several batches: whole steps
against the oracle in fixed-iteration mode, at 1e-12 of the velocity,
displacement, current and field scales (the bar of the whole-step parity tests;
the order changes no particle's arithmetic).  Orbits cross up to about six
knots; the counts leave a last block that is not full."""
import pytest

from tests.test_gpu_parity import both, compare_states, gpu  # noqa: F401
from tests.test_gpu_scatter import plasma

pytestmark = pytest.mark.gpu


# 524,288 is the first count with two batches of 256 per block
@pytest.mark.parametrize("np_,r", [(524288, 1), (524801, 2), (524801, 3)])
def test_ordered_gather_step_parity(np_, r):
    wl = plasma((16, 16, 16), np_, r, 0.5, seed=np_ + r)
    g, o = both(wl, tol=0.0, pmax=1)
    g.picard_step()
    o.step()
    compare_states(wl, g, o, f"ordered gather {np_} r={r}")
