"""The gather's blocks of four batches of 256 particles, which take their particles by the
knots that they cross: a whole step against the oracle in fixed-iteration mode, at 1e-12 of
the velocity, displacement, current and field scales (the bar of the whole-step parity
tests).  1,048,576 is the first such count; a last block that is not full."""
import pytest

from tests.test_gpu_parity import both, compare_states, gpu  # noqa: F401
from tests.test_gpu_scatter import plasma

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 2, 3])
def test_four_batches_step_parity(r):
    wl = plasma((16, 16, 16), 1048577, r, 0.5, seed=r)
    g, o = both(wl, tol=0.0, pmax=1)
    g.picard_step()
    o.step()
    compare_states(wl, g, o, f"four batches r={r}")
