"""The order of the particles of a scatter lane by the knots that they cross: whole
steps against the oracle in fixed-iteration mode, at 1e-12 of the velocity,
displacement, current and field scales (the bar of the whole-step parity tests:
the order changes no particle's arithmetic, only the order of the sums).  Orbits
cross several knots; last blocks that are not full.
"""
import pytest

from tests.test_gpu_parity import both, compare_states, gpu  # noqa: F401
from tests.test_gpu_scatter import plasma

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,np_,r,vth,chunk", [
    ((16, 8, 8), 9001, 1, 1.5, 2048),
    ((16, 8, 8), 9001, 1, 1.5, 4096),
    ((16, 8, 8), 9001, 2, 1.5, 2048),
    ((16, 8, 8), 9001, 2, 1.5, 4096),
    ((16, 8, 8), 9001, 3, 1.5, 2048),
    ((16, 16, 16), 2047, 2, 0.5, 2048),
    ((16, 16, 16), 1, 2, 0.5, 2048),
])
def test_scatter_lane_order(n, np_, r, vth, chunk):
    wl = plasma(n, np_, r, vth, seed=np_ + r)
    g, o = both(wl, tol=0.0, pmax=2, scatter_chunk=chunk)
    for step in range(2):
        g.picard_step()
        o.step()
        compare_states(wl, g, o, f"scatter lanes {n} {np_} r={r} chunk={chunk} step {step}")
