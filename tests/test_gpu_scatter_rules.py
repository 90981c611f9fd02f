"""The current scatter where its rules change: steps on both sides of leaving the
matrix-instruction kernel (thermal plasmas that leave it after a step, by the turns of its
groups or by pieces outside its tile; dense ones that keep it).  Whole steps against the oracle in fixed-iteration mode, at
1e-12 of the velocity, displacement, current and field scales (the bar of the whole-step
parity tests)."""
import pytest

from tests.test_gpu_parity import both, compare_states, gpu  # noqa: F401
from tests.test_gpu_scatter import plasma

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,np_,vth,steps", [
    ((8, 8, 4), 64 * 256 + 1, 0.2, 3),
    ((4, 4, 4), 511 * 64, 0.05, 2), ((4, 4, 4), 513 * 64, 0.05, 2),
    ((8, 8, 4), 513 * 256 + 1, 1.2, 2),
])
def test_scatter_kernel_change(n, np_, vth, steps):
    wl = plasma(n, np_, 2, vth, seed=np_)
    g, o = both(wl, tol=0.0, pmax=1)
    for step in range(steps):
        g.picard_step()
        o.step()
        compare_states(wl, g, o, f"scatter rule {n} {np_} vth={vth} step {step}")
