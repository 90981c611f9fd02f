"""The gather's order of particles in blocks of several batches: whole steps
against the oracle in fixed-iteration mode, at 1e-12 of the velocity,
displacement, current and field scales (the bar of the whole-step parity tests;
the order changes no particle's arithmetic).  Orbits cross up to about six
knots; the counts leave a last block that is not full."""
import pytest

import oracle as O
from paper_2606_15035_amd import ecpic as E
from tests.test_gpu_parity import both, compare_states, gpu, gpu_cfg  # noqa: F401
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


# One batch per block: 40,960 is the last count with four lanes per particle,
# 40,961 the first with one; meshes in LDS whole (512 nodes) and node boxes
# (4096 nodes), whose far orbits take the list (four lanes at any count).
@pytest.mark.parametrize("r", [1, 2, 3])
@pytest.mark.parametrize("n,np_,vth", [
    ((8, 8, 8), 40960, 0.5),
    ((8, 8, 8), 40961, 0.5),
    ((16, 16, 16), 4097, 1.5),
    ((16, 16, 16), 40961, 1.5),
])
def test_gather_lanes_step_parity(n, np_, r, vth):
    wl = plasma(n, np_, r, vth, seed=np_ + r)
    g, o = both(wl, tol=0.0, pmax=1)
    g.picard_step()
    o.step()
    compare_states(wl, g, o, f"gather lanes {n} {np_} r={r}")


@pytest.mark.parametrize("np_", [1, 4097, 40961])
def test_gather_lanes_unsplit(np_):
    wl = plasma((16, 16, 16), np_, 2, 1.0, seed=np_)
    g = E.Sim(gpu_cfg(wl, tol=0.0, pmax=1, split=False, quad_points=6), wl.np)
    o = O.OracleSim(O.make_cfg(**dict(wl.cfg_kwargs(), tol=0.0, pmax=1, split=False, nq=6)), wl.np)
    for s in (g, o):
        s.init_particles(wl.x, wl.v, wl.q, wl.m, wl.n0)
    g.picard_step()
    o.step()
    compare_states(wl, g, o, f"gather lanes unsplit {np_}")
