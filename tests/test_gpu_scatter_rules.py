"""The current scatter where its rules change: steps on both sides of leaving the
matrix-instruction kernel (thermal plasmas that leave it after a step, by the turns of its
groups or by pieces outside its tile; dense ones that keep it), and blocks in contiguous
runs per XCD (131,072 particles and more on up to 4096 cells), with numbers of blocks that
are and are not a multiple of 8; spans of dense plasmas.  Whole steps against the oracle in fixed-iteration mode, at
1e-12 of the velocity, displacement, current and field scales (the bar of the whole-step
parity tests)."""
import pytest

import oracle as O
from paper_2606_15035_amd import ecpic as E
from tests.test_gpu_parity import both, compare_states, gpu, gpu_cfg  # noqa: F401
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


@pytest.mark.parametrize("np_,r,chunk", [
    (131071, 1, 0), (131072, 1, 0),
    (135169, 1, 2048),   # 67 blocks
    (131073, 2, 0), (131073, 3, 0),
    (200001, 2, 0),      # 48 per cell and more: the matrix-instruction kernel
])
def test_scatter_blocks_by_xcd(np_, r, chunk):
    wl = plasma((16, 16, 16), np_, r, 0.2, seed=np_ + r)
    g, o = both(wl, tol=0.0, pmax=1, scatter_chunk=chunk)
    g.picard_step()
    o.step()
    compare_states(wl, g, o, f"scatter by XCD {np_} r={r}")


# more than 16384 particles under the lanes of a block: 1024 per cell
@pytest.mark.parametrize("r,kw", [(1, {}), (3, {}), (2, dict(sort_interval=2)),
                                  (2, dict(split=False, quad_points=4))])
def test_scatter_wide_span(r, kw):
    wl = plasma((8, 8, 4), 262145, r, 0.2, seed=r)
    g = E.Sim(gpu_cfg(wl, tol=0.0, pmax=1, **kw), wl.np)
    okw = dict(wl.cfg_kwargs(), tol=0.0, pmax=1)
    if "split" in kw:
        okw.update(split=False, nq=4)
    o = O.OracleSim(O.make_cfg(**okw), wl.np)
    for s in (g, o):
        s.init_particles(wl.x, wl.v, wl.q, wl.m, wl.n0)
    g.picard_step()
    o.step()
    compare_states(wl, g, o, f"scatter wide span r={r} {kw}")
