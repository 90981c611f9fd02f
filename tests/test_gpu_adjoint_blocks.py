"""The adjoint's push terms at the edges of their blocks and tiles: four lanes per
particle (up to 98,304 particles) and one, counts one off a block, orbits beyond
a block's node box, meshes whose half period the box reaches.  Against the
oracle's adjoint at the bar of the adjoint parity tests (1e-10 of each output's
largest entry: the same linear system solved to 1e-14, sums in another order).
"""
import numpy as np
import pytest

import oracle as O
from paper_2606_15035_amd import workloads as W
from tests.test_gpu_adjoint import gpu, gpu_sim, log, rel  # noqa: F401

pytestmark = pytest.mark.gpu


# n, particles, thermal speed (cells per step = 1.6 vth); fields weak enough that
# the step and its transpose converge at every speed
@pytest.mark.parametrize("n,np_,vth", [
    ((4, 4, 4), 1, 0.05),
    ((8, 8, 4), 127, 0.05),
    ((8, 8, 4), 129, 0.05),
    ((16, 16, 16), 4097, 0.05),   # blocks in two columns of a 16-cell period
    ((16, 8, 32), 1025, 0.05),    # fewer than one particle per cell: wide boxes
    ((16, 8, 8), 2047, 1.5),      # orbits of several cells: clipped boxes, the list
    ((8, 8, 8), 98305, 0.05),     # the first count with one lane per particle
])
def test_push_adjoint_blocks(n, np_, vth):
    L = tuple(0.125 * k for k in n)
    wl = W.random_plasma(n, L, np_, r=2, dt=0.2, vth=vth, drift=(0.05, -0.03, 0.02), seed=np_)
    F = 0.01 * W.random_fields(n, 9, seed=np_ + 1)
    x, v = wl.x, wl.v
    o = O.OracleSim(O.make_cfg(wl.n, wl.L, wl.dt, r=2, tol=0.0, pmax=12), wl.np)
    o.init_particles(x, v, wl.q, wl.m, 1.0)
    o.set_state(x, v, v, None, F, wl.q, wl.m)
    o.rebuild_P()
    o.step()
    w = o.get_state()["v"]
    rng = np.random.default_rng(np_ + 2)
    lx1, lv1, lF1 = rng.normal(size=x.shape), rng.normal(size=v.shape), rng.normal(size=F.shape)
    ox, ov, oF, oit = o.adjoint_step(x, v, w, F, lx1, lv1, lF1, tol=1e-14)
    g = gpu_sim(wl)
    gx, gv, gF, info = g.adjoint_step(x, v, w, F, lx1, lv1, lF1, tol=1e-14)
    gx, gv, gF = (t.cpu().numpy() for t in (gx, gv, gF))
    log(f"{n} {np_} vth={vth}: oracle {oit} iterations, GPU {info}; rel diff x {rel(gx, ox):.2e} "
        f"v {rel(gv, ov):.2e} F {rel(gF, oF):.2e}")
    assert info["converged"]
    assert rel(gx, ox) <= 1e-10 and rel(gv, ov) <= 1e-10 and rel(gF, oF) <= 1e-10
