"""The adjoint's push terms in blocks of several particles per lane, on a small mesh with a
last block that is not full.  Against the oracle's adjoint with the same number of transposed
iterations (a loose tolerance: the serial oracle takes seconds for each), from any v^{n+1},
which need not be a converged one; the bar of the adjoint parity tests, 1e-10 of each
output's largest entry.
"""
import numpy as np
import pytest

import oracle as O
from paper_2606_15035_amd import workloads as W
from tests.test_gpu_adjoint import gpu, gpu_sim, log, rel  # noqa: F401

pytestmark = pytest.mark.gpu


def compare_few_iterations(n, np_, vth):
    wl = W.random_plasma(n, tuple(0.125 * k for k in n), np_, r=2, dt=0.2, vth=vth,
                         drift=(0.05, -0.03, 0.02), seed=np_)
    rng = np.random.default_rng(np_)
    F = 0.01 * W.random_fields(n, 9, seed=np_ + 1)
    x, v = wl.x, wl.v
    w = v + 0.02 * rng.normal(size=v.shape)
    lx1, lv1, lF1 = rng.normal(size=x.shape), rng.normal(size=v.shape), rng.normal(size=F.shape)
    o = O.OracleSim(O.make_cfg(wl.n, wl.L, wl.dt, r=2), wl.np)
    o.init_particles(x, v, wl.q, wl.m, 1.0)
    ox, ov, oF, oit = o.adjoint_step(x, v, w, F, lx1, lv1, lF1, tol=0.5)
    gx, gv, gF, info = gpu_sim(wl).adjoint_step(x, v, w, F, lx1, lv1, lF1, tol=0.5)
    gx, gv, gF = (t.cpu().numpy() for t in (gx, gv, gF))
    log(f"{n} {np_}: {oit} iterations, GPU {info}; rel diff x {rel(gx, ox):.2e} "
        f"v {rel(gv, ov):.2e} F {rel(gF, oF):.2e}")
    assert info["iters"] == oit
    assert rel(gx, ox) <= 1e-10 and rel(gv, ov) <= 1e-10 and rel(gF, oF) <= 1e-10


# two and four particles per lane; orbits of half a cell and of two
@pytest.mark.parametrize("np_,vth", [(262145, 0.3), (524289, 0.3), (262145, 1.2)])
def test_adjoint_blocks_of_several_particles_per_lane(np_, vth):
    compare_few_iterations((8, 8, 8), np_, vth)
