"""The current scatter at the edges of its blocks, tiles and groups: whole steps
against the oracle in fixed-iteration mode, at 1e-12 of the velocity,
displacement, current and field scales (the bar of the whole-step parity
tests: FP64 sums of at most 81 terms per node and particle, in another order).
"""
import numpy as np
import pytest

from paper_2606_15035_amd import workloads as W
from tests.test_gpu_parity import both, compare_states, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def plasma(n, np_, r, vth, seed, dt=0.2):
    L = tuple(0.125 * k for k in n)
    return W.random_plasma(n, L, np_, r=r, dt=dt, vth=vth, drift=(0.05, -0.03, 0.02), seed=seed)


# n, particles, degree, thermal speed (cells per step = 1.6 vth), scatter_chunk
@pytest.mark.parametrize("n,np_,r,vth,chunk", [
    # matrix-instruction kernel (quadratic, 48 per cell and more): smallest mesh,
    # whose boxes wrap; counts one off a wavefront, a block, a chunk
    ((4, 4, 4), 3073, 2, 0.05, 0),
    ((8, 4, 4), 8191, 2, 0.05, 0),
    ((8, 8, 8), 48 * 512, 2, 0.05, 0),       # the first count it takes
    ((8, 8, 8), 48 * 512 - 1, 2, 0.05, 0),   # the last one it does not
    ((8, 8, 8), 33001, 2, 0.05, 4096),
    # orbits of several cells: groups of one particle, pieces outside the tile
    ((16, 8, 8), 50001, 2, 1.5, 0),
    ((16, 8, 8), 50001, 2, 1.5, 4096),
    # additions per lane: short chunks, clipped node boxes, far pieces
    ((16, 8, 8), 257, 2, 0.05, 0),
    ((16, 16, 16), 9001, 2, 1.5, 0),
    ((16, 16, 16), 9001, 1, 1.5, 0),
    ((16, 16, 16), 9001, 3, 1.5, 0),
])
def test_scatter_step_parity(n, np_, r, vth, chunk):
    wl = plasma(n, np_, r, vth, seed=np_)
    g, o = both(wl, tol=0.0, pmax=2, scatter_chunk=chunk)
    for step in range(2):
        g.picard_step()
        o.step()
        compare_states(wl, g, o, f"scatter {n} {np_} r={r} vth={vth} chunk={chunk} step {step}")


def test_scatter_two_species_dense():
    """Species coefficients in the matrix-instruction kernel: 56 particles per
    cell, electrons and ions."""
    n = (8, 4, 8)
    wl = W.electron_ion(n, tuple(0.125 * k for k in n), 56 * 256, r=2, dt=0.2, vth=0.1,
                        drift=(0.05, 0.0, 0.0))
    import oracle as O
    from tests.test_gpu_parity import E, gpu_cfg, orc_cfg
    g = E.Sim(gpu_cfg(wl, tol=0.0, pmax=2), wl.np)
    g.init_species(wl.x, wl.v, wl.species, wl.qs, wl.ms, 0.0)
    o = O.OracleSim(orc_cfg(wl, tol=0.0, pmax=2), wl.np)
    o.init_species(wl.x, wl.v, wl.species, wl.qs, wl.ms, 0.0)
    for step in range(2):
        g.picard_step()
        o.step()
        compare_states(wl, g, o, f"two species step {step}")
    assert np.isfinite(g.get_current()).all()
