"""A simulation that is given another set of particles after it has stepped: the
particles' species travel with them whatever arrays the earlier steps' sort moved.
FP64 against the oracle at the bar of the whole-step parity tests, mixed bitwise
against a new simulation of the same particles.
"""
import numpy as np
import pytest

import oracle as O
from mixed_storage import to_storage
from paper_2606_15035_amd import ecpic as E
from paper_2606_15035_amd import workloads as W
from tests.test_gpu_parity import compare_states, gpu, gpu_cfg, orc_cfg  # noqa: F401

pytestmark = pytest.mark.gpu

N, L = (8, 8, 4), (1.0, 1.0, 0.5)


def electron_ion(seed):
    wl = W.electron_ion(N, L, 3000, r=2, dt=0.25, vth=0.06, drift=(0.05, -0.02, 0.01), seed=seed)
    # species in an order of their own in every seed
    p = np.random.default_rng(seed).permutation(wl.np)
    wl.x, wl.v, wl.species = wl.x[:, p], wl.v[:, p], wl.species[p]
    return wl


def init(sim, wl):
    sim.init_species(wl.x, wl.v, wl.species, wl.qs, wl.ms, wl.n0)


@pytest.mark.parametrize("precision", [E.FP64, E.MIXED])
@pytest.mark.parametrize("before", ["one species", "two species", "restored"])
def test_species_after_earlier_steps(before, precision):
    wl = electron_ion(7)
    if precision == E.MIXED:
        wl.x, wl.v = to_storage(wl, wl.x, wl.v)
    cfg = gpu_cfg(wl, tol=0.0, pmax=3, precision=precision)
    g = E.Sim(cfg, wl.np)
    if before == "two species":
        init(g, electron_ion(8))
    else:
        one = W.random_plasma(N, L, wl.np, r=2, dt=wl.dt, vth=0.06, seed=9)
        g.init_particles(one.x, one.v, one.q, one.m, one.n0)
    for _ in range(3):  # every arrangement of the stores has been sorted once
        g.picard_step()
    fresh = E.Sim(cfg, wl.np)
    init(fresh, wl)
    if before == "restored":
        g.restore(fresh.checkpoint())
    else:
        init(g, wl)
    o = O.OracleSim(orc_cfg(wl, tol=0.0, pmax=3), wl.np)
    o.init_species(wl.x, wl.v, wl.species, wl.qs, wl.ms, wl.n0)
    for step in range(3):
        g.picard_step()
        if precision == E.FP64:
            o.step()
            compare_states(wl, g, o, f"after {before}, step {step}")
        else:
            fresh.picard_step()
            a, b = g.get_state(), fresh.get_state()
            for k in ("x", "v", "vprev", "fields"):
                assert np.array_equal(a[k], b[k]), (k, step)
