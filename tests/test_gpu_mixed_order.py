"""The mixed form at counts and speeds where particles leave their gather block's node
box: its results do not depend on the order of the particles, bitwise, and with it not
on which of them a block leaves to the list.  Meshes of more nodes than the LDS holds
whole; 40,961 is the first count with one lane per particle, 524,801 has two batches
per block.  Strong fields and a fine quantum of the current, so that a last bit of a
velocity shows in the current.
"""
import numpy as np
import pytest

from mixed_storage import to_storage
from paper_2606_15035_amd import ecpic as E
from paper_2606_15035_amd import workloads as W
from tests.test_gpu_parity import gpu, gpu_cfg  # noqa: F401
from tests.test_gpu_scatter import plasma

pytestmark = pytest.mark.gpu


def run(wl, x, v, order, steps=2, **kw):
    g = E.Sim(gpu_cfg(wl, tol=0.0, precision=E.MIXED, fixed_point_scale=2.0 ** 46, **kw), wl.np)
    g.init_particles(x[:, order], v[:, order], wl.q, wl.m, wl.n0)
    g.set_state(fields=0.3 * W.random_fields(wl.n, 9, seed=7))
    for _ in range(steps):
        g.picard_step()
    s = g.get_state()
    out = [np.empty_like(s[k]) for k in ("x", "v", "vprev")]
    for o, k in zip(out, ("x", "v", "vprev")):
        o[:, order] = s[k]
    g_out = out + [s["fields"], g.get_current()]
    g.close()
    return g_out


# thermal speeds: 1.6 vth cells per step
@pytest.mark.parametrize("np_,r,vth", [
    (9001, 2, 1.5),
    (41001, 1, 1.5), (41001, 2, 0.5), (41001, 2, 1.5), (41001, 3, 1.5),
    (524801, 2, 1.5),
])
def test_mixed_step_does_not_depend_on_the_order(np_, r, vth):
    wl = plasma((16, 16, 16), np_, r, vth, seed=np_ + r)
    x, v = to_storage(wl, wl.x, wl.v)
    given = np.arange(np_)
    perm = np.random.Generator(np.random.PCG64(5)).permutation(np_)
    ref = run(wl, x, v, given, pmax=2)
    for order, sort in ((given, 0), (perm, 0), (given, -1)):
        out = run(wl, x, v, order, pmax=2, sort_interval=sort)
        for name, a, b in zip(("x", "v", "vprev", "fields", "J"), ref, out):
            assert np.array_equal(a, b), (name, sort, np.count_nonzero(a != b), a.size)


def test_unsorted_mixed_run_with_anderson_mixing_repeats_itself():
    """Never sorted, the mixed form with mixing over one difference takes its sums over
    the particles in the order in which they are given: two runs are the same bits."""
    wl = plasma((16, 16, 16), 41001, 2, 1.5, seed=3)
    x, v = to_storage(wl, wl.x, wl.v)
    given = np.arange(wl.np)
    a, b, c = (run(wl, x, v, given, pmax=4, sort_interval=-1, anderson=1) for _ in range(3))
    for name, u, w, t in zip(("x", "v", "vprev", "fields", "J"), a, b, c):
        assert np.array_equal(u, w) and np.array_equal(u, t), name
