"""A step that failed leaves nothing behind for the next one: the same simulation,
given slow particles, steps as a new one does.  FP64 to 1e-12 of each quantity's
largest value (the order of the atomic additions), mixed bitwise.
"""
import numpy as np
import pytest

from paper_2606_15035_amd import ecpic as E
from paper_2606_15035_amd import workloads as W
from mixed_storage import to_storage
from tests.test_gpu_parity import gpu, gpu_cfg  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,scale,speed,text", [
    (E.FP64, 0.0, 80.0, "knots"),          # 160 cells of orbit per step
    (E.MIXED, 2.0 ** 40, 80.0, "knots"),
    (E.MIXED, 2.0 ** 52, 0.5, "fixed-point"),  # 2^51 quanta per particle
    (E.FP64, 0.0, np.inf, "non-finite"),
])
def test_step_after_a_failed_step(precision, scale, speed, text):
    wl = W.random_plasma((8, 8, 4), (1.0, 1.0, 0.5), 500, r=2, dt=0.25, vth=0.02, seed=43)
    x, v = to_storage(wl, wl.x, wl.v)
    fast = v.copy()
    fast[0, ::7] += speed
    kw = dict(tol=0.0, pmax=2, precision=precision, fixed_point_scale=scale)
    g = E.Sim(gpu_cfg(wl, **kw), wl.np)
    g.init_particles(x, v, wl.q, wl.m, wl.n0)
    fields = g.get_state()["fields"]
    g.set_state(x, fast, fast, fields, wl.q, wl.m)
    with pytest.raises(E.EcpicError) as ei:
        g.picard_step()
    assert text in str(ei.value)
    fresh = E.Sim(gpu_cfg(wl, **kw), wl.np)
    fresh.init_particles(x, v, wl.q, wl.m, wl.n0)
    for s in (g, fresh):
        s.set_state(x, v, v, fields, wl.q, wl.m)
    for _ in range(2):
        assert g.picard_step()["iters"] == fresh.picard_step()["iters"] == 3
        a, b = g.get_state(), fresh.get_state()
        for k in ("x", "v", "vprev", "fields"):
            if precision == E.MIXED:
                assert np.array_equal(a[k], b[k]), k
            else:
                d = a[k] - b[k]
                if k == "x":
                    d -= np.round(d / np.reshape(wl.L, (3, 1))) * np.reshape(wl.L, (3, 1))
                assert np.abs(d).max() <= 1e-12 * np.abs(b[k]).max(), k
