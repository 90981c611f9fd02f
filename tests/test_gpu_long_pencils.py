"""The field transforms at 256 points, the longest that a mesh may have: as the x pencils of
the field solve (two per block), in planes that fit LDS, and where a plane does not fit as
strided passes and as the rows behind the gather buffer (two per block).  The Fourier
symbols and the spectra against numpy's transforms, to 1e-12 of each field's largest entry
(the bar of the field tests: log2 N roundings of the largest entry).
"""
import numpy as np
import pytest

from paper_2606_15035_amd import ecpic as E
from paper_2606_15035_amd import workloads as W
from tests.test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def symbols(n, L):
    out = []
    for a in range(3):
        m = np.fft.fftfreq(n[a], 1.0 / n[a])
        k = 2 * np.pi * m / L[a]
        k[n[a] // 2] = 0.0  # Nyquist
        out.append(k.reshape([-1 if b == a else 1 for b in range(3)]))
    return out


def solve(F, J, n, L, dt):
    """One continuity + Crank-Nicolson step of the nine fields (kappa = sigma = 1)."""
    fh = np.fft.fftn(F, axes=(1, 2, 3))
    jh = np.fft.fftn(J, axes=(1, 2, 3))
    k = symbols(n, L)
    w2 = sum(q * q for q in k)
    a = 0.5 * dt
    rho1 = fh[8] - dt * 1j * sum(k[l] * jh[l] for l in range(3))
    out = np.empty_like(fh)
    for val, rate, src in ((0, 1, 0.5 * (fh[8] + rho1)),) + tuple(
            (2 + l, 5 + l, jh[l]) for l in range(3)):
        r1 = ((1 - a * a * w2) * fh[rate] - 2 * a * w2 * fh[val] + dt * src) / (1 + a * a * w2)
        out[val], out[rate] = fh[val] + a * (fh[rate] + r1), r1
    out[8] = rho1
    return np.fft.ifftn(out, axes=(1, 2, 3)).real


@pytest.mark.parametrize("n", [(256, 4, 4), (4, 256, 4), (4, 4, 256), (256, 32, 4), (4, 16, 256),
                               (4, 32, 256), (4, 256, 32), (8, 256, 256)])
def test_field_solve_with_256_points(n):
    import torch
    L, dt = tuple(0.1 * k for k in n), 0.05
    g = E.Sim(E.make_config(n, L, dt, r=2), 0)
    rng = np.random.default_rng(n[0] + n[2])
    F = W.random_fields(n, 9, seed=3) + 0.1 * rng.normal(size=(9,) + n)
    J = rng.normal(size=(3,) + n)
    g.set_state(fields=F, q=-1.0, m=1.0)
    back = g.get_state()["fields"]
    assert np.abs(back - F).max() <= 1e-12 * np.abs(F).max()
    ref = F
    for step in range(2):  # the second from the first's spectra
        g.field_solve(torch.as_tensor(J, device="cuda"))
        ref = solve(ref, J, n, L, dt)
        out = g.get_state()["fields"]
        for f in range(9):
            err = np.abs(out[f] - ref[f]).max() / np.abs(ref[f]).max()
            assert err <= 1e-12, (step, f, err)


@pytest.mark.parametrize("n", [(256, 4, 4), (4, 32, 256), (4, 256, 32)])
def test_step_with_256_points(n):
    """The gather buffer behind the transforms: a step of particles against the oracle."""
    from tests.test_gpu_parity import both, compare_states
    from tests.test_gpu_scatter import plasma
    wl = plasma(n, 5001, 2, 0.2, seed=n[0])
    g, o = both(wl, tol=0.0, pmax=1)
    for step in range(2):
        g.picard_step()
        o.step()
        compare_states(wl, g, o, f"256 points {n} step {step}")
