"""The adjoint's workspace at the sizes that include/ecpic.h states: 372 B per particle
beside the mesh arrays, and the counts named there as fitting the library's own array.
Sizing runs on the host."""
import os

import pytest

from paper_2606_15035_amd import ecpic as E


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(E.LIB_PATH):
        from paper_2606_15035_amd import build as B
        B.build()


def need(n, np_):
    return E.adjoint_workspace_bytes(E.make_config(n=n, L=(1.0, 1.0, 1.0), dt=0.2, r=2), np_)


@pytest.mark.parametrize("n,np_", [((32, 32, 32), 76000), ((16, 16, 16), 167000)])
def test_stated_counts_fit_the_static_array(n, np_):
    assert need(n, np_) <= E.STATIC_SCRATCH_BYTES


@pytest.mark.parametrize("n", [(4, 4, 4), (16, 16, 16), (64, 32, 16)])
def test_bytes_per_particle(n):
    for base, more in ((1, 1000), (1000, 99999), (167000, 1000000)):
        # 19 arrays, each padded to 256 bytes
        assert need(n, base + more) - need(n, base) <= 372 * more + 19 * 256
