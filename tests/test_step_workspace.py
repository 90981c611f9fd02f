"""The step's workspace per particle: 24 B for the next pass's vbar (plain iteration), an
order of 1 B for the scatter and 2 B for the gather, and 1.3 B of node boxes and partial
sums per block of 256.  Sizing runs on the host."""
import os

import pytest

from paper_2606_15035_amd import ecpic as E


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(E.LIB_PATH):
        from paper_2606_15035_amd import build as B
        B.build()


@pytest.mark.parametrize("kw", [dict(n=(32, 32, 32)), dict(n=(64, 64, 64), precision=E.MIXED)])
def test_bytes_per_particle(kw):
    cfg = E.make_config(L=(1.0, 1.0, 1.0), dt=0.1, r=2, **kw)
    a, b = 2 ** 21, 2 ** 25
    per = (E.state_bytes(cfg, b)[1] - E.state_bytes(cfg, a)[1]) / (b - a)
    assert per <= 24 + 1 + 2 + 1.3
