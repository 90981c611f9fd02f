"""The adjoint's order of particles inside the segments that its lanes take: segments of
256 (several wavefronts of particles each), 8 and 16, a last one that is not full,
orbits that cross several knots.  Against the oracle's adjoint, as the tests of the
blocks' edges.
"""
import pytest

from tests.test_gpu_adjoint import gpu  # noqa: F401
from tests import test_gpu_adjoint_blocks as blocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,np_,vth", [
    ((4, 4, 4), 98401, 0.5),      # 1537 per cell: segments of 256
    ((32, 32, 16), 98401, 0.5),   # 6 per cell: segments of 8
    ((16, 8, 8), 2049, 0.5),      # four lanes per particle: segments of 16
])
def test_adjoint_segments(n, np_, vth):
    blocks.test_push_adjoint_blocks(n, np_, vth)
