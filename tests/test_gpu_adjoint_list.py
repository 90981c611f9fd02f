"""The adjoint's push terms of particles from global memory: sparse plasmas whose blocks'
node boxes do not fit (fewer than 0.3 particles per cell: 128 of a block over more than 400
cells), at lists shorter than the lanes of their kernel and at one longer.  Against the
oracle's adjoint, as the tests of the blocks' edges.
"""
import pytest

from tests import test_gpu_adjoint_blocks as blocks
from tests.test_gpu_adjoint import gpu  # noqa: F401
from tests.test_gpu_adjoint_large import compare_few_iterations

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,np_,vth", [((16, 16, 16), 1000, 0.05), ((16, 16, 16), 1025, 1.0)])
def test_adjoint_list(n, np_, vth):
    blocks.test_push_adjoint_blocks(n, np_, vth)


def test_adjoint_list_longer_than_its_lanes():
    compare_few_iterations((64, 64, 64), 66001, 0.05)  # 256 blocks of 256 lanes
