"""The allocation-free adjoint at the counts that include/ecpic.h names as fitting the
library's own array, against the adjoint with a caller's workspace."""
import pytest

from tests.test_zz_no_alloc import compare, converged_case, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,np_", [((32, 32, 32), 76000), ((16, 16, 16), 167000)])
def test_noalloc_adjoint_at_the_stated_counts(n, np_):
    compare(*converged_case(n, tuple(k / 16 for k in n), np_, seed=5), "stated count")
