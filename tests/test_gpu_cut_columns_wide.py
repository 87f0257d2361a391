"""GPU parity of the split with columns cut along the inner dimension where there are many columns, as the library chooses it: rows that fit a
workgroup's registers and (beyond 16384 positions) do not."""
import pytest

import test_gpu_cut_columns as cut_columns
from test_gpu_cut_columns import oz  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,p,k", [(501, 16385, 2105, 5), (300, 8190, 2101, 20)])
def test_many_columns_beside_rows(oz, m, n, p, k):
    cut_columns.test_columns_beside_rows(oz, m, n, p, k, "rn")
