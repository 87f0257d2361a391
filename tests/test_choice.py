"""Which way the library runs a call, by its own choice (a host function: no GPU)."""
import os

import pytest

torch = pytest.importorskip("torch")
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_13313_amd", "libozimmu.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libozimmu.so not built")


@pytest.fixture(scope="module")
def oz():
    from paper_2409_13313_amd import ozimmu
    return ozimmu


@pytest.mark.parametrize("m,n,p", [(47, 11948, 48), (1, 4096, 1), (64, 20001, 97), (300, 5937, 174)])
@pytest.mark.parametrize("k", range(3, 17))
def test_one_scale_per_slice_is_never_cut_whatever_the_room(oz, m, n, p, k):
    # (the sums of cut tiles are added up with one exponent per row and column)
    assert oz.choose(m, n, p, k, "per_slice", "per_pair", workspace_bytes=1 << 34).parts == 1
    assert oz.choose(m, n, p, 3, "rn", "grouped", workspace_bytes=1 << 34).parts > 1
