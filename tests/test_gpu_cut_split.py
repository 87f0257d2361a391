"""Few long vectors: both operands split in two launches along the inner dimension, at the edges of its pieces (512 positions of 16
columns, 2048 of 4 rows), against the oracle in full."""
import numpy as np
import pytest

import oracle
from paper_2409_13313_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2409_13313_amd import ozimmu
    return ozimmu


def padded(x, pad):
    rows, cols = x.shape
    v = torch.full((rows, cols + pad), float("nan"), dtype=torch.float64, device="cuda")[:, :cols]
    v.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return v


@pytest.mark.parametrize("m,n,p,k", [(1, 6145, 1, 3), (5, 8192, 17, 8), (4, 8191, 16, 14), (3, 6656, 15, 9), (33, 12289, 31, 8),
                                     (2, 40000, 3, 7), (40, 7200, 20, 16), (7, 140001, 18, 4)])
def test_cut_split(oz, m, n, p, k):
    A, B = inputs.phi_pair(m, n, p, 2.0, seed=601)
    A[:, n // 3:] *= 2.0 ** -30            # the maxima of a vector's pieces differ, those of the last piece lowest
    B[n // 3:] *= 2.0 ** -30
    A[m - 1, n - 1], B[n - 1, p - 1] = 2.0 ** 40, -2.0 ** 35
    if m > 3 and p > 3:
        A[1], B[:, 2] = 0.0, 0.0
    want = oracle.dgemm(A, B, k)
    assert oz.SPLIT_WAYS[oz.choose(m, n, p, k).split_way] == "cut"
    ws = oz.alloc_workspace(m, n, p, k)
    ws.fill_(0xA7)
    assert np.array_equal(oz.dgemm(padded(A, 1), padded(B, 3), k, workspace=ws).cpu().numpy(), want)
    for ta in (False, True):               # rows and columns, either operand
        for tb in (False, True):
            C = padded(np.zeros((m, p)), 1)
            oz.gemm_ex(ta, tb, 1.0, padded(A.T if ta else A, 2), padded(B.T if tb else B, 0), 0.0, C, k)
            assert np.array_equal(C.cpu().numpy(), want), (ta, tb)
    if k <= 9:
        want = oracle.dgemm_variant(A, B, k, "bitmask", "grouped")
        assert np.array_equal(oz.dgemm_variant(padded(A, 0), padded(B, 0), k, "bitmask", "grouped").cpu().numpy(), want)
