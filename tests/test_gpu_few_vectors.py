"""GPU parity of the split of few vectors, whose slices stay in the L2 that the product's only tile reads (the others are written through it): the
last number of vectors that does and the first that does not, rows and columns on either side, and a second call in the same workspace, which
may find nothing of the first."""
import numpy as np
import pytest

import oracle
from paper_2409_13313_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# rows: eight workgroups of 4, 2 or 1; columns: four of 16 (up to 256 positions) or 4
@pytest.mark.parametrize("n,k,split,transA,transB", [
    *((n, k, "rn", ta, tb) for n, k in ((300, 3), (2047, 4), (2300, 16)) for ta in (False, True) for tb in (False, True)),
    *((n, k, "bitmask", False, False) for n, k in ((200, 5), (1030, 9), (5000, 3)))])
def test_few_vectors(n, k, split, transA, transB):
    from paper_2409_13313_amd import ozimmu as oz
    for m, p in ((1, 1), (8, 16), (9, 17), (16, 16), (17, 4), (32, 16), (33, 16), (32, 64), (5, 65)):
        ws = torch.full((oz.workspace_bytes(m, n, p, k),), 0x5A, dtype=torch.uint8, device="cuda")
        for seed in (901, 902):
            A, B = inputs.phi_pair(m, n, p, 1.0, seed=seed)
            want = oracle.dgemm_variant(A, B, k, split, "grouped")
            dA = torch.from_numpy(np.ascontiguousarray(A.T if transA else A)).cuda()
            dB = torch.from_numpy(np.ascontiguousarray(B.T if transB else B)).cuda()
            D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
            if transA or transB:
                oz.gemm_ex(transA, transB, 1.0, dA, dB, 0.0, D[:, :p], k, workspace=ws)
            else:
                oz.dgemm_variant(dA, dB, k, split, "grouped", D=D[:, :p], workspace=ws)
            assert np.array_equal(D[:, :p].cpu().numpy(), want) and bool(torch.isnan(D[:, p]).all()), (m, p, seed)
