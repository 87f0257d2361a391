"""GPU parity of the split with columns cut along the inner dimension (k_split_and_maxima, k_cut_columns): against the same product with the
operand stored by rows, which has no columns to cut, and the oracle; offsets, sums of the stored bytes, edges of groups and pieces."""
import numpy as np
import pytest

import oracle
from paper_2409_13313_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    from paper_2409_13313_amd import ozimmu
    return ozimmu


def check_corners(got, A, B, k, split):
    rows, cols = np.unique([0, A.shape[0] // 2, A.shape[0] - 1]), np.unique([0, 15, B.shape[1] // 2, B.shape[1] - 1])
    want = oracle.dgemm_variant(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), k, split, "grouped")
    assert np.array_equal(got.cpu().numpy()[np.ix_(rows, cols)], want)


# inner dimensions: whole pieces of 512, one more, one less, ends inside a step; columns: whole groups of 16 and not; rows that fit a
# workgroup's registers and (beyond 16384) do not, and of 2048 to 8192
@pytest.mark.parametrize("m,n,p,k,split", [
    (640, 14848, 256, 8, "rn"), (641, 14849, 255, 8, "rn"), (909, 14947, 85, 4, "bitmask"), (701, 16385, 1513, 5, "rn"), (523, 31111, 815, 8, "rn"),
    (130, 33000, 721, 20, "rn"), (2500, 10753, 130, 14, "bitmask"), (1900, 8192, 300, 16, "rn"), (1300, 8190, 901, 20, "rn")])
def test_columns_beside_rows(oz, m, n, p, k, split):
    assert oz.SPLIT_WAYS[oz.choose(m, n, p, k, split).split_way] == "cut_columns"
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=601)
    B[:, p // 3] = 0.0
    B[:, p // 2] *= 2.0 ** 300                       # (columns of any scale, an empty one)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    ws = oz.alloc_workspace(m, n, p, k)
    ws.fill_(0x5A)
    D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
    oz.dgemm_variant(dA, dB, k, split, "grouped", D=D[:, :p], workspace=ws)
    assert bool(torch.isnan(D[:, p]).all())
    check_corners(D[:, :p], A, B, k, split)
    if split == "rn":
        ref = torch.zeros((m, p), dtype=torch.float64, device="cuda")
        oz.gemm_ex(False, True, 1.0, dA, dB.t().contiguous(), 0.0, ref, k)
        assert torch.equal(D[:, :p], ref)


def test_two_operands_of_columns_and_a_graph(oz):
    m, n, p, k = 256, 40001, 700, 8
    A, B = inputs.phi_pair(m, n, p, 0.5, seed=602)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    At = dA.t().contiguous()
    ref = torch.zeros((m, p), dtype=torch.float64, device="cuda")
    oz.gemm_ex(False, True, 1.0, dA, dB.t().contiguous(), 0.0, ref, k)
    C = torch.zeros((m, p), dtype=torch.float64, device="cuda")
    ws = torch.empty(oz.workspace_bytes(m, n, p, k) + (64 << 20), dtype=torch.uint8, device="cuda")
    oz.gemm_ex(True, False, 1.0, At, dB, 0.0, C, k, workspace=ws)
    assert torch.equal(C, ref)
    check_corners(C, A, B, k, "rn")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        oz.gemm_ex(True, False, 1.0, At, dB, 0.0, C, k, workspace=ws)
    for _ in range(3):
        C.zero_()
        ws.fill_(0x33)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, ref)
