"""GPU parity of the split kernels at the sizes where they can go wrong: the batches a workgroup walks when a vector does not
fit its registers (8 waves of 64 lanes with 16 or 64 elements each), the number of vectors per workgroup (1, 2, 4 rows;
4, 8, 16 columns), remainders of all of these, alignment, and the few long columns that are cut across workgroups.
Slices and exponents bit for bit against the oracle; the sums behind the slices through a product."""
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


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# (vectors, length): 4 rows / 2 rows / 1 row a workgroup; one batch and several; lengths around 64, 256, 512 and 8192
SHAPES = [(1, 1), (3, 63), (5, 64), (33, 255), (130, 513), (7, 2047), (6, 2049), (9, 4100), (5, 8192), (3, 8193), (2, 16390),
          (515, 8200), (2050, 130), (4100, 70), (3, 70000),
          (300, 257), (300, 1030), (300, 2100), (200, 1100), (300, 5001), (270, 8194), (260, 10300), (520, 16390)]


@pytest.mark.parametrize("split", ["rn", "bitmask"])
@pytest.mark.parametrize("rows,n", SHAPES)
def test_rows_and_columns_match_the_oracle_bit_for_bit(oz, rows, n, split):
    k = 5 if rows * n > 100000 else 9
    A, _ = inputs.phi_pair(rows, n, 1, 2.0, seed=301)
    A[0, : n // 2] = 0.0                       # (a vector whose largest element sits in its last batch)
    pad = n % 3                                # rows with and without the alignment for 16-byte loads
    Ap = torch.zeros((rows, n + pad), dtype=torch.float64, device="cuda")
    Ap[:, :n] = dev(A)
    beta, _ = oracle.params(n)
    want, we = oracle.split_rows(A, k, beta, form="int" if split == "rn" else "bitmask")
    S, e = oz.split_A(Ap[:, :n], k, split)
    assert np.array_equal(e.cpu().numpy(), we)
    assert np.array_equal(oz.export_slices(rows, n, k, S).cpu().numpy(), want)
    Bp = torch.zeros((n, rows + pad), dtype=torch.float64, device="cuda")
    Bp[:, :rows] = dev(A.T)
    S, e = oz.split_B(Bp[:, :rows], k, split)
    assert np.array_equal(e.cpu().numpy(), we)
    assert np.array_equal(oz.export_slices(rows, n, k, S).cpu().numpy(), want)
    few = np.ascontiguousarray(A[:2])          # the same vectors as rows and as columns of one call
    got = oz.dgemm_variant(Ap[:, :n], dev(few.T), k, split).cpu().numpy()
    assert np.array_equal(got, oracle.dgemm_variant(A, few.T, k, split))
    got = oz.dgemm_variant(dev(few), Bp[:, :rows], k, split).cpu().numpy()
    assert np.array_equal(got, oracle.dgemm_variant(few, A.T, k, split))


@pytest.mark.parametrize("transA,transB", [(True, True), (True, False), (False, True)])
def test_both_operands_by_columns_or_by_rows(oz, transA, transB):
    # operand pairs of one kind, with different numbers of vectors (the smaller choice of columns / rows a workgroup serves both)
    m, n, p, k = 2100, 600, 40, 6
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=302)
    a, b = (np.ascontiguousarray(A.T) if transA else A), (np.ascontiguousarray(B.T) if transB else B)
    C = torch.full((m, p), float("nan"), dtype=torch.float64, device="cuda")
    oz.gemm_ex(transA, transB, 1.0, dev(a), dev(b), 0.0, C, k)
    assert np.array_equal(C.cpu().numpy(), oracle.dgemm(A, B, k))


# (vectors, length, k): the forms that only large operands take - rows whose slices leave the caches (four, two a workgroup, 32
# and 64 elements a thread), columns by 16, 8 and 4 a workgroup, one more than fills the compute units
@pytest.mark.parametrize("rows,n,k", [(13000, 1300, 9), (8010, 2100, 9), (2110, 8100, 9), (1710, 10300, 12), (4353, 4700, 5),
                                      (2117, 6000, 4), (1030, 5000, 6), (4100, 200, 4), (20001, 3, 8)])
@pytest.mark.parametrize("split", ["rn", "bitmask"])
def test_large_operands_match_the_oracle_on_sampled_vectors(oz, rows, n, k, split):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(303)
    A = torch.rand((rows, n), dtype=torch.float64, device="cuda", generator=gen) - 0.5
    A *= torch.exp(torch.randn((rows, n), dtype=torch.float64, device="cuda", generator=gen))
    beta, _ = oracle.params(n)
    pick = np.unique(np.concatenate([[0, 1, rows - 1, rows - 2], inputs.sample_indices(rows, 12, seed=7)]))
    at = torch.from_numpy(pick).cuda()
    want, we = oracle.split_rows(A[at].cpu().numpy(), k, beta, form="int" if split == "rn" else "bitmask")
    for S, e in (oz.split_A(A, k, split), oz.split_B(A.T.contiguous(), k, split)):
        got = oz.export_slices(rows, n, k, S)
        assert np.array_equal(e[at].cpu().numpy(), we)
        assert np.array_equal(got[:, at].cpu().numpy(), want)
        del got


@pytest.mark.parametrize("columns,n,k,cut", [(60, 16384, 8, False), (60, 65536, 1, True), (500, 65536, 8, True),
                                             (1000, 65536, 8, True), (700, 200000, 1, True), (4000, 16384, 8, False),
                                             (1000, 4096, 8, False), (2100, 80000, 2, True), (20000, 10, 1, False),
                                             (60, 24000, 1, False), (200, 20000, 8, False)])
def test_long_columns_are_cut_where_that_is_faster(oz, columns, n, k, cut):
    # measured 1.2 to 2.7 times faster than taking them whole (and the other way round).  Which way a call takes shows in the
    # padding of the stack: only the cut way writes it
    B = torch.ones((n, columns), dtype=torch.float64, device="cuda")
    S = torch.full((oz.slices_bytes(columns, n, k),), 0x5A, dtype=torch.int8, device="cuda")
    e = torch.empty(columns, dtype=torch.int32, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    assert oz._lib.ozimmu_split_B(n, columns, B.data_ptr(), columns, k, S.data_ptr(), e.data_ptr(), st) == 0
    row_block = -(-n // 256) * 256 * 256                      # bytes of 256 packed rows; row r of a tile at 64 r
    at = (-(-columns // 256) - 1) * row_block + 255 * 64
    assert bool((S[at:at + 64] != 0x5A).any()) == cut
