"""GPU parity for the GEMM-routine form C <- alpha op(A) op(B) + beta C against the oracle."""
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


@pytest.mark.parametrize("transA", [False, True])
@pytest.mark.parametrize("transB", [False, True])
@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (1.0 / 3.0, -0.7), (0.0, 2.0), (-2.0, 1.0)])
def test_gemm_ex_matches_oracle_bit_for_bit(oz, transA, transB, alpha, beta):
    m, n, p, k = 300, 520, 270, 7
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=51)
    C0 = np.random.Generator(np.random.PCG64(52)).standard_normal((m, p))
    if beta == 0.0:
        C0[0, 0] = np.nan          # must not propagate: the old C is not read
    As = np.ascontiguousarray(A.T) if transA else A
    Bs = np.ascontiguousarray(B.T) if transB else B
    want = oracle.gemm_ex(transA, transB, alpha, As, Bs, beta, C0, k)
    # leading dimensions larger than the extents, and a poisoned frame around C
    Ab = torch.zeros((As.shape[0], As.shape[1] + 3), dtype=torch.float64, device="cuda")
    Bb = torch.zeros((Bs.shape[0], Bs.shape[1] + 5), dtype=torch.float64, device="cuda")
    Cb = torch.full((m + 1, p + 2), -3.0, dtype=torch.float64, device="cuda")
    Ab[:, :As.shape[1]] = dev(As)
    Bb[:, :Bs.shape[1]] = dev(Bs)
    Cb[:m, :p] = dev(C0)
    oz.gemm_ex(transA, transB, alpha, Ab[:, :As.shape[1]], Bb[:, :Bs.shape[1]], beta, Cb[:m, :p], k)
    got = Cb.cpu().numpy()
    assert np.isfinite(got[:m, :p]).all()
    assert np.abs(got[:m, :p] - want).max() <= 2 * np.spacing(np.abs(want)).max()
    assert np.array_equal(got[:m, :p], want)
    assert (got[m:, :] == -3.0).all() and (got[:, p:] == -3.0).all()


def test_gemm_ex_without_old_c_needs_no_extra_buffer(oz):
    # beta == 0: the sum is formed in C itself and fl(alpha d) is applied by the last chunk's epilogue, so the
    # least workspace of ozimmu_dgemm is enough; beta != 0 needs the m x p buffer on top
    m, n, p, k = 520, 300, 270, 5
    A, B = inputs.phi_pair(m, n, p, 0.5, seed=61)
    want = oracle.gemm_ex(False, False, -0.375, A, B, 0.0, np.zeros((m, p)), k)
    small = torch.empty(oz.workspace_bytes_min(m, n, p, k), dtype=torch.uint8, device="cuda")
    C = torch.full((m, p), float("nan"), dtype=torch.float64, device="cuda")
    oz.gemm_ex(False, False, -0.375, dev(A), dev(B), 0.0, C, k, workspace=small)
    assert np.array_equal(C.cpu().numpy(), want)
    with pytest.raises(oz.OzimmuError):
        oz.gemm_ex(False, False, -0.375, dev(A), dev(B), 0.5, C, k, workspace=small)


def test_gemm_ex_single_slice_first_chunk_is_also_the_last(oz):
    # k = 1: one chunk, which is first (D not read) and last (step (v) applied) at once
    m, n, p = 300, 260, 280
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=62)
    C0 = np.random.Generator(np.random.PCG64(63)).standard_normal((m, p))
    for alpha, beta in ((2.5, 0.0), (-0.3, 1.25)):
        want = oracle.gemm_ex(False, False, alpha, A, B, beta, C0, 1)
        C = dev(C0)
        oz.gemm_ex(False, False, alpha, dev(A), dev(B), beta, C, 1)
        assert np.array_equal(C.cpu().numpy(), want)


def test_gemm_ex_empty_inner_dimension_scales_c(oz):
    C0 = np.random.Generator(np.random.PCG64(53)).standard_normal((5, 7))
    C = dev(C0)
    oz.gemm_ex(False, False, 1.5, torch.empty((5, 0), dtype=torch.float64, device="cuda"),
               torch.empty((0, 7), dtype=torch.float64, device="cuda"), 0.25, C, 8)
    assert np.array_equal(C.cpu().numpy(), 0.25 * C0)
    oz.gemm_ex(False, False, 1.5, torch.empty((5, 0), dtype=torch.float64, device="cuda"),
               torch.empty((0, 7), dtype=torch.float64, device="cuda"), 0.0, C, 8)
    assert (C == 0).all()


def test_gemm_ex_large_output_with_a_cut_tail_round(oz):
    # 272 tiles of 256 x 256 (for the persistent launch one full round and 16 tiles more; k_resident takes it); transposed
    # operands and step (v) on top.  Rows / columns from every band of 256 (every tile, so also the cut tail
    # round) are recomputed by the oracle.
    m, n, p, k = 4352, 520, 4096, 4
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=95)
    C0 = inputs.phi_pair(m, 1, p, 0.5, seed=96)[0] @ np.ones((1, p))
    alpha, beta = -1.75, 0.3
    C = torch.from_numpy(C0).cuda()
    oz.gemm_ex(True, True, alpha, torch.from_numpy(np.ascontiguousarray(A.T)).cuda(),
               torch.from_numpy(np.ascontiguousarray(B.T)).cuda(), beta, C, k)
    assert torch.isfinite(C).all()
    I = inputs.band_indices(m, 256, seed=97)
    J = inputs.band_indices(p, 256, seed=98)
    want = oracle.gemm_ex(False, False, alpha, np.ascontiguousarray(A[I]), np.ascontiguousarray(B[:, J]), beta,
                          np.ascontiguousarray(C0[np.ix_(I, J)]), k)
    got = C[torch.from_numpy(I).cuda()][:, torch.from_numpy(J).cuda()].cpu().numpy()
    assert np.array_equal(got, want)
    # every entry: the library's own product (one launch forced) followed by the three rounded operations
    # of step (v) as torch evaluates them in FP64 (a consistency check on top of the oracle comparison)
    D = oz.dgemm_variant(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), k, "rn", "grouped",
                         schedule="one_launch")
    assert torch.equal(C, alpha * D + beta * torch.from_numpy(C0).cuda())
