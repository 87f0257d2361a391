"""k_small: the whole call in one launch (small outputs of at most 256 inner positions), against the oracle in full."""
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


def view(x, pad, shift=0):
    """x on the GPU with `pad` more columns, beginning `shift` elements into its memory"""
    rows, cols = x.shape
    flat = torch.full((shift + rows * (cols + pad),), float("nan"), dtype=torch.float64, device="cuda")
    v = flat[shift:].view(rows, cols + pad)[:, :cols]
    v.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return v


def operands(m, n, p, seed):
    A, B = inputs.phi_pair(m, n, p, 2.0, seed=seed)
    if m > 2 and p > 2:
        A[1], B[:, 1] = 0.0, 0.0
        A[2, 0], B[n // 2, 2] = 2.0 ** 9, -2.0 ** -7      # exact powers of two, far from the rest
    return A, B


# edges of the 16 x 16 tiles, of the inner steps of 64 and of the 4 positions of a thread; every k
@pytest.mark.parametrize("m,n,p,k", [(1, 1, 1, 3), (16, 64, 16, 8), (17, 65, 15, 8), (33, 256, 47, 16), (128, 129, 100, 7),
                                     (100, 255, 100, 3), (31, 200, 250, 9), (2, 3, 5, 4), (3, 254, 3, 5), (48, 63, 16, 6),
                                     (20, 128, 20, 10), (40, 190, 18, 11), (15, 193, 33, 12), (64, 32, 64, 13), (65, 96, 63, 14),
                                     (16, 256, 16, 15), (256, 256, 256, 8), (257, 256, 255, 8), (16, 257, 16, 8)])
@pytest.mark.parametrize("pad,shift", [(0, 0), (3, 1)])
def test_dgemm(oz, m, n, p, k, pad, shift):
    assert (oz.WAYS[oz.choose(m, n, p, k).way] == "small") == (n <= 256)
    A, B = operands(m, n, p, 501)
    want = oracle.dgemm(A, B, k)
    D = view(np.zeros((m, p)), 2)
    dA, dB = view(A, pad, shift), view(B, pad, shift)
    oz.dgemm(dA, dB, k, D=D)
    assert np.array_equal(D.cpu().numpy(), want)
    assert bool(torch.isnan(D.as_strided((m, 2), (p + 2, 1), D.storage_offset() + p)).all()) or m * p == 0
    oz.dgemm_static(dA, dB, k, D.zero_())
    assert np.array_equal(D.cpu().numpy(), want)
    assert np.array_equal(oz.dgemm_variant(dA, dB, k, "rn", "wide").cpu().numpy(), want)


@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (-1.0, 0.5), (2.0, 0.0)])
def test_gemm_ex(oz, ta, tb, alpha, beta):
    m, n, p, k = 35, 131, 50, 9
    A, B = operands(m, n, p, 502)
    C0 = np.random.default_rng(1).standard_normal((m, p))
    C = view(C0, 3)
    if beta == 0.0:
        C.fill_(float("nan"))     # not read
    oz.gemm_ex(ta, tb, alpha, view(A.T if ta else A, 1), view(B.T if tb else B, 2), beta, C, k)
    d = oracle.dgemm(A, B, k)
    assert np.array_equal(C.cpu().numpy(), alpha * d + beta * C0 if beta else alpha * d)


@pytest.mark.parametrize("which", ["A", "B", "inside"])
def test_output_over_an_operand(oz, which):
    # the operands are split before anything is written, as in a call of two launches
    n, k = 96, 8
    A, B = operands(n, n, n, 503)
    want = oracle.dgemm(A, B, k)
    dA, dB = view(A, 1), view(B, 0)
    D = dA if which == "A" else dB
    if which == "inside":
        flat = torch.empty(2 * n * n, dtype=torch.float64, device="cuda")
        dA = flat[n * n // 2:n * n // 2 + n * n].view(n, n)
        dA.copy_(torch.from_numpy(A))
        D = flat[:n * n].view(n, n)
    oz.dgemm(dA, dB, k, D=D)
    assert np.array_equal(D.cpu().numpy(), want)


def test_graph(oz):
    m, n, p, k = 100, 200, 60, 8
    A, B = operands(m, n, p, 504)
    dA, dB, D = view(A, 0), view(B, 0), view(np.zeros((m, p)), 0)
    ws = oz.alloc_workspace(m, n, p, k)
    oz.init()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        oz.dgemm(dA, dB, k, D=D, workspace=ws)
    for rep in range(3):
        dA.mul_(0.5)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(D.cpu().numpy(), oracle.dgemm(A * 0.5 ** (rep + 1), B, k))
