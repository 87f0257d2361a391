"""Few tiles of a long inner dimension: k_resident with the inner dimension cut among workgroups and k_add_parts, against the
persistent launch in full and the oracle on corner elements."""
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


def operands(m, n, p, seed):
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=seed)
    return A, B, dev(A), dev(B)


def check_corners(D, A, B, k, split, accumulate):
    rows, cols = np.unique([0, A.shape[0] // 2, A.shape[0] - 1]), np.unique([0, B.shape[1] // 2, B.shape[1] - 1])
    want = oracle.dgemm_variant(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), k, split, accumulate)
    assert np.array_equal(D.cpu().numpy()[np.ix_(rows, cols)], want)


@pytest.mark.parametrize("m,n,p,k,split,accumulate", [
    (1, 4096, 1, 3, "rn", "grouped"), (33, 8129, 31, 8, "rn", "grouped"), (47, 11948, 48, 8, "rn", "grouped"),
    (64, 20001, 97, 4, "rn", "grouped"),          # chunks of four
    (130, 65537, 70, 10, "rn", "grouped"),        # r = 2: 30 sums
    (30, 140000, 33, 4, "rn", "grouped"),         # beta = 6
    (465, 1864, 40, 14, "rn", "grouped"), (40, 6000, 500, 5, "rn", "wide"), (75, 12000, 80, 10, "bitmask", "per_pair")])
def test_cut_inner_dimension(oz, m, n, p, k, split, accumulate):
    assert oz.choose(m, n, p, k, split, accumulate).parts > 1
    A, B, dA, dB = operands(m, n, p, 401)
    ref = oz.dgemm_variant(dA, dB, k, split, accumulate, schedule="one_launch")
    ws = oz.alloc_workspace(m, n, p, k)
    for fill in (0x5A, 0xC3):                     # what the blocks held before does not matter
        ws.fill_(fill)
        D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
        oz.dgemm_variant(dA, dB, k, split, accumulate, D=D[:, :p], workspace=ws)
        assert torch.equal(D[:, :p], ref) and bool(torch.isnan(D[:, p]).all())
    check_corners(ref, A, B, k, split, accumulate)
    least = torch.empty(oz.workspace_bytes_min(m, n, p, k), dtype=torch.uint8, device="cuda")   # as much cutting as fits
    assert torch.equal(oz.dgemm_variant(dA, dB, k, split, accumulate, workspace=least), ref)


# Chunk lengths by the inner dimensions and the accumulate mode that give them (see test_gpu_resident)
CHUNKS = {"whole groups": ("grouped", (257, 1090)), "8": ("grouped", (8200,)), "4": ("grouped", (16400,)),
          "2": ("grouped", (32800,)), "1": ("per_pair", (300, 1090))}


@pytest.mark.parametrize("k,chunk", [(k, c) for c in CHUNKS for k in range(3, 17) if not (c in "842" and k <= int(c))])
def test_every_instance(oz, k, chunk):
    # the compile-time order of fetches, copies and counted waits is another one for every instance; parts of two steps, of three and
    # of more, of equal and of different lengths, by fours and by sixteens in k_add_parts
    accumulate, inner = CHUNKS[chunk]
    m, p, cut = 77, 101, 0
    for n in inner:
        A, B, dA, dB = operands(m, n, p, 404)
        ref = oz.dgemm_variant(dA, dB, k, "rn", accumulate, schedule="one_launch")
        check_corners(ref, A, B, k, "rn", accumulate)
        ws = torch.empty(oz.workspace_bytes_min(m, n, p, k) + (256 << 20), dtype=torch.uint8, device="cuda")
        for tile in range(oz.RESIDENT_TILES - 1):
            size = oz.resident_tile(n, k, accumulate, tile)
            if size is None or size[0] * size[1] > 32 * 64:
                continue
            for parts in (2, 3, 5, 8, 9, 17, 64):
                if 2 * parts > (n + 63) // 64:
                    continue
                ws.fill_(0xC3)
                D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
                oz.dgemm_tile(dA, dB, k, tile, parts, "rn", accumulate, D=D[:, :p], workspace=ws)
                assert torch.equal(D[:, :p], ref) and bool(torch.isnan(D[:, p]).all()), (n, tile, parts)
                cut += 1
    assert cut > 0 or (accumulate == "per_pair" and k > 10) or (chunk == "2" and k > 15)   # more than 64 chunk sums


@pytest.mark.parametrize("shift", [-520, 497])
def test_scales_at_the_ends_of_the_exponent_range(oz, shift):
    m, n, p, k = 70, 2100, 45, 8
    A, B = inputs.phi_pair(m, n, p, 0.5, seed=405)
    rng = np.random.Generator(np.random.PCG64(406))
    A = np.ldexp(A, (shift + rng.integers(-10, 11, size=(m, 1))).astype(np.int32))
    B = np.ldexp(B, (shift - 2 + rng.integers(-10, 11, size=(1, p))).astype(np.int32))
    dA, dB = dev(A), dev(B)
    ref = oz.dgemm_variant(dA, dB, k, schedule="one_launch")
    assert bool(torch.isfinite(ref).all())
    for parts in (3, 11):
        assert torch.equal(oz.dgemm_tile(dA, dB, k, 5, parts), ref)


@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (-1.0, 0.5), (0.75, -0.25), (2.0, 0.0)])
def test_cut_with_step_v(oz, alpha, beta):
    m, n, p, k = 70, 5000, 45, 8
    assert oz.choose(m, n, p, k).parts > 1
    A, B, dA, dB = operands(m, n, p, 402)
    C0 = np.random.default_rng(5).standard_normal((m, p))
    C = torch.full((m, p + 3), float("nan"), dtype=torch.float64, device="cuda")
    C[:, :p] = dev(C0)
    oz.gemm_ex(True, True, alpha, dev(A.T), dev(B.T), beta, C[:, :p], k)
    d = oz.dgemm_variant(dA, dB, k, schedule="one_launch").cpu().numpy()
    want = alpha * d + beta * C0 if beta else alpha * d
    assert np.array_equal(C[:, :p].cpu().numpy(), want) and bool(torch.isnan(C[:, p:]).all())


def test_cut_in_the_static_workspace_and_a_graph(oz):
    m, n, p, k = 75, 2212, 80, 8
    assert oz.choose(m, n, p, k).parts > 1 and oz.choose(m, n, p, k, workspace_bytes=oz.STATIC_WORKSPACE_BYTES).parts > 1
    A, B, dA, dB = operands(m, n, p, 403)
    ref = oz.dgemm_variant(dA, dB, k, schedule="one_launch")
    D = torch.zeros((m, p), dtype=torch.float64, device="cuda")
    assert torch.equal(oz.dgemm_static(dA, dB, k, D), ref)
    ws = oz.alloc_workspace(m, n, p, k)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        oz.dgemm(dA, dB, k, D=D, workspace=ws)
    for _ in range(3):
        D.zero_()
        ws.fill_(0x33)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(D, ref)
