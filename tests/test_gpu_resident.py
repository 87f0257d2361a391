"""GPU parity of the kernel that keeps all chunk sums of a tile in registers (ozimmu_resident.hip): every one of its instances
(slice count x chunk length x tile) forced, and the library's own choice at the sizes where it can go wrong: the edges of its
tiles (32 to 128 rows and columns), inner dimensions around the step of 64, chunks shorter than the groups (long inner
dimensions, per-pair accumulation), step (v), strided outputs, and exponents at which the scaled summation has to give way to
the term-by-term one.  Each D is compared bit for bit with the oracle and / or the persistent launch."""
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


@pytest.mark.parametrize("k", range(3, 17))
@pytest.mark.parametrize("m,n,p", [(1, 1, 1), (31, 63, 33), (65, 64, 63), (129, 65, 97), (64, 129, 257), (257, 300, 128)])
def test_tile_and_step_edges_match_the_oracle_bit_for_bit(oz, m, n, p, k):
    # (forced: by its own choice the library takes most of these in one launch with the split, k_small)
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=201)
    dA, dB, want = dev(A), dev(B), oracle.dgemm(A, B, k)
    for tile in range(oz.RESIDENT_TILES):
        if oz.resident_tile(n, k, "grouped", tile) is None:
            continue
        D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
        oz.dgemm_resident(dA, dB, k, tile, D=D[:, :p])
        got = D.cpu().numpy()
        assert np.array_equal(got[:, :p], want) and np.isnan(got[:, p]).all(), tile


# Chunk lengths r by the inner dimensions and the accumulate mode that give them; inner dimensions of one step, an odd and an
# even number of steps
CHUNKS = {"whole groups": ("grouped", (60, 130, 257)), "8": ("grouped", (8200, 8260)), "4": ("grouped", (16400, 16500)),
          "2": ("grouped", (32800, 32900)), "1": ("per_pair", (64, 129, 250))}


@pytest.mark.parametrize("k,chunk", [(k, c) for c in CHUNKS for k in range(3, 17) if not (c in "842" and k <= int(c))])
def test_every_tile_of_every_instance(oz, k, chunk):
    # the compile-time order of fetches, copies and counted waits is another one for every instance
    accumulate, inner = CHUNKS[chunk]
    m, p, tiles = 293, 261, 0
    for n in inner:
        A, B = inputs.phi_pair(m, n, p, 1.0, seed=207)
        dA, dB = dev(A), dev(B)
        ref = oz.dgemm_variant(dA, dB, k, "rn", accumulate, schedule="one_launch")
        rows, cols = np.array([0, 31, 130, m - 1]), np.array([0, 33, 128, p - 1])
        want = oracle.dgemm_variant(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), k, "rn", accumulate)
        assert np.array_equal(ref.cpu().numpy()[np.ix_(rows, cols)], want)
        for tile in range(oz.RESIDENT_TILES):
            if oz.resident_tile(n, k, accumulate, tile) is None:
                continue
            tiles += 1
            D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
            oz.dgemm_resident(dA, dB, k, tile, "rn", accumulate, D=D[:, :p])
            assert torch.equal(D[:, :p], ref) and bool(torch.isnan(D[:, p]).all()), (n, tile)
    assert tiles > 0 or (accumulate == "per_pair" and k > 10) or (chunk == "2" and k > 15)   # more than 64 chunk sums


def test_no_tile_where_the_kernel_has_none(oz):
    A = torch.zeros((40, 40), dtype=torch.float64, device="cuda")
    for k, tile, split, accumulate in ((2, 0, "rn", "grouped"), (17, 0, "rn", "grouped"), (8, 6, "rn", "grouped"),
                                       (8, -1, "rn", "grouped"), (11, 0, "rn", "per_pair"), (8, 0, "per_slice", "per_pair"),
                                       (8, 0, "bitmask", "wide")):
        with pytest.raises(oz.OzimmuError) as err:
            oz.dgemm_resident(A, A, k, tile, split, accumulate, workspace=oz.alloc_workspace(40, 40, 40, 20))
        assert err.value.status == -3


@pytest.mark.parametrize("m,n,p,k,split,accumulate", [
    (2040, 1990, 2049, 3, "rn", "grouped"), (2048, 2048, 2048, 4, "rn", "grouped"),
    (1990, 2047, 2000, 5, "rn", "grouped"), (2000, 1999, 2047, 6, "bitmask", "grouped"),
    (1000, 1999, 2047, 7, "rn", "grouped"), (1024, 2050, 2048, 8, "rn", "grouped"),
    (1030, 8200, 1000, 9, "rn", "grouped"), (1030, 8200, 1000, 12, "rn", "grouped"),
    (2050, 8200, 1990, 14, "rn", "grouped"),
    (1500, 16400, 1500, 8, "rn", "grouped"), (1500, 16400, 1500, 5, "bitmask", "grouped"),
    (1030, 300, 1000, 7, "bitmask", "per_pair"), (1030, 300, 1000, 9, "bitmask", "per_pair"),
    (1030, 300, 1000, 3, "rn", "per_pair"), (1030, 300, 1000, 5, "rn", "per_pair"), (1030, 300, 1000, 6, "rn", "per_pair"),
    (1030, 300, 1000, 10, "rn", "per_pair"), (1030, 300, 1000, 11, "rn", "wide")])
def test_larger_outputs_match_the_persistent_launch_and_sampled_oracle_entries(oz, m, n, p, k, split, accumulate):
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=202)
    dA, dB = dev(A), dev(B)
    ref = oz.dgemm_variant(dA, dB, k, split, accumulate, schedule="one_launch")
    got = oz.dgemm_variant(dA, dB, k, split, accumulate)
    assert torch.equal(got, ref)
    I, J = inputs.sample_indices(m, 24, seed=3), inputs.sample_indices(p, 24, seed=4)
    want = oracle.dgemm_variant(np.ascontiguousarray(A[I]), np.ascontiguousarray(B[:, J]), k, split, accumulate)
    assert np.array_equal(got[torch.from_numpy(I).cuda()][:, torch.from_numpy(J).cuda()].cpu().numpy(), want)


@pytest.mark.parametrize("k", [4, 8, 9, 13])
@pytest.mark.parametrize("alpha,beta", [(-1.5, 0.0), (0.75, -0.25)])
def test_step_v_on_ragged_tiles(oz, k, alpha, beta):
    m, n, p = 333, 290, 277          # (up to 256 inner positions k_small takes it)
    choice = oz.choose(m, n, p, k)
    assert oz.WAYS[choice.way] == "resident" and choice.parts == 1
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=203)
    C0 = np.random.Generator(np.random.PCG64(204)).standard_normal((m, p))
    C = torch.full((m, p + 3), -7.0, dtype=torch.float64, device="cuda")
    C[:, :p] = dev(C0)
    oz.gemm_ex(False, False, alpha, dev(A), dev(B), beta, C[:, :p], k)
    got = C.cpu().numpy()
    assert np.array_equal(got[:, :p], oracle.gemm_ex(False, False, alpha, A, B, beta, C0, k)) and (got[:, p:] == -7.0).all()


@pytest.mark.parametrize("shift", [-520, -480, 0, 480, 497])
def test_scales_at_the_ends_of_the_exponent_range(oz, shift):
    # rows and columns scaled by powers of two (the products by 2^(2 shift - 20) to 2^(2 shift + 20), at most 2^1014, and
    # the sums stay below 2^1024): some tiles hold terms (or results) that are
    # subnormal or close to overflow and are summed term by term, the others take the scaled sum; same bits as the
    # persistent launch, which always sums term by term
    # (forced, every tile, k_extended's among them: by its own choice the library takes a call of this size in one launch with the
    # split, k_small, which sums term by term too)
    m, n, p, k = 200, 130, 300, 9
    A, B = inputs.phi_pair(m, n, p, 0.5, seed=205)
    rng = np.random.Generator(np.random.PCG64(206))
    A = np.ldexp(A, (shift + rng.integers(-10, 11, size=(m, 1))).astype(np.int32))
    B = np.ldexp(B, (shift + rng.integers(-10, 11, size=(1, p))).astype(np.int32))
    dA, dB = dev(A), dev(B)
    ref = oz.dgemm_variant(dA, dB, k, schedule="one_launch")
    assert bool(torch.isfinite(ref).all())
    tiles = [t for t in range(oz.RESIDENT_TILES) if oz.resident_tile(n, k, "grouped", t) is not None]
    assert oz.RESIDENT_TILES - 1 in tiles and len(tiles) >= 5
    for tile in tiles:
        assert torch.equal(oz.dgemm_resident(dA, dB, k, tile), ref), tile
    assert torch.equal(oz.dgemm(dA, dB, k), ref)
