"""GPU parity of k_held, the tiles that hold slices of A while those of B pass by: every instance forced, and by the library's own choice."""
import numpy as np
import pytest

import oracle
from paper_2409_13313_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# chunk lengths r by the inner dimensions that give them: fewer steps than a place has copies on their way, an odd and an even number
CHUNKS = {"whole groups": (1, 64, 65, 129, 257, 600), "8": (8200, 8260), "4": (16400, 16500), "2": (32800,)}
SHAPES = [(293, 261), (1, 1), (96, 128), (129, 97)]


@pytest.fixture(scope="module")
def oz():
    from paper_2409_13313_amd import ozimmu
    return ozimmu


@pytest.mark.parametrize("k,chunk", [(k, c) for c in CHUNKS for k in range(5, 15) if not (c in "842" and k <= int(c))])
def test_every_instance(oz, k, chunk):
    # (the compile-time order of fetches, copies and counted waits is another one for every instance)
    for n in CHUNKS[chunk]:
        if oz.resident_tile(n, k, "grouped", oz.HELD_TILE) is None:
            continue
        for m, p in SHAPES:
            A, B = inputs.phi_pair(m, n, p, 1.0, seed=501)
            dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
            ref = oz.dgemm_variant(dA, dB, k, schedule="one_launch")
            rows, cols = np.unique([0, m // 2, m - 1]), np.unique([0, p // 2, p - 1])
            want = oracle.dgemm(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), k)
            assert np.array_equal(ref.cpu().numpy()[np.ix_(rows, cols)], want)
            D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
            oz.dgemm_resident(dA, dB, k, oz.HELD_TILE, D=D[:, :p])
            assert torch.equal(D[:, :p], ref) and bool(torch.isnan(D[:, p]).all()), (n, m, p)


@pytest.mark.parametrize("m,n,p,k,alpha,beta", [(1537, 515, 1283, 9, -1.0, 0.5), (2000, 600, 2000, 6, 1.0, 0.0), (1300, 700, 1301, 11, 0.75, -0.25)])
def test_library_choice_with_step_v(oz, m, n, p, k, alpha, beta):
    assert oz.choose(m, n, p, k).tile == oz.HELD_TILE
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=502)
    C0 = np.random.default_rng(503).standard_normal((m, p))
    C = torch.full((m, p + 3), -7.0, dtype=torch.float64, device="cuda")
    C[:, :p] = torch.from_numpy(C0).cuda()
    dA, dB = torch.from_numpy(np.ascontiguousarray(A.T)).cuda(), torch.from_numpy(B).cuda()
    oz.gemm_ex(True, False, alpha, dA, dB, beta, C[:, :p], k)
    d = oz.dgemm_variant(dA.t().contiguous(), dB, k, schedule="one_launch").cpu().numpy()
    got = C.cpu().numpy()
    assert np.array_equal(got[:, :p], alpha * d + beta * C0 if beta else alpha * d) and (got[:, p:] == -7.0).all()
