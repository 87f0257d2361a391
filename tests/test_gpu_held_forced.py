"""GPU parity of k_held, forced where its offsets and orders are others than for short inner dimensions of 7-bit digits, and by the library's own choice."""
import numpy as np
import pytest

import oracle
from paper_2409_13313_amd import inputs
from test_gpu_held import CHUNKS, oz  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the slice counts that have a k_held at each of them
INSTANCES = {"whole groups": (6, 7, 8, 9, 10, 11, 13, 14), "8": (9, 10, 11, 12), "4": (5, 6, 7, 8, 9), "2": (5, 6, 7)}


def test_there_is_no_other_instance(oz):
    for c in CHUNKS:
        for k in range(1, oz.MAX_SLICES + 1):
            here = c == "whole groups" or k > int(c)        # (up to chunks of whole groups it is the instance of those)
            assert all((oz.resident_tile(n, k, "grouped", oz.HELD_TILE) is not None) == (k in INSTANCES[c]) for n in CHUNKS[c]) or not here, (k, c)


# chunks of 2 again where digits have 6 bits, bit-mask digits, wide chunks
@pytest.mark.parametrize("n,k,split,accumulate", [(131073, 7, "rn", "grouped"), (200001, 5, "bitmask", "grouped"), (600, 9, "bitmask", "grouped"),
                                                  (262144, 6, "rn", "grouped"), (40001, 9, "rn", "wide"), (300001, 7, "rn", "wide")])
def test_other_digits_and_chunks(oz, n, k, split, accumulate):
    m, p = 97, 131
    assert oz.resident_tile(n, k, accumulate, oz.HELD_TILE) is not None
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=504)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    ref = oz.dgemm_variant(dA, dB, k, split, accumulate, schedule="one_launch")
    rows, cols = [0, 96], [0, 130]
    want = oracle.dgemm_variant(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), k, split, accumulate)
    assert np.array_equal(ref.cpu().numpy()[np.ix_(rows, cols)], want)
    assert torch.equal(oz.dgemm_resident(dA, dB, k, oz.HELD_TILE, split, accumulate), ref)


def test_the_longest_inner_dimension(oz):
    # row blocks of 2 GiB, and tiles of 96 columns with columns in two of them: offsets of up to 4 GiB
    m, n, p, k = 3, 64 * (2**17 - 1), 300, 7
    assert oz.resident_tile(n, k, "wide", oz.HELD_TILE) == (96, 96)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(505)
    dA = torch.rand((m, n), dtype=torch.float64, device="cuda", generator=gen) - 0.5
    dB = torch.rand((n, p), dtype=torch.float64, device="cuda", generator=gen) - 0.5
    ws = oz.alloc_workspace(m, n, p, k)
    got = oz.dgemm_resident(dA, dB, k, oz.HELD_TILE, accumulate="wide", workspace=ws)
    ref = oz.dgemm_variant(dA, dB, k, accumulate="wide", schedule="one_launch", workspace=ws)
    assert torch.equal(got, ref)
    at = [0, 191, 192, 255, 256, 287, 299]
    want = (dA @ dB[:, at]).cpu().numpy()
    # 7 slices of at least 4 bits leave 2^-28 of the largest elements of a row and a column, per product
    assert np.abs(got[:, at].cpu().numpy() - want).max() <= n * 2.0**-26


# (2000 x 600 x 2000, k = 6, is left to 64 x 64 tiles, two to a compute unit: 51.9 us, with k_held 53.3; 1537 x 515 x 1283, k = 9, to 32 x 32, 54.3 and 56.4)
@pytest.mark.parametrize("m,n,p,k,alpha,beta", [(1537, 1603, 1283, 9, -1.0, 0.5), (2000, 1500, 2000, 6, 1.0, 0.0), (1300, 700, 1301, 11, 0.75, -0.25)])
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
