"""GPU parity of k_extended by the library's own choice: sizes at which it is chosen, off its tiles' edges by one, against the
persistent launch (in full) and the oracle (sampled rows and columns).  Forced, every instance of it runs in test_gpu_resident
(the last of the resident tiles)."""
import numpy as np
import pytest

import oracle
from paper_2409_13313_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,p,k,split,accumulate", [
    (1023, 130, 1025, 11, "bitmask", "per_pair"), (33, 250, 31, 12, "rn", "per_pair"), (1, 64, 1, 13, "bitmask", "per_pair"),
    (2047, 257, 2049, 9, "bitmask", "per_pair"), (2047, 3000, 4088, 5, "rn", "grouped"), (4090, 500, 4088, 9, "rn", "grouped"),
    (4090, 500, 4088, 10, "rn", "grouped"), (4097, 4100, 4088, 6, "rn", "grouped"), (700, 33000, 2050, 10, "rn", "grouped")])
def test_library_choice(m, n, p, k, split, accumulate):
    from paper_2409_13313_amd import ozimmu as oz
    choice = oz.choose(m, n, p, k, split, accumulate)
    assert oz.WAYS[choice.way] == "resident" and choice.tile == oz.RESIDENT_TILES - 1 and choice.parts == 1
    A, B = inputs.phi_pair(m, n, p, 1.0, seed=301)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    ref = oz.dgemm_variant(dA, dB, k, split, accumulate, schedule="one_launch")
    D = torch.full((m, p + 1), float("nan"), dtype=torch.float64, device="cuda")
    oz.dgemm_variant(dA, dB, k, split, accumulate, D=D[:, :p])
    assert torch.equal(D[:, :p], ref) and bool(torch.isnan(D[:, p]).all())
    rows, cols = np.unique([0, m // 2, m - 1]), np.unique([0, p // 2, p - 1])
    want = oracle.dgemm_variant(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), k, split, accumulate)
    assert np.array_equal(ref.cpu().numpy()[np.ix_(rows, cols)], want)
