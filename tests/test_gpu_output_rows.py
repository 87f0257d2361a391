"""Outputs whose rows begin anywhere: kept in L2 for short inner dimensions, streamed for long ones, same bits, nothing beside them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_2409_13313_amd import inputs, ozimmu  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,p,k,pad,shift", [
    (65, 40, 131, 3, 0, 0),     # odd pitch, one step
    (65, 40, 131, 3, 5, 0),     # pitch a multiple of 8, base aligned: streamed
    (65, 40, 131, 3, 5, 3),     # the same, base in the middle of a line
    (200, 1216, 67, 8, 2, 1),   # 36 pairs x 19 steps = 684: kept
    (200, 1217, 67, 8, 2, 1),   # x 20 steps = 720: streamed
    (300, 129, 259, 14, 1, 0),  # 105 pairs
    (90000, 160, 77, 4, 0, 0),  # output, operands and slices beyond the memory-side cache: streamed
])
def test_rows_of_any_alignment(m, n, p, k, pad, shift):
    # (every tile forced: by its own choice the library takes the short ones in one launch with the split, k_small)
    A, B = inputs.phi_pair(m, n, p, 0.5, seed=m + n)
    dA, dB, want = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), oracle.dgemm(A, B, k)
    pitch = p + pad
    for tile in range(-1, ozimmu.RESIDENT_TILES):
        if tile >= 0 and ozimmu.resident_tile(n, k, "grouped", tile) is None:
            continue
        flat = torch.full((shift + m * pitch + 64,), 7.0, dtype=torch.float64, device="cuda")
        D = flat[shift:shift + m * pitch].view(m, pitch)[:, :p]
        if tile < 0:
            ozimmu.dgemm(dA, dB, k, D=D)
        else:
            ozimmu.dgemm_resident(dA, dB, k, tile, D=D)
        host = flat.cpu().numpy()
        rows = host[shift:shift + m * pitch].reshape(m, pitch)
        assert np.array_equal(rows[:, :p], want), tile
        assert (rows[:, p:] == 7.0).all() and (host[:shift] == 7.0).all() and (host[shift + m * pitch:] == 7.0).all(), tile
