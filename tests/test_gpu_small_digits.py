"""Digits of the one-launch way (k_small), taken from the element itself seven slices at a time: ties at every slice, digits of -64 and 64, the
places where the elements become their remainders (slices 8 and 15)."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def tie_matrix(rows, cols, seed):
    """a few bits at places that end at a digit's half, or at a full digit, of both signs, under a largest element of 1 or just below"""
    rng = np.random.default_rng(seed)
    at = rng.integers(0, 16, size=(rows, cols, 3))
    place = -7.0 * at - rng.choice([0, 1, 6, 7], size=at.shape)
    X = (rng.choice([-1.0, 1.0], size=at.shape) * 2.0 ** place).sum(axis=2)
    X[rng.random((rows, cols)) < 0.1] = 0.0
    X = np.clip(X, -1.0, 1.0)
    X[:, 0] = rng.choice([1.0, -1.0, 1.0 - 2.0 ** -53, 127.0 / 128.0, 0.5 + 2.0 ** -30], size=rows)
    return np.ldexp(X, rng.integers(-40, 41, size=(rows, 1)).astype(np.int32))


@pytest.mark.parametrize("k", range(3, 17))
@pytest.mark.parametrize("n", [1, 64, 250])
def test_ties_and_extreme_digits(k, n):
    from paper_2409_13313_amd import ozimmu as oz
    m, p = 33, 47
    assert oz.WAYS[oz.choose(m, n, p, k).way] == "small"
    A, B = tie_matrix(m, n, 701 + k), np.ascontiguousarray(tie_matrix(p, n, 801 + k).T)
    for x, y in ((A, B), (1.0 / 3.0 * A, 1.0 / 7.0 * B)):
        got = oz.dgemm(torch.from_numpy(np.ascontiguousarray(x)).cuda(), torch.from_numpy(np.ascontiguousarray(y)).cuda(), k)
        assert np.array_equal(got.cpu().numpy(), oracle.dgemm(x, y, k))
