"""The nearest-neighbour search of the overlap ratio at the edges of its
leaves (16 points), query groups (32), superblocks (1,024 points) and rounds of
64 superblocks, and where its pruning has least to go by: query groups that
straddle distant clusters, and points on a line.  Matches are integer decisions
on one FP32 rounding sequence: equality with brute force."""

import numpy as np
import pytest

from oracle import overlap as O
from tests.test_gpu_overlap import _gpu, _rigid

pytestmark = pytest.mark.gpu


def _points(rng, n, kind):
    if kind == "clusters":
        return rng.choice(rng.uniform(-50, 50, (7, 3)), n) + rng.normal(scale=0.01, size=(n, 3))
    if kind == "line":
        return rng.uniform(-2, 2, (n, 1)) * np.array([1.0, 0.5, 0.25])
    if kind == "grid":  # every distance many times: ties
        return rng.integers(0, 6, (n, 3)) * 0.25
    return rng.uniform(-2, 2, (n, 3))


@pytest.mark.parametrize("n_p,n_q,kind", [
    (1, 1, "box"), (15, 33, "box"), (16, 32, "grid"), (17, 31, "line"), (64, 65, "clusters"), (1023, 1025, "box"),
    (1024, 16, "grid"), (2049, 2047, "clusters"), (3000, 700, "line"), (2500, 2500, "grid"), (66000, 40, "box"),
    (35, 65537, "clusters"),
])
def test_matches_equal_brute_force(gpu, n_p, n_q, kind):
    rng = np.random.default_rng(n_p + n_q)
    P, Q = (_points(rng, n, kind).astype(np.float32) for n in (n_p, n_q))
    T = _rigid(rng, 3.0, 0.1) if kind != "grid" else np.eye(4)
    got, ref = _gpu(P, Q, T, 0.1), O.overlap_ratio(P, Q, T, 0.1)
    assert got[1:3] == ref[1:3]
    np.testing.assert_array_equal(got[3], ref[3])
    np.testing.assert_array_equal(got[4], ref[4])
