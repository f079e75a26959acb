"""Workspace sizes (host only): room for a size is room for every smaller one."""

import numpy as np

from paper_2408_10154_amd import lib as L
from tests.test_abi import _host_pair

# around the sizes where a radix sort's blocks, and the pair sort's spans, become longer
EDGES = sorted({max(0, (k << 16) + d) for k in (0, 1, 4, 8, 12, 16, 24, 32, 64, 128, 256, 512, 2048)
                for d in (-1, 0, 1, 1025)})


def _non_decreasing(sizes):
    return all(a <= b for a, b in zip(sizes, sizes[1:]))


def test_registration_workspace_grows_with_the_capacity():
    prm = L.ls_reg_params(10, 0.01, 0.01, 0.9, 0.999, 1e-8)
    # the lists by chunks, by pairs, and by pairs up to 33 M, 10 M and 2 M instances
    for w, h, views in ((64, 48, 3), (6000, 6000, 100), (6000, 6000, 7), (2000, 2000, 60), (1200, 680, 16)):
        pair, keep = _host_pair(vp=views, vq=views, w=w, h=h)
        assert _non_decreasing([L.ls_register_workspace_size(pair, prm, c) for c in EDGES]), (w, h)


def test_overlap_workspace_grows_with_the_points():
    """In each set alone, in both together, and against the static scratch."""
    size = L.ls_overlap_workspace_size
    for other in (0, 1, 1 << 16, 1 << 18, (1 << 18) + 1, 1 << 19):
        assert _non_decreasing([size(n, other) for n in EDGES]), other
        assert _non_decreasing([size(other, n) for n in EDGES]), other
    assert _non_decreasing([size(n, n) for n in EDGES])
    mx = L.LS_OVERLAP_NOALLOC_MAX_POINTS
    assert max(size(a, b) for a in EDGES for b in EDGES if max(a, b) <= mx) <= L.LS_OVERLAP_NOALLOC_BYTES


def test_fewer_views_fit_in_the_workspace_of_all():
    """A registration that keeps its best views runs them in the workspace of the
    full set, whatever form their lists take."""
    rng = np.random.default_rng(0)
    lg = lambda a, b: int(round(a * (b / a) ** rng.random()))  # noqa: E731
    prm = L.ls_reg_params(10, 0.01, 0.01, 0.9, 0.999, 1e-8)
    for _ in range(2000):
        v, n, w, cap = (lg(1, 60), lg(1, 60)), (lg(100, 500_000), lg(100, 500_000)), lg(16, 4000), lg(1000, 50_000_000)
        k = int(rng.choice([1, 2, max(1, min(v) - 1), max(1, max(v) - 1)]))
        size = []
        for a, b in (v, (min(v[0], k), min(v[1], k))):
            pair, keep = _host_pair(vp=a, vq=b, n_p=n[0], n_q=n[1], w=w, h=max(16, int(0.7 * w)))
            size.append(L.ls_register_workspace_size(pair, prm, cap))
        assert size[1] <= size[0], (v, n, w, cap, k)
