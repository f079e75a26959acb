"""Workspace sizes (host only): room for a size is room for every smaller one."""

from paper_2408_10154_amd import lib as L
from tests.test_abi import _host_pair

# around the sizes where a radix sort's blocks, and the pair sort's spans, become longer
EDGES = sorted({max(0, k + d) for k in (0, 1 << 16, 1 << 18, 1 << 19, 3 << 18, 1 << 20, 3 << 19, 1 << 21, 1 << 22, 1 << 23)
                for d in (-1, 0, 1, 1025)})


def _non_decreasing(sizes):
    return all(a <= b for a, b in zip(sizes, sizes[1:]))


def test_registration_workspace_grows_with_the_capacity():
    prm = L.ls_reg_params(10, 0.01, 0.01, 0.9, 0.999, 1e-8)
    for w, h in ((64, 48), (6000, 6000)):  # the lists by chunks and by pairs
        pair, keep = _host_pair(w=w, h=h)
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
