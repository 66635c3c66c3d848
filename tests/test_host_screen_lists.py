"""Trimer lists of mbe3_screen_lists from the sorted close pairs, against every
triple: sparse, dense and no close pairs, either orientation, mean metrics on both
sides of the threshold, and an output that is exactly or not quite large enough."""
import itertools

import numpy as np
import pytest


@pytest.mark.parametrize("n,keep,lo", [(3, 1.0, 0.1), (9, 0.5, 0.0), (20, 1.0, 0.0),
                                       (20, 0.15, 0.15), (12, 1.0, 0.3), (5, 1.0, 1.0)])
def test_screen_lists_all_triples(n, keep, lo):
    import paper_2603_16575_amd as pkg
    from paper_2603_16575_amd import _lib
    rng = np.random.default_rng(n)
    pr = np.array([p for p in itertools.combinations(range(n), 2) if rng.random() < keep])
    s = rng.uniform(lo, 0.4, len(pr)) if lo < 1.0 else np.full(len(pr), 1e-3)
    val = {tuple(p): v for p, v in zip(pr, s)}
    close = {p: v for p, v in val.items() if v >= pkg.S2B_CLOSE}
    tri = [(i, j, k) for i, j, k in itertools.combinations(range(n), 3)
           if (i, j) in close and (i, k) in close and (j, k) in close
           and (close[i, j] + close[i, k] + close[j, k]) / 3.0 >= pkg.S3B_KEEP]
    flip = rng.random(len(pr)) < 0.5
    order = rng.permutation(len(pr))
    given = np.where(flip[:, None], pr[:, ::-1], pr)[order].astype(np.int32)
    out = pkg.screen_lists(n, given, s[order])
    assert out["trimers"].tolist() == [list(t) for t in tri]
    assert [tuple(p) for p in out["close"]] == sorted(close)
    m = len(tri)
    buf = np.full((m + 4, 3), -1, dtype=np.int32)
    nc, nw, nt = (np.zeros(1, dtype=np.int64) for _ in range(3))
    g, v = np.ascontiguousarray(given), np.ascontiguousarray(s[order])
    for cap in {m, max(m - 1, 0)}:
        rc = _lib.load().mbe3_screen_lists(
            n, _lib.ptr(g), len(g), _lib.ptr(v), pkg.S2B_DISTANT, pkg.S2B_CLOSE, pkg.S3B_KEEP,
            None, None, _lib.ptr(nc), None, _lib.ptr(nw), _lib.ptr(buf), cap, _lib.ptr(nt))
        assert (rc == 0) == (cap >= m)
        assert buf[:cap].tolist() == [list(t) for t in tri[:cap]]
        assert (buf[m:] == -1).all()
