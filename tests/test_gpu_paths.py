"""Paths of the search that only some shapes and ranks take, at the sizes where
they can go wrong, against the FP64 oracle bit for bit."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2407_11290_amd import FN_HILBERT, FN_SEPSUM, PREC_FP64
from paper_2407_11290_amd.api import TTCross, batch_run

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[case]", *a, flush=True)


def _sepsum(n, r, seed):
    rng = np.random.default_rng(seed)
    return np.concatenate([[float(r)], 0.5 + rng.random(r * int(np.sum(n)))])


def _same(g, o):
    st, ost = g.stats(), o.stats()
    assert list(g.ranks()) == list(o.ranks())
    for key in ("sweeps", "pivoted", "evaluated", "rms", "tau"):
        assert st[key] == ost[key], key
    for k in range(1, g.d):
        gr, gc = g.pivots(k)
        orows, ocols, *_ = o.pivots(k)
        assert np.array_equal(gr, orows) and np.array_equal(gc, ocols), k
        assert np.array_equal(g.history(k), o.history(k)), k
    assert np.array_equal(g.cores_flat(), o.cores_flat())


@pytest.mark.parametrize("n,caps,grid", [
    ([21, 34, 17, 40], [9, 1, 8], 1),          # the middle unfolding stops at once
    ([40, 33, 65], [1, 12], 3),                # one side never grows
    ([33, 20, 31, 18, 25], [2, 9, 1, 7], 2),
])
@pytest.mark.parametrize("fn", [FN_HILBERT, FN_SEPSUM])
def test_unfoldings_that_stop_early(n, caps, grid, fn):
    """Stored entries of an unfolding that committed nothing are not visited
    again; its largest |residual| must still be the whole superblock's in
    every sweep, and its pivots, counts and cores the oracle's."""
    _say("stops early", n, caps, grid, fn)
    params = _sepsum(n, 14, 3) if fn == FN_SEPSUM else None
    kw = dict(seed=4, precision=PREC_FP64, grid=[grid] * len(n))
    g, h = (TTCross(n, 0.0, fn, params, **kw) for _ in range(2))
    o = Oracle(n, 0.0, fn, params, seed=4, rank_caps=caps)
    for x in (g, h):
        x.set_rank_caps(caps)
    assert g.run() == o.run() == 1
    _same(g, o)
    batch_run([h])
    _same(h, o)
