"""Residuals that fall into the subnormal numbers: the matrix instructions of
the search keep the fma chain's bits there too, so pivots, histories and cores
are the oracle's."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2407_11290_amd import FN_SEPSUM, PREC_FP64
from paper_2407_11290_amd.api import TTCross, batch_run

pytestmark = pytest.mark.gpu


def sepsum_falling(n, r, first, step, seed):
    """r separable terms, term m of size 10^(first - step m)."""
    rng = np.random.default_rng(seed)
    g = 0.5 + rng.random((r, int(np.sum(n))))
    g[:, :n[0]] *= 10.0 ** (first - step * np.arange(r))[:, None]
    return np.concatenate([[float(r)], g.ravel()])


@pytest.mark.parametrize("n,r", [([40, 33, 50], 6), ([33, 20, 18, 35], 5), ([70, 64, 40], 18)])
def test_subnormal_residuals(n, r):
    print("[case]", n, r, flush=True)
    # pivots of 1e-302 to 1e-305, below them residuals of 1e-317
    params = sepsum_falling(n, r, -302.5, 2.0 / (r - 1), 3)
    caps = [r] * (len(n) - 1)
    kw = dict(seed=2, precision=PREC_FP64, grid=[2] * len(n))
    g, h = (TTCross(n, 0.0, FN_SEPSUM, params, **kw) for _ in range(2))
    o = Oracle(n, 0.0, FN_SEPSUM, params, seed=2, rank_caps=caps)
    for x in (g, h):
        x.set_rank_caps(caps)
    assert g.run() == o.run()
    batch_run([h])
    for x in (g, h):
        assert list(x.ranks()) == list(o.ranks()) == [1] + caps + [1]
        for k in range(1, len(n)):
            hist = o.history(k)
            assert 0.0 < np.min(hist[hist > 0.0]) < 1e-310
            assert np.array_equal(x.history(k).view(np.uint64), hist.view(np.uint64)), k
            assert all(np.array_equal(a, b) for a, b in zip(x.pivots(k), o.pivots(k)[:2])), k
        assert np.isfinite(o.cores_flat()).all()
        assert np.array_equal(x.cores_flat().view(np.uint64), o.cores_flat().view(np.uint64))
