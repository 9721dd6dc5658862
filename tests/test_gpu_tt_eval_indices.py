"""Index lists on the device are not checked; an index outside its mode may
spoil its own value but no other one."""
import numpy as np
import pytest

from paper_2407_11290_amd import FN_SEPSUM, PREC_FP64
from paper_2407_11290_amd.api import TTCross

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,m", [
    ([40, 256, 30, 20], 12, 65536),            # sorted modes, counted into bins
    ([33, 300, 64, 45], 20, 98304),            # the first inner mode is not sorted
])
def test_one_index_out_of_range_leaves_the_others(n, r, m):
    """Only counts whose kernel keeps every index inside its mode (it sorts by
    them), so that no access leaves the cores."""
    import torch
    print("[case]", n, r, m, flush=True)
    rng = np.random.default_rng(1)
    params = np.concatenate([[float(r)], 0.5 + rng.random(r * int(np.sum(n)))])
    g = TTCross(n, 1e-13, FN_SEPSUM, params, seed=1, precision=PREC_FP64)
    g.run()
    assert int(max(g.ranks())) == r
    idx = np.stack([rng.integers(0, j, m) for j in n], axis=1).astype(np.int32)
    want = g.tt_eval(torch.from_numpy(idx).cuda()).cpu().numpy()
    bad = idx.copy()
    rows = rng.choice(m, 40, replace=False)
    for t, row in enumerate(rows):
        k = t % len(n)
        bad[row, k] = [-1, n[k], 1 << 30, -(1 << 31)][(t // len(n)) % 4]
    got = g.tt_eval(torch.from_numpy(bad).cuda()).cpu().numpy()
    keep = np.ones(m, dtype=bool)
    keep[rows] = False
    assert np.array_equal(got[keep].view(np.uint64), want[keep].view(np.uint64))
