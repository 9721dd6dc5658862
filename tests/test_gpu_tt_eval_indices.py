"""Index lists on the device are not checked; an index outside its mode may
spoil its own value but no other one."""
import numpy as np
import pytest

from paper_2407_11290_amd import FN_SEPSUM, PREC_FP64
from paper_2407_11290_amd.api import TTCross

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,m", [
    ([40, 256, 30, 20], 12, 200000),           # sorted modes, counted into bins
    ([33, 300, 64, 45], 20, 131072),           # the first inner mode is not sorted
])
def test_one_index_out_of_range_leaves_the_others(n, r, m):
    """One place before or past an inner mode: whatever kernel reads such an
    index by itself reads a neighbouring fibre or core, so no access leaves
    the cores."""
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
        k = 1 + t % (len(n) - 2)
        bad[row, k] = [-1, n[k]][(t // 2) % 2]
    got = g.tt_eval(torch.from_numpy(bad).cuda()).cpu().numpy()
    keep = np.ones(m, dtype=bool)
    keep[rows] = False
    assert np.array_equal(got[keep].view(np.uint64), want[keep].view(np.uint64))


@pytest.mark.parametrize("n,r,m", [
    ([33, 256, 3, 257, 40], 16, 262145),       # sorted and unsorted modes, two rounds of chunks
    ([60, 128, 129, 50], 17, 131072),          # ranks up to 32
    ([50, 64, 60, 70], 33, 131073),            # up to 64: sorted modes only
    ([50, 64, 65, 70], 33, 131072),            # the lane groups
    ([20] * 6, 8, 65537),                      # in LDS, two workgroups a CU
])
def test_values_on_both_sides_of_the_kernels(n, r, m):
    """The kernel follows from ranks, modes and count: the same bits as few
    indices at a time, which the lane groups take."""
    print("[case]", n, r, m, flush=True)
    rng = np.random.default_rng(3)
    params = np.concatenate([[float(r)], 0.5 + rng.random(r * int(np.sum(n)))])
    g = TTCross(n, 1e-13, FN_SEPSUM, params, seed=1, precision=PREC_FP64)
    g.run()
    assert int(max(g.ranks())) == r
    idx = np.stack([rng.integers(0, j, m) for j in n], axis=1).astype(np.int32)
    idx[:300] = idx[0]
    y = g.tt_eval(idx)
    for lo in range(0, m, 4000):
        assert np.array_equal(y[lo:lo + 4000].view(np.uint64), g.tt_eval(idx[lo:lo + 4000]).view(np.uint64)), lo
