"""Top-k where its kernel changes path: rows at the number of scores one
workgroup keeps in registers (8,192), results at the pairwise-ranking limit
(128), scores that differ in one byte only, in all bytes, or not at all.
Against numpy's lexsort, tolerance 0."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

I32 = np.iinfo(np.int32)


def _scores(kind, n, rng):
    if kind == "equal":
        return np.full(n, 41, np.int32)
    if kind == "low byte":
        return rng.integers(0, 200, n).astype(np.int32)
    if kind == "high byte":
        return (rng.integers(-128, 128, n) << 24).astype(np.int32)
    s = rng.integers(I32.min, I32.max, n, dtype=np.int64).astype(np.int32)
    s[rng.integers(0, n, 3)] = I32.max
    s[rng.integers(0, n, 3)] = I32.min
    return s


@pytest.mark.parametrize("kind", ["equal", "low byte", "high byte", "any"])
@pytest.mark.parametrize("n", [1, 127, 1024, 8191, 8192, 8193, 16385, 40_001, 1_100_000])
def test_rows_and_results_at_the_limits(gpu, n, kind):
    import torch
    rng = np.random.default_rng(n)
    s = _scores(kind, n, rng)
    d = torch.from_numpy(s).cuda()
    for k in (1, 127, 128, 129, 1024):
        want = oracle.topk(s, k)
        one = (torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(k, dtype=torch.int64, device="cuda"))
        gpu.sw_topk(d, n, k, *one)                 # one launch
        for ts, ti in (one, gpu.topk(d, k)):       # and in pieces
            torch.cuda.synchronize()
            assert (ts.cpu().numpy() == want[0]).all() and (ti.cpu().numpy() == want[1]).all(), (n, k)
