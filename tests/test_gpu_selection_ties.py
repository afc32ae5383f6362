"""Selection under exact ties.  The samples sit on a grid so coarse that every kernel value is exactly 1
(same point) or 0, in fp32 and in fp64 alike, so f takes few values, most samples tie at every step, and
the pair of every step (smallest value, then smallest index) must be the oracle's to the end."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_14908_amd import svmx

pytestmark = pytest.mark.gpu


def _grid(n, seed):
    """x = 64 (c1, c2), c below 64: rows and their squared norms are exact in every path, and distinct
    points are at least 64 apart, exp(-4096) = 0."""
    rng = np.random.default_rng(seed)
    side = max(2, min(64, int(np.sqrt(n / 4))))
    X = (64.0 * rng.integers(0, side, (n, 2))).astype(np.float32)
    y = np.where(rng.random(n) < 0.5, 1, -1).astype(np.int32)
    y[:2] = 1, -1
    return X, y


# one workgroup with 1, 2, 4, 8 and 16 samples a thread (ragged), then several: one poller, two, two levels
@pytest.mark.parametrize("n,wgs,gram", [
    (2, 0, svmx.GRAM_ON), (65, 0, svmx.GRAM_ON), (257, 0, svmx.GRAM_ON), (700, 0, svmx.GRAM_ON), (1500, 0, svmx.GRAM_ON),
    (2500, 0, svmx.GRAM_ON), (4096, 0, svmx.GRAM_ON), (4097, 0, svmx.GRAM_ON), (900, 3, svmx.GRAM_ON), (900, 70, svmx.GRAM_ON),
    (900, 140, svmx.GRAM_ON), (300, 1, svmx.GRAM_OFF), (900, 2, svmx.GRAM_OFF), (3000, 1, svmx.GRAM_OFF), (2000, 140, svmx.GRAM_OFF)])
def test_every_pair_under_ties(n, wgs, gram):
    X, y = _grid(n, n + wgs)
    steps = 400
    ref = oracle.train(X, y, 1.0, 1.0, 1e-3, max_iter=steps, trace_len=steps)
    out = svmx.svm_train(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 1.0, 1.0, 1e-3, gram=gram,
                         workgroups=wgs, max_iter=steps, trace_len=steps)
    assert out.stats["iterations"] == ref.iterations
    k = min(len(ref.trace_ul), len(out.trace_ul))
    np.testing.assert_array_equal(out.trace_ul[:k], ref.trace_ul[:k])
    np.testing.assert_array_equal(out.alpha.cpu().numpy(), ref.alpha)


def test_one_vs_one_pairs_under_ties():
    """Two-range problems in one launch: every pair's multipliers are those of the pair trained alone."""
    n, k = 1203, 3
    X, _ = _grid(n, 5)
    lab = (np.arange(n) % k).astype(np.int32)
    Xd = torch.from_numpy(X).cuda()
    out = svmx.svm_train_ovo(Xd, torch.from_numpy(lab).cuda(), k, 1.0, 1.0, 1e-3)
    offs, sizes = svmx.ovo_offsets(lab, k)
    p = 0
    for a in range(k):
        for b in range(a + 1, k):
            idx = np.concatenate([np.nonzero(lab == a)[0], np.nonzero(lab == b)[0]])
            yy = np.where(lab[idx] == a, 1, -1).astype(np.int32)
            ref = oracle.train(X[idx], yy, 1.0, 1.0, 1e-3)
            got = out.alpha[int(offs[p]):int(offs[p]) + int(sizes[p])].cpu().numpy()
            np.testing.assert_array_equal(got, ref.alpha)
            p += 1
