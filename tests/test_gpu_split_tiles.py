"""The split-fp16 Gram at the edges of its tiles, chunks and stores: row counts around the 8-row load
chunks and the 128-row tiles, feature counts around the 32-feature stages and past what a lane keeps
in registers, row pitches of every alignment (plain and non-temporal stores), and X at an odd
address."""
import numpy as np
import pytest
import torch

from paper_2311_14908_amd import svmx

pytestmark = pytest.mark.gpu

# fp32 accumulation of d products of values below 1 and the fp32 epilogue: |dot| <= d/4 on average,
# so the exponent's absolute error is at most about gamma * d * 2^-22, below 1e-6 for gamma = 4 / d.
REL = 1e-5


def _x(n, d, seed, shift=0):
    g = np.random.default_rng(seed)
    flat = torch.from_numpy(g.random(n * d + shift, dtype=np.float32)).cuda()
    return flat[shift:].reshape(n, d)


def _gram64(X, gamma):
    X = X.double()
    s = X.square().sum(1)
    K = torch.exp(-gamma * (s[:, None] + s[None, :] - 2.0 * X @ X.T).clamp_(min=0.0))
    return K.fill_diagonal_(1.0)


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 63, 64, 65, 127, 128, 129, 200, 257])
@pytest.mark.parametrize("d,shift", [(1, 0), (31, 1), (32, 0), (33, 0), (100, 3), (2049, 0)])
def test_gram_tile_edges(n, d, shift):
    X = _x(n, d, 100 * n + d, shift)
    ref = _gram64(X, 4.0 / d)
    for ld in (n, n + 1, n + 2, (n + 3) // 4 * 4):
        G = svmx.svm_gram(X, 4.0 / d, ld=ld)[:, :n]
        assert torch.equal(G, G.T), (n, d, ld)
        assert float(((G.double() - ref).abs() / ref).max()) <= REL, (n, d, ld)


@pytest.mark.parametrize("ld", [8128, 8129, 8192])
def test_gram_store_kinds(ld):
    """264 MB and more: non-temporal stores where the rows are aligned, plain ones elsewhere, with a last
    tile of 63 rows; what lies past a row's n entries is not written."""
    n, d = 8127, 40
    X = _x(n, d, ld)
    G = svmx.svm_gram(X, 4.0 / d, ld=ld)
    small = svmx.svm_gram(X[:2001].contiguous(), 4.0 / d, ld=2001)
    assert torch.equal(G[:2001, :2001], small)  # the same value wherever a pair's tile lies
    rows = torch.tensor([0, 127, 128, 4095, 8064, n - 1], device="cuda")
    s = X.double().square().sum(1)
    ref = torch.exp(-4.0 / d * (s[rows, None] + s[None, :] - 2.0 * X[rows].double() @ X.double().T).clamp_(min=0.0))
    ref[torch.arange(len(rows)), rows] = 1.0
    assert float(((G[rows, :n].double() - ref).abs() / ref).max()) <= REL
    assert torch.equal(G[:, rows], G[rows, :n].T.contiguous())
