"""Input that only the device looks at: labels and values are checked there while the solve is already
queued, and the call still refuses them; the sums over a problem's samples, taken by several
workgroups, at the edges of their shares and when the solve is cut into many launches."""
import numpy as np
import pytest
import torch

from paper_2311_14908_amd import svmx, synth

pytestmark = pytest.mark.gpu


def _problem(n, d, seed=0):
    X, y = synth.two_blobs(n, d, seed)
    return torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()


@pytest.mark.parametrize("kw", [dict(), dict(gram=svmx.GRAM_OFF), dict(gram_mfma=svmx.MFMA_F32), dict(working_set=8),
                                dict(working_set=8, gram=svmx.GRAM_OFF), dict(working_set=-1)])
@pytest.mark.parametrize("n", [3, 300, 5000])
def test_refused(n, kw):
    X, y = _problem(n, 7)
    for at, value in ((0, 0), (n - 1, 2), (n // 2, -2147483648)):
        bad = y.clone()
        bad[at] = value
        if at + 1 < n:
            bad[n - 1] = 7  # the first one is reported
        with pytest.raises(svmx.SvmError) as e:
            svmx.svm_train(X, bad, 1.0, 0.1, 1e-3, **kw)
        assert e.value.status == svmx.SVM_EINVAL and f"y[{at}] = {value} " in str(e.value)
    for only in (1, -1):
        with pytest.raises(svmx.SvmError) as e:
            svmx.svm_train(X, torch.full_like(y, only), 1.0, 0.1, 1e-3, **kw)
        assert e.value.status == svmx.SVM_EINVAL and "both classes" in str(e.value)
    for at, value in ((0, float("nan")), (X.numel() - 1, float("inf")), (X.numel() // 2, -float("inf"))):
        Xb = X.clone()
        Xb.view(-1)[at] = value
        with pytest.raises(svmx.SvmError) as e:
            svmx.svm_train(Xb, y, 1.0, 0.1, 1e-3, **kw)
        assert e.value.status == svmx.SVM_EINVAL and "not finite" in str(e.value)
    big = X.clone()
    big.view(-1)[0] = 3e38  # finite, though its square is not
    assert svmx.svm_train(big, y, 1.0, 0.1, 1e-3, **kw).status == svmx.SVM_OK
    assert svmx.svm_train(X, y, 1.0, 0.1, 1e-3, **kw).status == svmx.SVM_OK


def test_refused_one_vs_one():
    X, _ = _problem(600, 9)
    lab = (torch.arange(600, device="cuda") % 4).int()
    for kw in (dict(), dict(gram=svmx.GRAM_OFF), dict(gram_mfma=svmx.MFMA_F32)):
        for at in (0, X.numel() - 1):
            Xb = X.clone()
            Xb.view(-1)[at] = float("nan")
            with pytest.raises(svmx.SvmError) as e:
                svmx.svm_train_ovo(Xb, lab, 4, 1.0, 0.1, 1e-3, **kw)
            assert e.value.status == svmx.SVM_EINVAL and "not finite" in str(e.value)


@pytest.mark.parametrize("n,check_every", [(2, 0), (1024, 50), (1025, 0), (2047, 37), (30000, 0), (30000, 400)])
def test_sums(n, check_every):
    """Objective and counts from alpha and f: at most 24 shares of n samples, ragged ones among them."""
    X, y = _problem(n, 5, 3)
    f = torch.empty(n, dtype=torch.float64, device="cuda")
    out = svmx.svm_train(X, y, 1.0, 0.2, 1e-3, check_every=check_every, f_out=f)
    a, yy, ff = out.alpha.cpu().numpy(), y.cpu().numpy().astype(np.float64), f.cpu().numpy()
    W = 0.5 * a.sum() - 0.5 * (a * yy * ff).sum()
    assert abs(out.stats["dual_obj"] - W) <= 1e-12 * np.abs(a).sum()
    assert out.stats["n_sv"] == int((a > 0).sum()) and out.stats["n_bound_sv"] == int((a >= 1.0).sum())
    if check_every:
        assert out.stats["launches"] > 1
