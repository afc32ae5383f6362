"""Input that only the device looks at: labels and values are checked there while the solve is already
queued, and the call still refuses them; the sums over a problem's samples, taken by several
workgroups, at the edges of their shares and when the solve is cut into many launches."""
import ctypes as C

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


def _refusals(X, y):
    bad = y.clone()
    bad[len(y) // 2] = 3
    Xb = X.clone()
    Xb.view(-1)[-1] = float("inf")
    return ((X, bad), (X, torch.ones_like(y)), (Xb, y))


@pytest.mark.parametrize("kw", [dict(), dict(gram=svmx.GRAM_OFF), dict(gram_mfma=svmx.MFMA_F32), dict(working_set=8),
                                dict(working_set=8, gram=svmx.GRAM_OFF), dict(working_set=-1),
                                dict(selection=svmx.SELECT_SECOND_ORDER)])
@pytest.mark.parametrize("n", [300, 5000])
@pytest.mark.parametrize("warm", [False, True])
def test_refused_leaves_the_outputs(n, warm, kw):
    """A call refused for its labels or values has written neither alpha nor b, with and without a warm
    start from another buffer."""
    lib = svmx.load()
    X, y = _problem(n, 7)
    zero = torch.zeros(n, dtype=torch.float64, device="cuda")
    o = svmx.options(alpha_init=zero if warm else None, **kw)
    size = lib.svm_train_workspace_bytes(n, 7, C.byref(o))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    for Xr, yr in _refusals(X, y):
        alpha = torch.full((n,), 0.125, dtype=torch.float64, device="cuda")
        b = C.c_double(7.0)
        assert lib.svm_train(svmx._ptr(Xr), svmx._ptr(yr), n, 7, 1.0, 0.1, 1e-3, svmx._ptr(alpha), C.byref(b),
                             svmx._ptr(ws), size, C.byref(o), None) == svmx.SVM_EINVAL
        assert bool((alpha == 0.125).all()) and b.value == 7.0
    # and a call that is not refused does not read it
    ref = svmx.svm_train(X, y, 1.0, 0.1, 1e-3, **kw)
    assert lib.svm_train(svmx._ptr(X), svmx._ptr(y), n, 7, 1.0, 0.1, 1e-3, svmx._ptr(alpha), C.byref(b), svmx._ptr(ws),
                         size, C.byref(o), None) == svmx.SVM_OK
    if not warm:
        assert torch.equal(alpha, ref.alpha) and b.value == ref.b


def test_refused_one_vs_one_leaves_the_outputs():
    lib = svmx.load()
    X, _ = _problem(600, 9)
    X[-1, -1] = float("nan")
    lab = (torch.arange(600, device="cuda") % 4).int()
    for kw in (dict(), dict(gram=svmx.GRAM_OFF), dict(gram_mfma=svmx.MFMA_F32)):
        o = svmx.options(**kw)
        size = lib.svm_train_ovo_workspace_bytes(600, 9, 4, C.byref(o))
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        alpha = torch.full((1800,), 0.125, dtype=torch.float64, device="cuda")
        b = np.full(6, 7.0)
        assert lib.svm_train_ovo(svmx._ptr(X), svmx._ptr(lab), 600, 9, 4, 1.0, 0.1, 1e-3, svmx._ptr(alpha),
                                 b.ctypes.data_as(C.c_void_p), svmx._ptr(ws), size, C.byref(o), None) == svmx.SVM_EINVAL
        assert bool((alpha == 0.125).all()) and (b == 7.0).all()


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
