"""What a call asks for changes nothing of what it returns: the order of a file's
sums depends on the features, classes, feature type and table type alone, so labels
and log posteriors are the same bits with and without raw scores, in whatever kernel
a call runs (16 classes on the BF16 table have one of their own without raw scores,
up to 4,096 features)."""
import pytest
import torch

import paper_1905_13746_amd as nbg
from synth import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("kind", ["multinomial", "bernoulli"])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("C,F", [(15, 600), (16, 60), (16, 1000), (16, 4096), (16, 4100), (17, 600), (32, 300)])
def test_raw_scores_change_no_other_output(C, F, fp8, kind):
    print(f"[case] outputs C={C} F={F} fp8={fp8} {kind}", flush=True)
    wl = W.Workload(wid=6, n_classes=C, n_features=F, p_zero=0.6, clip255=True, group=C * 8192 + F)
    X, y = wl.train_set(12 * C, device=DEV)
    m = nbg.Model(C, F, kind)
    nbg.train(m, X, y)
    T, _ = wl.test_set(6007, device=DEV)
    T[:, : F // 2] *= 7          # sums that round
    x = W.to_fp8_e4m3(T) if fp8 else T
    for n in (1, 37, 6007):
        lab, lp, _ = nbg.score(m, x[:n], wtype=nbg.W_BF16, fp8=fp8)
        lab2, lp2, sc = nbg.score(m, x[:n], wtype=nbg.W_BF16, fp8=fp8, scores=True)
        assert torch.equal(lab, lab2) and torch.equal(lp, lp2), n
        assert torch.isfinite(sc).all()


@pytest.mark.parametrize("C,wtype,scores", [(16, nbg.W_BF16, False), (16, nbg.W_BF16, True), (16, nbg.W_F32, False),
                                            (20, nbg.W_BF16, False)])
def test_nan_features(C, wtype, scores):
    """A file with an FP8 NaN among its features has NaN log posteriors and label 0,
    wherever it lies (the last 16 files run with guarded loads), and the files
    beside it are what they are without it."""
    F, n = 500, 75
    wl = W.Workload(wid=6, n_classes=C, n_features=F, p_zero=0.6, clip255=True, group=C)
    X, y = wl.train_set(12 * C, device=DEV)
    m = nbg.Model(C, F, "multinomial")
    nbg.train(m, X, y)
    x = W.to_fp8_e4m3(wl.test_set(n, device=DEV)[0])
    want = nbg.score(m, x, wtype=wtype, fp8=True, scores=scores)
    bad = torch.tensor([0, 5, 33, 64, 73, 74], device=DEV)
    x[bad, torch.arange(len(bad), device=DEV) * 99] = 0x7F
    lab, lp, _ = nbg.score(m, x, wtype=wtype, fp8=True, scores=scores)
    good = torch.ones(n, dtype=torch.bool, device=DEV)
    good[bad] = False
    assert torch.isnan(lp[bad]).all() and (lab[bad] == 0).all()
    assert torch.equal(lp[good], want[1][good]) and torch.equal(lab[good], want[0][good])


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("C,F", [(129, 60), (200, 388), (255, 132)])
def test_many_classes_many_files_equal_small_calls(C, F, fp8):
    """More than 128 score rows: another kernel for more files than a unit per wave."""
    print(f"[case] many classes C={C} F={F} fp8={fp8}", flush=True)
    n, base = 40_005, 1999
    wl = W.Workload(wid=6, n_classes=C, n_features=F, p_zero=0.6, clip255=True, group=C * 512 + F)
    X, y = wl.train_set(12 * C, device=DEV)
    m = nbg.Model(C, F, "multinomial")
    nbg.train(m, X, y)
    T, _ = wl.test_set(base, device=DEV)
    x = W.to_fp8_e4m3(T) if fp8 else T
    want = nbg.score(m, x, wtype=nbg.W_BF16, fp8=fp8, scores=True)
    at = torch.arange(n, device=DEV) % base
    pad = torch.full((n, F + 4), 0x7F, dtype=torch.uint8, device=DEV)
    pad[:, :F] = x[at]
    for u, v in zip(nbg.score(m, pad[:, :F], wtype=nbg.W_BF16, fp8=fp8, scores=True), want):
        assert torch.equal(u, v[at])
