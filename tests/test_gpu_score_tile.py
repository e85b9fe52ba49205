"""GPU parity of the matrix-core scoring of byte features for more than two
classes (FP32 table in three BF16 parts, BF16 table): class counts at the edges
of the 16-class column tiles, feature counts at the edges of the 64-feature
windows, 128-feature sums and 512-feature slices, file counts at the edges of a
16-file tile and a workgroup's 64 and 128 files, and enough files for the wide
tiles (more than 32,768), whose results must equal those of small calls bit for
bit.  Tolerances: tests/parity.py (the bounds of a deeper sum than this one)."""
import numpy as np
import pytest
import torch

import paper_1905_13746_amd as nbg
from oracle import nb, precision as P
from synth import workloads as W
from tests.parity import X_FP8, X_U8, assert_scores, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _model(C, F, kind, n=None):
    wl = W.Workload(wid=6, n_classes=C, n_features=F, p_zero=0.8, clip255=True, group=C * 8192 + F)
    X, y = wl.train_set(n or max(2000, 12 * C), device=DEV)
    m = nbg.Model(C, F, kind)
    nbg.train(m, X, y)
    return wl, m, nb.train(to_np(X), to_np(y), C, kind)


# (classes, features, files, raw scores): FP32 table, at most 32 score rows
F32 = [(3, 4, 1, True), (15, 60, 15, True), (16, 64, 16, True), (16, 512, 17, True), (16, 516, 127, False),
       (16, 1024, 128, True), (16, 1028, 129, True), (17, 124, 300, True), (31, 1540, 65, True), (32, 128, 200, False)]


@pytest.mark.parametrize("kind", [nb.MULTINOMIAL, nb.BERNOULLI])
@pytest.mark.parametrize("C,F,n,scores", F32, ids=[f"C{c}_F{f}_n{n}" for c, f, n, _ in F32])
def test_fp32_table(C, F, n, scores, kind):
    print(f"[case] fp32 tile C={C} F={F} n={n} {kind}", flush=True)
    wl, m, om = _model(C, F, kind)
    X, _ = wl.test_set(n, device=DEV)
    lab, lp, sc = nbg.score(m, X, scores=scores)
    torch.cuda.synchronize()
    assert_scores(om, to_np(X), to_np(lab), to_np(lp), to_np(sc) if scores else None)


# BF16 table: up to 256 score columns
BF16 = [(3, 60, 17, True), (15, 508, 130, True), (16, 1028, 65, True), (32, 512, 127, True), (33, 516, 129, False),
        (48, 1024, 63, True), (49, 1540, 64, False), (64, 260, 257, True), (65, 132, 128, False), (128, 132, 33, True),
        (255, 388, 70, True), (256, 128, 16, False)]


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("C,F,n,scores", BF16, ids=[f"C{c}_F{f}_n{n}" for c, f, n, _ in BF16])
def test_bf16_table(C, F, n, scores, fp8):
    print(f"[case] bf16 tile C={C} F={F} n={n} fp8={fp8}", flush=True)
    wl, m, om = _model(C, F, nb.MULTINOMIAL)
    X, _ = wl.test_set(n, device=DEV)
    x = W.to_fp8_e4m3(X) if fp8 else X
    lab, lp, sc = nbg.score(m, x, wtype=nbg.W_BF16, fp8=fp8, scores=scores)
    torch.cuda.synchronize()
    assert_scores(om, P.e4m3_value(to_np(x)) if fp8 else to_np(x), to_np(lab), to_np(lp),
                  to_np(sc) if scores else None, wtype=nbg.W_BF16, xtype=X_FP8 if fp8 else X_U8)


@pytest.mark.parametrize("C,F,n,wtype", [(16, 260, 65_536 + 37, 0), (16, 1540, 33_000, 0), (7, 60, 98_305, 1),
                                         (40, 260, 40_001, 1)])
def test_wide_tiles_equal_small_calls(C, F, n, wtype):
    print(f"[case] wide tiles C={C} F={F} n={n} wtype={wtype}", flush=True)
    wl, m, _ = _model(C, F, nb.MULTINOMIAL)
    ld = F + 4
    X = torch.full((n, ld), 255, dtype=torch.uint8, device=DEV)
    X[:, :F] = wl.test_set(n, device=DEV)[0]
    X = X[:, :F]
    full = nbg.score(m, X, wtype=wtype, scores=True)
    for a, b in ((0, 1), (100, 229), (32_767, 32_800), (n - 150, n)):
        part = nbg.score(m, X[a:b], wtype=wtype, scores=True)
        for u, v in zip(full, part):
            assert torch.equal(u[a:b], v)
    # unrequested outputs change nothing
    lab, none, _ = nbg.score(m, X, wtype=wtype, log_post=False)
    assert none is None and torch.equal(lab, full[0])


def test_fp8_values_past_the_last_feature():
    """NaN encodings in the padding bytes are not features."""
    C, F = 20, 500
    wl, m, _ = _model(C, F, nb.MULTINOMIAL)
    X, _ = wl.test_set(300, device=DEV)
    pad = torch.full((300, 512), 0x7F, dtype=torch.uint8, device=DEV)
    pad[:, :F] = W.to_fp8_e4m3(X)
    for wtype in (nbg.W_F32, nbg.W_BF16):
        got = nbg.score(m, pad[:, :F], wtype=wtype, fp8=True)[1]
        want = nbg.score(m, pad[:, :F].contiguous(), wtype=wtype, fp8=True)[1]
        assert torch.isfinite(got).all() and torch.equal(got, want)


@pytest.mark.parametrize("kind", [nb.MULTINOMIAL, nb.BERNOULLI])
def test_three_parts_are_the_fp32_table(kind):
    """One feature per file: the score is bias + x W of one FP32 entry, which
    the three BF16 parts must carry whole (x a power of two: exact products)."""
    C, F = 16, 640
    _, m, _ = _model(C, F, kind)
    X = torch.zeros((F, F), dtype=torch.uint8, device=DEV)
    X.fill_diagonal_(1)
    lab, lp, sc = nbg.score(m, X, scores=True)
    torch.cuda.synchronize()
    rows, b = to_np(m.form_f32())[:, :F], to_np(m.form_bias())
    # fl(fl(W) + bias) of the centred row, plus that of the aux row: FP32
    want = (rows[:C] + b[:C, None]) + (rows[C] + b[C])[None, :]
    assert np.array_equal(to_np(sc).T, want.astype(np.float32))
