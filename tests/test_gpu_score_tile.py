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
from tests.parity import X_FP8, X_I32, X_U8, assert_scores, to_np

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


@pytest.mark.parametrize("C,F,n", [(16, 1028, 131_072 + 301), (20, 1540, 140_001)])
def test_four_units_per_slice_equal_small_calls(C, F, n):
    """FP32 tables that do not stay in LDS, enough files for four units per wave."""
    print(f"[case] four units C={C} F={F} n={n}", flush=True)
    wl, m, _ = _model(C, F, nb.MULTINOMIAL)
    base, _ = wl.test_set(1999, device=DEV)
    X = base.repeat(n // 1999 + 1, 1)[:n]
    want = nbg.score(m, base, scores=True)
    rows = torch.arange(n, device=DEV) % 1999
    for u, v in zip(nbg.score(m, X, scores=True), want):
        assert torch.equal(u, v[rows])


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


# int32 features on FP32 MFMAs: feature counts at the edges of a lane's four, of
# the 16-feature sums and of the 256-feature slices, and padding that is no feature
I32 = [(3, 1, 1, 3, True), (15, 3, 17, 1, True), (16, 64, 130, 0, True), (16, 255, 129, 1, False), (16, 257, 64, 0, True),
       (17, 512, 33, 0, True), (31, 516, 200, 4, True), (32, 1030, 65, 2, False), (7, 2049, 300, 0, True)]


@pytest.mark.parametrize("wtype", [0, 1])
@pytest.mark.parametrize("kind", [nb.MULTINOMIAL, nb.BERNOULLI])
@pytest.mark.parametrize("C,F,n,pad,scores", I32, ids=[f"C{c}_F{f}_n{n}" for c, f, n, _, _ in I32])
def test_int32_features(C, F, n, pad, scores, kind, wtype):
    print(f"[case] int32 tile C={C} F={F} n={n} {kind} wtype={wtype}", flush=True)
    wl = W.Workload(wid=6, n_classes=C, n_features=F, p_zero=0.7, clip255=False, group=C * 8192 + F)
    X, y = wl.train_set(max(1000, 12 * C), device=DEV)
    m = nbg.Model(C, F, kind)
    nbg.train(m, X, y)
    om = nb.train(to_np(X), to_np(y), C, kind)
    wide = torch.full((n, F + pad), -9, dtype=torch.int32, device=DEV)
    wide[:, :F] = wl.test_set(n, device=DEV)[0]
    x = wide.flatten()[:(n - 1) * (F + pad) + F].as_strided((n, F), (F + pad, 1))
    lab, lp, sc = nbg.score(m, x, wtype=wtype, scores=scores)
    torch.cuda.synchronize()
    assert_scores(om, to_np(x), to_np(lab), to_np(lp), to_np(sc) if scores else None, wtype=wtype, xtype=X_I32)


def test_int32_wide_tiles_and_limits():
    C, F, n = 16, 300, 40_003
    wl = W.Workload(wid=6, n_classes=C, n_features=F, p_zero=0.7, clip255=False, group=5)
    X, y = wl.train_set(1000, device=DEV)
    m = nbg.Model(C, F, nb.MULTINOMIAL)
    nbg.train(m, X, y)
    T, _ = wl.test_set(n, device=DEV)
    full = nbg.score(m, T, scores=True)
    for a, b in ((0, 1), (100, 229), (32_767, 32_800), (n - 150, n)):
        for u, v in zip(full, nbg.score(m, T[a:b], scores=True)):
            assert torch.equal(u[a:b], v)
    for wtype in (nbg.W_F32, nbg.W_BF16):        # 33 score rows stay refused
        with pytest.raises(nbg.NBError) as e:
            nbg.score(nbg.Model(32, 8, nb.MULTINOMIAL), T[:10, :8].contiguous(), wtype=wtype, scores=True)
        assert e.value.code == -1
