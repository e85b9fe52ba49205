"""Short rows: a few classes on the vector ALUs (up to 128 bytes for three and four
classes, 64 for five, int32 up to seven) and the matrix-core kernel's short slices
(up to 256 features, 128 for int32), at the edges of both rules, of a 64-byte
sub-step, of a 128-feature slice and of the waves' files, with padding that is no
feature and a buffer that ends with the last row's last feature.  Tolerances:
tests/parity.py."""
import pytest
import torch

import paper_1905_13746_amd as nbg
from oracle import nb, precision as P
from synth import workloads as W
from tests.parity import X_FP8, X_I32, X_U8, assert_scores, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"
XT = {"u8": X_U8, "i32": X_I32, "fp8": X_FP8}


def _case(C, F, x, kind, n, pad):
    wl = W.Workload(wid=6, n_classes=C, n_features=F, p_zero=0.6, clip255=x != "i32", group=C * 512 + F)
    X, y = wl.train_set(max(600, 12 * C), device=DEV)
    m = nbg.Model(C, F, kind)
    nbg.train(m, torch.nn.functional.pad(X, (0, -F % 4))[:, :F], y)
    T, _ = wl.test_set(n, device=DEV)
    if x == "fp8":
        T = W.to_fp8_e4m3(T)
    wide = torch.full((n, F + pad), 0x7F if x == "fp8" else (255 if x == "u8" else -9), dtype=T.dtype, device=DEV)
    wide[:, :F] = T
    rows = wide.flatten()[:(n - 1) * (F + pad) + F].as_strided((n, F), (F + pad, 1))
    return m, nb.train(to_np(X), to_np(y), C, kind), rows


# classes, features, feature type, files, padding, raw scores
CASES = [(3, 1, "u8", 1, 3, True), (3, 64, "u8", 257, 0, True), (3, 127, "u8", 63, 1, False), (4, 128, "u8", 65, 4, True),
         (4, 129, "u8", 130, 3, True), (5, 61, "u8", 300, 3, True), (5, 68, "u8", 129, 0, False),
         (3, 100, "fp8", 200, 4, True), (4, 13, "fp8", 70, 3, False), (5, 64, "fp8", 64, 4, True),
         (3, 32, "i32", 300, 1, True), (4, 33, "i32", 129, 0, True), (7, 16, "i32", 257, 3, True), (7, 17, "i32", 65, 0, True),
         (6, 1, "i32", 66, 1, False), (8, 16, "i32", 300, 0, True),
         (6, 128, "u8", 200, 0, True), (15, 132, "u8", 65, 4, True), (16, 256, "u8", 129, 0, True), (16, 252, "fp8", 64, 4, False),
         (16, 64, "i32", 300, 1, True), (15, 127, "i32", 63, 0, True), (17, 128, "i32", 129, 2, True), (31, 65, "i32", 64, 0, True)]


@pytest.mark.parametrize("wtype", [0, 1])
@pytest.mark.parametrize("kind", [nb.MULTINOMIAL, nb.BERNOULLI])
@pytest.mark.parametrize("C,F,x,n,pad,scores", CASES, ids=[f"C{c}_F{f}_{x}_n{n}" for c, f, x, n, *_ in CASES])
def test_against_the_oracle(C, F, x, n, pad, scores, kind, wtype):
    print(f"[case] short rows C={C} F={F} {x} n={n} {kind} wtype={wtype}", flush=True)
    m, om, rows = _case(C, F, x, kind, n, pad)
    lab, lp, sc = nbg.score(m, rows, wtype=wtype, fp8=x == "fp8", scores=scores)
    torch.cuda.synchronize()
    vals = P.e4m3_value(to_np(rows)) if x == "fp8" else to_np(rows)
    assert_scores(om, vals, to_np(lab), to_np(lp), to_np(sc) if scores else None, wtype=wtype, xtype=XT[x])


@pytest.mark.parametrize("C,F,x", [(3, 64, "u8"), (5, 20, "u8"), (7, 9, "i32"), (12, 200, "u8"), (16, 100, "i32"),
                                   (24, 100, "i32")])
def test_many_files_equal_small_calls(C, F, x):
    print(f"[case] short rows, many files C={C} F={F} {x}", flush=True)
    n, base = 140_003, 1999
    m, _, rows = _case(C, F, x, nb.MULTINOMIAL, base, 4)
    rows = rows.contiguous()
    want = nbg.score(m, rows, scores=True)
    at = torch.arange(n, device=DEV) % base
    for scores in (False, True):
        for u, v in zip(nbg.score(m, rows[at].contiguous(), scores=scores), want):
            assert u is None or torch.equal(u, v[at])
