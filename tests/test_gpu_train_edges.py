"""Training at the edges of the count pass: rows at the end of the buffer (whose
last load crosses it), feature counts at the edges of a lane's features, of its
int32 groups of four and of a 1,024-feature chunk, row counts at the edges of
a 64-row window, of a wave's list and of a slot, and padding that is no feature
(negative or large values there must change nothing).  Counts are exact."""
import numpy as np
import pytest
import torch

import paper_1905_13746_amd as nbg
from oracle import nb
from synth import workloads as W
from tests.parity import assert_tables, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _fit(X, y, C, kind):
    m = nbg.Model(C, X.shape[1], kind)
    nbg.train(m, X, y)
    assert m.trained
    assert_tables(m, nb.train(to_np(X), to_np(y), C, kind), kind)


# classes, features, rows, row padding (elements)
CASES = [(2, 1, 64, 3), (2, 3, 65, 1), (2, 4, 255, 0), (2, 17, 256, 3), (2, 64, 257, 0), (2, 255, 1023, 1),
         (2, 1000, 2049, 0), (2, 1028, 300, 0), (3, 64, 1025, 4), (7, 1023, 511, 1), (12, 260, 4097, 0),
         (16, 2049, 513, 7)]


@pytest.mark.parametrize("kind", [nb.MULTINOMIAL, nb.BERNOULLI, nb.GAUSSIAN])
@pytest.mark.parametrize("x", ["u8", "i32"])
@pytest.mark.parametrize("C,F,n,pad", CASES, ids=[f"C{c}_F{f}_n{n}_pad{p}" for c, f, n, p in CASES])
def test_edges(C, F, n, pad, x, kind):
    print(f"[case] training edges C={C} F={F} n={n} pad={pad} {x} {kind}", flush=True)
    wl = W.Workload(wid=8, n_classes=C, n_features=F, p_zero=0.6, clip255=x == "u8", group=C * 4096 + F)
    X, y = wl.train_set(n, device=DEV)
    X[0, 0] = 3      # no Gaussian model is all zero variance
    wide = torch.full((n, F + pad), 255 if x == "u8" else -5, dtype=X.dtype, device=DEV)
    wide[:, :F] = X
    # the buffer ends with the last row's last feature
    _fit(wide.flatten()[:(n - 1) * (F + pad) + F].as_strided((n, F), (F + pad, 1)), y, C, kind)


@pytest.mark.parametrize("F", [5, 1027])
def test_int32_errors_only_from_features(F):
    """A negative value is found in every feature, also in the last, partial
    group of four, and a Gaussian model refuses values of 65,536 there."""
    n = 130
    y = (torch.arange(n, device=DEV) % 2).to(torch.int32)
    for f in (0, F - 2, F - 1):
        for value, kind, code in ((-1, nb.MULTINOMIAL, -5), (-1, nb.BERNOULLI, -5), (65_536, nb.GAUSSIAN, -2)):
            X = torch.randint(0, 9, (n, F), dtype=torch.int32, device=DEV)
            X[n - 1, f] = value
            with pytest.raises(nbg.NBError) as e:
                nbg.train(nbg.Model(2, F, kind), X, y)
            assert e.value.code == code
