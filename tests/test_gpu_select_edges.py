"""Feature selection at the edges of the register-held keys (256, 1,024 and
2,048 features, and one model beyond them in the launch), with ties that reach
the index digits, and the one-launch k-feature models at the edges of its
workgroup's features (256 and 1,024) and beyond: index lists are exact, tables
as in tests/parity.py, and equal bit for bit to training on the columns."""
import numpy as np
import pytest
import torch

import paper_1905_13746_amd as nbg
from oracle import nb, select
from tests.parity import assert_tables, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _model(F, kind, seed, top):
    rng = np.random.default_rng(seed)
    X = rng.integers(0, top, size=(90, F)).astype(np.int32)
    X[:, rng.random(F) < 0.3] = 1        # tied columns
    y = (np.arange(90) % 2).astype(np.int32)
    m = nbg.Model(2, F, kind)
    nbg.train(m, torch.from_numpy(X).to(DEV), torch.from_numpy(y).to(DEV))
    return m, nb.train(X, y, 2, kind), X, y


@pytest.mark.parametrize("kind", [nb.MULTINOMIAL, nb.BERNOULLI])
@pytest.mark.parametrize("F", [2, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049])
def test_select_widths(F, kind):
    print(f"[case] select widths F={F} {kind}", flush=True)
    for top in (2, 300, 20_000_000):
        made = [_model(F, kind, 10 * F + i, top) for i in range(2)]
        for k in sorted({1, 2, F // 2, F - 1, F} - {0}):
            idx = to_np(nbg.select_features([m for m, *_ in made], k))
            for row, (_, om, *_) in zip(idx, made):
                assert row.tolist() == select.select_model_features(om, k).tolist(), (top, k)


def test_select_mixed_widths():
    made = [_model(F, nb.MULTINOMIAL, F, 50) for F in (300, 3000, 64)]
    idx = to_np(nbg.select_features([m for m, *_ in made], 60))
    for row, (_, om, *_) in zip(idx, made):
        assert row.tolist() == select.select_model_features(om, 60).tolist()


@pytest.mark.parametrize("kind", [nb.MULTINOMIAL, nb.BERNOULLI])
@pytest.mark.parametrize("k", [1, 255, 256, 257, 1023, 1024, 1025])
def test_k_feature_models(k, kind):
    print(f"[case] k-feature models k={k} {kind}", flush=True)
    m, om, X, y = _model(1500, kind, k, 40)
    idx = np.random.default_rng(k).integers(0, 1500, size=k).astype(np.int32)     # any order, repeats
    km = nbg.model_on_features(m, torch.from_numpy(idx).to(DEV), alpha=0.5)
    assert km.trained
    direct = nbg.Model(2, k, kind)
    columns = torch.empty((X.shape[0], k), dtype=torch.int32, device=DEV)
    columns.copy_(torch.from_numpy(X[:, idx]))
    nbg.train(direct, columns, torch.from_numpy(y).to(DEV), alpha=0.5)
    for part in ("counts", "class_totals", "class_sums", "log_theta", "log_1m_theta", "weight", "bias", "form_f32",
                 "form_bf16", "form_bias"):
        assert torch.equal(getattr(km, part)(), getattr(direct, part)()), part
    assert_tables(nbg.model_on_features(m, torch.from_numpy(idx).to(DEV)), select.model_on_features(om, idx), kind)


@pytest.mark.parametrize("k", [5, 1024, 1030])
def test_bad_index(k):
    m, *_ = _model(1500, nb.MULTINOMIAL, 1, 9)
    for bad in (-1, 1500):
        idx = torch.arange(k, dtype=torch.int32, device=DEV)
        idx[k - 1] = bad
        with pytest.raises(nbg.NBError) as e:
            nbg.model_on_features(m, idx)
        assert e.value.code == -5
