"""The work a user of the library has it do, as cases that can be timed and
checked: training, scoring, the size groups, feature selection and gather, each
through the package's public functions, over the ranges they are used at.

Inputs are drawn as the method's data is: class rates from Gamma(0.5, 2),
Poisson occurrence counts that are zeroed with probability 0.8 (0.7 for int32
counts), clipped at 255 where they are bytes; labels balanced or from Dirichlet(1)
class priors.  They depend on the seed alone.  Every case's `path` names
the entry points that one pass goes through:

  train     nb_train of one model; outputs: the exact counts and class totals,
            the FP64 tables and the scoring rows
  score     nb_score of n files by a trained model; outputs: labels, log
            posteriors and, where asked for, raw scores
  gaussian  nb_train of a Gaussian model, then nb_score of new files by it
  groups    one grouped launch over size groups, each with its own model
            (a captured plan's replay, or the eager call)
  select    the top-k features of each size group's model and the k-feature
            models on them
  gather    the k selected columns of every file
"""
import math

import numpy as np
import torch

import paper_1905_13746_amd as nbg

CHUNK = 1 << 27          # elements drawn or computed at once


def listed():
    return [
        # one size group's files of the paper's experiment, scanned as they come in (768 files, the
        # group's 200 selected opcodes): the smallest call
        dict(name="score_one_group", path="score", kind="multinomial", x="u8", w="f32", C=2, F=200, n=768, scores=True),
        # the smallest training: 64 int32 occurrence counts of 2,000 files, waiting for the outcome
        dict(name="train_tiny", path="train", kind="multinomial", x="i32", C=2, F=64, n=2000, wait=True),
        # the two-class detector at the benchmark's sizes, trained step by step
        dict(name="train_detector", path="train", kind="multinomial", x="u8", C=2, F=1000, n=200_000, wait=False),
        # malware families with skewed priors
        dict(name="train_families", path="train", kind="multinomial", x="u8", C=16, F=4096, n=200_003, wait=False),
        # the Gaussian variant: fit, then classify new files
        dict(name="gaussian_step", path="gaussian", kind="gaussian", x="u8", w="f32", C=2, F=1000, n=200_000,
             n_test=200_001, wait=False),
        # the two-class detector over a large batch of files
        dict(name="score_detector", path="score", kind="multinomial", x="u8", w="f32", C=2, F=1000, n=1_000_000,
             scores=False),
        # malware families in full precision, raw scores kept
        dict(name="score_families_f32", path="score", kind="multinomial", x="u8", w="f32", C=16, F=4096, n=400_003,
             scores=True),
        # malware families in reduced precision: FP8 features, BF16 table
        dict(name="score_families_fp8", path="score", kind="multinomial", x="fp8", w="bf16", C=16, F=4096, n=500_000,
             scores=False),
        # more families than a matrix tile holds, presence of opcodes, raw scores kept
        dict(name="score_many_classes", path="score", kind="bernoulli", x="u8", w="bf16", C=40, F=1000, n=400_001,
             scores=True),
        # 256 size groups of lognormal size, each with its own model, replayed step by step
        dict(name="groups_plan", path="groups", kind="multinomial", x="u8", w="f32", C=2, F=2000, groups=256, mu=7.0,
             plan=True),
        # the per-group top-200 opcodes of 20 size groups and the groups' models on them
        dict(name="select_models", path="select", kind="multinomial", x="u8", C=2, F=1024, k=200, groups=20),
        # the selected opcodes of every file
        dict(name="gather_selected", path="gather", x="u8", F=2000, k=200, n=500_001),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["train", "train", "score", "score", "score", "gaussian", "groups", "select", "gather"])
    most = 800_000_000   # bytes of features in a drawn case
    if path == "train":
        x = rng.choice(["u8", "u8", "i32"])
        C = rng.choice([2, 2, 3, 7, 16])
        F = 4 * _logint(rng, 12, 1024)
        n = min(_logint(rng, 60 * C, 400_000), most // (F * (4 if x == "i32" else 1)))
        return dict(path=path, kind=rng.choice(["multinomial", "bernoulli"]), x=x, C=C, F=F, n=n,
                    wait=rng.random() < 0.5)
    if path == "score":
        x = rng.choice(["u8", "u8", "u8", "fp8", "i32"])
        C = rng.choice([2, 2, 3, 7, 16, 16, 24, 40, 100])
        w = rng.choice(["f32", "bf16"]) if C <= 24 else "bf16"
        if C > 24 and x == "i32":
            x = "u8"
        # the k-feature models of the paper for two classes, wider ones for the families
        F = 4 * (_logint(rng, 5, 1250) if C == 2 else _logint(rng, 64, 1024))
        n = min(_logint(rng, 100, 1_000_000), most // (F * (4 if x == "i32" else 1)))
        if C > 16:
            n = min(n, 150_000)
        return dict(path=path, kind=rng.choice(["multinomial", "multinomial", "bernoulli"]), x=x, w=w, C=C, F=F, n=n,
                    scores=rng.random() < 0.4)
    if path == "gaussian":
        F = 4 * _logint(rng, 16, 1000)
        n = min(_logint(rng, 500, 300_000), most // F)
        return dict(path=path, kind="gaussian", x="u8", w="f32", C=2, F=F, n=n, n_test=_logint(rng, 100, n),
                    wait=rng.random() < 0.5)
    if path == "groups":
        F = rng.choice([40, 200, 512, 1000, 2000])
        groups = rng.randint(8, 128)
        return dict(path=path, kind=rng.choice(["multinomial", "bernoulli"]), x="u8", w=rng.choice(["f32", "bf16"]),
                    C=2, F=F, groups=groups, mu=round(rng.uniform(4.0, 7.0), 2), plan=rng.random() < 0.6)
    if path == "select":
        F = _logint(rng, 64, 2000)
        return dict(path=path, kind=rng.choice(["multinomial", "bernoulli"]), x="u8", C=2, F=F,
                    k=rng.randint(10, min(200, F)), groups=rng.randint(2, 20))
    F = 4 * _logint(rng, 64, 1250)
    return dict(path=path, x=rng.choice(["u8", "u8", "i32"]), F=F, k=rng.randint(20, 200),
                n=min(_logint(rng, 1000, 500_000), most // (4 * F)))


# ----------------------------------------------------------------- inputs

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _torch_rng(seed, stream):
    g = torch.Generator(device=_device())
    g.manual_seed(1_000_003 * int(seed) + stream)
    return g


def _features(rates, y, g, x, ld):
    """[n, F] occurrence counts of files with labels y (rows `ld` apart)."""
    n, F = y.numel(), rates.shape[1]
    p_keep = 0.3 if x == "i32" else 0.2
    dtype = torch.int32 if x == "i32" else torch.uint8
    out = torch.zeros((n, ld), dtype=dtype, device=y.device)
    for r in range(0, n, max(1, CHUNK // F)):
        yy = y[r:r + max(1, CHUNK // F)].long()
        v = torch.poisson(rates[yy], generator=g)
        keep = torch.empty(v.shape, dtype=torch.float32, device=v.device).uniform_(generator=g) < p_keep
        v.mul_(keep)
        if x != "i32":
            v.clamp_(max=255.0)
        if x == "fp8":
            v = v.clamp_(max=240.0).to(torch.float8_e4m3fn).view(torch.uint8)
        out[r:r + yy.numel(), :F] = v.to(dtype)
    return out[:, :F]


def _class_rates(C, F, seed, stream):
    rng = np.random.default_rng([int(seed), stream])
    return torch.from_numpy(rng.gamma(0.5, 2.0, size=(C, F)).astype(np.float32)).to(_device())


def _labels(C, n, seed, stream):
    """Balanced labels for two classes, Dirichlet(1) priors (bounded below) for
    more; the first 6 C files hold six of every class."""
    i = torch.arange(n, device=_device())
    if C == 2:
        return (i % 2).to(torch.int32)
    prior = 0.8 * np.random.default_rng([int(seed), stream]).dirichlet(np.ones(C)) + 0.2 / C
    cum = torch.from_numpy(np.cumsum(prior)[:-1].astype(np.float32)).to(i.device)
    u = torch.empty(n, dtype=torch.float32, device=i.device).uniform_(generator=_torch_rng(seed, stream))
    y = torch.bucketize(u, cum)
    return torch.where(i < 6 * C, i % C, y).to(torch.int32)


def _stride(case):
    return -(-case["F"] // 4) * 4


def _train_inputs(case, seed, n, x=None, stream=0):
    rates = _class_rates(case["C"], case["F"], seed, 100 + stream)
    y = _labels(case["C"], n, seed, 200 + stream)
    return _features(rates, y, _torch_rng(seed, 300 + stream), x or case["x"], _stride(case)), y


def _test_inputs(case, seed, n, x=None, stream=0):
    rates = _class_rates(case["C"], case["F"], seed, 100 + stream)
    y = _labels(case["C"], n, seed, 400 + stream)
    return _features(rates, y, _torch_rng(seed, 500 + stream), x or case["x"], _stride(case))


def _train_type(case):
    return "i32" if case["x"] == "i32" else "u8"


def _model_files(case):
    """Training files of a model that is only scored with."""
    return max(4000, 200 * case["C"])


def _group_sizes(case):
    """File counts of the groups: lognormal(mu, 1.5) in [100, 100,000], the same for every seed."""
    rng = np.random.default_rng([case["groups"], int(round(100 * case["mu"]))])
    return np.clip(np.rint(rng.lognormal(case["mu"], 1.5, size=case["groups"])), 100, 100_000).astype(np.int64)


# ------------------------------------------------------------------- passes

def _wtype(case):
    return nbg.W_BF16 if case["w"] == "bf16" else nbg.W_F32


def _model_outputs(m):
    """The parts of a trained model's buffer that scoring and export read."""
    out = {"counts": m.counts(), "class_totals": m.class_totals(), "weight": m.weight(), "bias": m.bias(),
           "form_f32": m.form_f32(), "form_bias": m.form_bias()}
    if m.kind == nbg.GAUSSIAN:
        out.update(sumsq=m.sumsq(), mean=m.mean(), var=m.var(), form2_f32=m.form2_f32())
    else:
        out.update(log_theta=m.log_theta())
    return out


def _fitted(case, seed, stream=0, n=None):
    X, y = _train_inputs(case, seed, n or _model_files(case), _train_type(case), stream)
    m = nbg.Model(case["C"], case["F"], case["kind"])
    nbg.train(m, X, y)
    return m


def prepare(case, seed):
    path = case["path"]
    s = {"case": case}
    if path in ("train", "gaussian"):
        s["x"], s["y"] = _train_inputs(case, seed, case["n"])
        s["model"] = nbg.Model(case["C"], case["F"], case["kind"])
        s["ws"] = nbg.train_workspace(s["model"], case["n"], nbg.X_I32 if case["x"] == "i32" else nbg.X_U8)
        s["outputs"] = _model_outputs(s["model"])
        if path == "gaussian":
            s["xt"] = _test_inputs(case, seed, case["n_test"])
    elif path == "score":
        s["model"] = _fitted(case, seed)
        s["xt"] = _test_inputs(case, seed, case["n"])
    elif path == "groups":
        G, sizes = case["groups"], _group_sizes(case)
        at = np.concatenate([[0], np.cumsum(sizes)])
        s["models"] = [_fitted(case, seed, stream=1000 * (g + 1), n=1000) for g in range(G)]
        x = torch.empty((int(at[-1]), case["F"]), dtype=torch.uint8, device=_device())
        for g in range(G):
            x[at[g]:at[g + 1]] = _test_inputs(case, seed, int(sizes[g]), stream=1000 * (g + 1))
        s["labels"] = torch.empty(x.shape[0], dtype=torch.int32, device=x.device)
        s["log_post"] = torch.empty((x.shape[0], 2), dtype=torch.float32, device=x.device)
        s["x"] = x
        s["groups"] = [(g, x[at[g]:at[g + 1]]) for g in range(G)]
        s["outs"] = [(s["labels"][at[g]:at[g + 1]], s["log_post"][at[g]:at[g + 1]], None) for g in range(G)]
        if case["plan"]:
            s["plan"] = nbg.GroupPlan(s["models"], s["groups"], wtype=_wtype(case), outs=s["outs"])
    elif path == "select":
        G, k = case["groups"], case["k"]
        s["models"] = [_fitted(case, seed, stream=1000 * (g + 1), n=1000) for g in range(G)]
        s["idx"] = torch.empty((G, k), dtype=torch.int32, device=_device())
        s["kmodels"] = [nbg.Model(2, k, case["kind"]) for _ in range(G)]
        nbytes = nbg.load().nb_model_select_workspace_bytes(2, k)
        s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=_device())
        s["outputs"] = [(m.weight(), m.bias(), m.form_f32()) for m in s["kmodels"]]
    else:
        s["x"] = _test_inputs(dict(case, C=2), seed, case["n"])
        order = np.random.default_rng([int(seed), 8]).permutation(case["F"])[:case["k"]]
        s["idx"] = torch.from_numpy(np.sort(order).astype(np.int32)).to(_device())
        s["out"] = torch.empty((case["n"], -(-case["k"] // 4) * 4), dtype=s["x"].dtype, device=_device())
        s["out"].zero_()
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "train":
        nbg.train(s["model"], s["x"], s["y"], workspace=s["ws"], asynchronous=not case["wait"])
        return s["outputs"]
    if path == "score":
        return nbg.score(s["model"], s["xt"], wtype=_wtype(case), fp8=case["x"] == "fp8", scores=case["scores"])
    if path == "gaussian":
        nbg.train(s["model"], s["x"], s["y"], workspace=s["ws"], asynchronous=not case["wait"])
        return s["outputs"], nbg.score(s["model"], s["xt"], scores=True)
    if path == "groups":
        if case["plan"]:
            s["plan"].launch()
        else:
            nbg.score_groups(s["models"], s["groups"], wtype=_wtype(case), outs=s["outs"])
        return s["labels"], s["log_post"]
    if path == "select":
        nbg.select_features(s["models"], case["k"], out=s["idx"])
        for g, (full, km) in enumerate(zip(s["models"], s["kmodels"])):
            nbg.model_on_features(full, s["idx"][g], workspace=s["ws"], asynchronous=True, out=km)
        return s["idx"], s["outputs"]
    nbg.gather_features(s["x"], s["idx"], out=s["out"])
    return s["out"]


# ------------------------------------------------- what a pass cannot do without

def work(case):
    path, F = case["path"], case["F"]
    eb = 4 if case["x"] == "i32" else 1
    if path == "gather":
        return {"bytes": case["n"] * (F + case["k"]) * eb, "flops": 0}
    C = case["C"]

    def model_bytes(F, kind):
        # counts, FP64 tables, FP32 and BF16 scoring rows of F features
        rows = 2 if C == 2 else C + 1
        return C * F * (4 + 3 * 8) + rows * F * 6 * (2 if kind == "gaussian" else 1)

    def outputs(n, scores):
        return n * (4 + 4 * C * (2 if scores else 1))

    if path in ("train", "gaussian"):
        b = case["n"] * (F * eb + 4) + model_bytes(F, case["kind"])
        fl = case["n"] * F * (1 if path == "train" else 3)
        if path == "gaussian":
            b += case["n_test"] * F * eb + outputs(case["n_test"], True)
            fl += case["n_test"] * F * 6
        return {"bytes": b, "flops": fl}
    if path == "score":
        n = case["n"]
        return {"bytes": n * F * eb + outputs(n, case["scores"]), "flops": 2 * n * F * (1 if C == 2 else C)}
    if path == "groups":
        n = int(_group_sizes(case).sum())
        return {"bytes": n * F + outputs(n, False), "flops": 2 * n * F}
    return {"bytes": case["groups"] * (2 * F * 4 + case["k"] * 4 + model_bytes(case["k"], case["kind"])),
            "flops": case["groups"] * F * 3}


# --------------------------------------------------------- results in 64 bits

def _values(x, case):
    """The feature values, in float64, of a block of rows."""
    return x.view(torch.float8_e4m3fn).to(torch.float64) if case["x"] == "fp8" else x.to(torch.float64)


def _moments(X, y, C, kind):
    """Class totals, per-class sums (of presence for Bernoulli) and squares."""
    n, F = X.shape
    tot = torch.zeros(C, dtype=torch.float64, device=X.device)
    T = torch.zeros((C, F), dtype=torch.float64, device=X.device)
    Q = torch.zeros_like(T)
    step = max(1, (CHUNK // 2) // F)
    for r in range(0, n, step):
        one = torch.nn.functional.one_hot(y[r:r + step].long(), C).to(torch.float64).T.contiguous()
        v = X[r:r + step].to(torch.float64)
        if kind == "bernoulli":
            v = (v > 0).to(torch.float64)
        tot += one.sum(dim=1)
        T += one @ v
        if kind == "gaussian":
            Q += one @ (v * v)
    return tot, T, Q


def _tables(tot, T, Q, kind):
    """The model of these counts (Laplace smoothing 1), as _model_outputs."""
    C, F = T.shape
    prior = tot.log() - tot.sum().log()
    pad = -(-F // 1024) * 1024

    def padded(rows):
        out = torch.zeros((rows.shape[0], pad), dtype=torch.float64, device=rows.device)
        out[:, :F] = rows
        return out

    out = {"counts": T.round().to(torch.int64), "class_totals": tot.round().to(torch.int64)}
    if kind == "gaussian":
        N = tot.sum()
        eps = 1e-9 * ((N * Q.sum(0) - T.sum(0) ** 2) / N / N).max()
        mean = T / tot[:, None]
        var = (tot[:, None] * Q - T * T) / tot[:, None] / tot[:, None] + eps
        W = -0.5 / var
        b = prior - 0.5 * (2 * math.pi * var).log().sum(1)
        out.update(sumsq=Q.round().to(torch.int64), mean=mean, var=var, weight=W, bias=b, form_f32=None,
                   form2_f32=None, form_bias=torch.stack([b[1] - b[0], b[0]]))
        return out
    if kind == "multinomial":
        lt = (T + 1.0).log() - (T.sum(1, keepdim=True) + F).log()
        W, b = lt, prior
    else:
        den = (tot + 2.0).log()[:, None]
        lt, l1 = (T + 1.0).log() - den, (tot[:, None] - T + 1.0).log() - den
        W, b = lt - l1, prior + l1.sum(1)
    if C == 2:
        rows, rb = torch.stack([W[1] - W[0], W[0]]), torch.stack([b[1] - b[0], b[0]])
    else:
        m, mb = W.mean(0), b.mean()
        rows, rb = torch.cat([W - m, m[None]]), torch.cat([b - mb, mb[None]])
    out.update(weight=W, bias=b, log_theta=lt, form_f32=padded(rows), form_bias=rb)
    return out


def _decided(s, scores):
    best = s.argmax(1)
    return best.to(torch.int64), s - torch.logsumexp(s, 1, keepdim=True), s if scores else None


def _scored(tab, X, case, scores):
    """Labels, log posteriors and raw scores of the files X."""
    parts = []
    step = max(1, (CHUNK // 2) // X.shape[1])
    for r in range(0, X.shape[0], step):
        v = _values(X[r:r + step], case)
        if case["kind"] == "gaussian":
            s = torch.stack([tab["bias"][c] + (tab["weight"][c] * (v - tab["mean"][c]) ** 2).sum(1)
                             for c in range(case["C"])], dim=1)
        else:
            if case["kind"] == "bernoulli":
                v = (v > 0).to(torch.float64)
            s = v @ tab["weight"].T.contiguous() + tab["bias"]
        parts.append(_decided(s, scores))
    return tuple(None if p[0] is None else torch.cat(p) for p in zip(*parts))


def _fitted_tables(case, seed, stream=0, n=None):
    X, y = _train_inputs(case, seed, n or _model_files(case), _train_type(case), stream)
    return _tables(*_moments(X, y, case["C"], case["kind"]), case["kind"])


def exact(case, seed):
    path = case["path"]
    if path == "gather":
        return None          # bytes, no computed numbers
    if path == "train":
        X, y = _train_inputs(case, seed, case["n"])
        return _tables(*_moments(X, y, case["C"], case["kind"]), case["kind"])
    if path == "gaussian":
        X, y = _train_inputs(case, seed, case["n"])
        tab = _tables(*_moments(X, y, 2, "gaussian"), "gaussian")
        return tab, _scored(tab, _test_inputs(case, seed, case["n_test"]), case, True)
    if path == "score":
        return _scored(_fitted_tables(case, seed), _test_inputs(case, seed, case["n"]), case, case["scores"])
    if path == "groups":
        got = []
        for g, n in enumerate(_group_sizes(case)):
            tab = _fitted_tables(case, seed, stream=1000 * (g + 1), n=1000)
            got.append(_scored(tab, _test_inputs(case, seed, int(n), stream=1000 * (g + 1)), case, False))
        return torch.cat([p[0] for p in got]), torch.cat([p[1] for p in got])
    # the ranking |T_1 S_0 - T_0 S_1| is an integer: exact in int64 at these counts
    rows, outs = [], []
    for g in range(case["groups"]):
        X, y = _train_inputs(case, seed, 1000, "u8", 1000 * (g + 1))
        tot, T, Q = _moments(X, y, 2, case["kind"])
        Ti = T.round().to(torch.int64)
        S = Ti.sum(1) if case["kind"] == "multinomial" else tot.round().to(torch.int64)
        d = (Ti[1] * S[0] - Ti[0] * S[1]).abs().cpu().numpy()
        top = np.sort(np.lexsort((np.arange(d.size), -d))[:case["k"]])
        idx = torch.from_numpy(top.astype(np.int64)).to(T.device)
        tab = _tables(tot, T[:, idx], Q[:, idx], case["kind"])
        rows.append(idx)
        outs.append((tab["weight"], tab["bias"], tab["form_f32"]))
    return torch.stack(rows), outs
