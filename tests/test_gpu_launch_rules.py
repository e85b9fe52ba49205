"""Launch rules that leave a shape waiting on memory: a call's time against the time
of reading as many bytes as it has to touch (the read probe), taken as the best of
several batches in turn.  The factors lie between what a rule that fills the device
takes and what one measured that does not."""
import pytest
import torch

import paper_1905_13746_amd as nbg

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _us(*calls, batches=7, reps=20):
    """Best time per call of each, in microseconds."""
    best = [float("inf")] * len(calls)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for batch in range(batches + 1):
        for i, call in enumerate(calls):
            a.record()
            for _ in range(reps):
                call()
            b.record()
            b.synchronize()
            if batch:
                best[i] = min(best[i], a.elapsed_time(b) / reps * 1e3)
    return best


@pytest.mark.parametrize("dtype,F,ld,n", [(torch.int32, 4000, 4000, 50_000), (torch.uint8, 2000, 2001, 50_000)])
def test_gather_of_rows_that_are_not_staged(dtype, F, ld, n):
    """Every selected element is a cache line of its own (128 bytes)."""
    k = 20
    x = torch.zeros((n, ld), dtype=dtype, device=DEV)[:, :F]
    idx = torch.arange(k, dtype=torch.int32, device=DEV) * (F // k)
    out = torch.empty((n, k), dtype=dtype, device=DEV)
    lines = torch.zeros(n * min(k * 128, ld * x.element_size() // 16 * 16), dtype=torch.uint8, device=DEV)
    sink = torch.empty(nbg.load().nb_probe_sink_words(), dtype=torch.int32, device=DEV)
    gather, read = _us(lambda: nbg.gather_features(x, idx, out=out), lambda: nbg.probe_read(lines, sink))
    print(f"[time] gather {gather:.1f} us, read of its lines {read:.1f} us", flush=True)
    assert gather < 1.7 * read


def _score_against_read(C, F, n, wtype, factor):
    g = torch.Generator(device=DEV).manual_seed(1)
    x = torch.randint(0, 9, (n, F), generator=g, dtype=torch.uint8, device=DEV)
    y = (torch.arange(20 * C, device=DEV) % C).to(torch.int32)
    m = nbg.Model(C, F)
    nbg.train(m, x[:20 * C], y)
    out = (torch.empty(n, dtype=torch.int32, device=DEV), torch.empty((n, C), dtype=torch.float32, device=DEV), None)
    moved = torch.zeros(n * (F + 4 + 4 * C) // 16 * 16, dtype=torch.uint8, device=DEV)
    sink = torch.empty(nbg.load().nb_probe_sink_words(), dtype=torch.int32, device=DEV)
    score, read = _us(lambda: nbg.score(m, x, wtype=wtype, out=out), lambda: nbg.probe_read(moved, sink))
    print(f"[time] score {score:.1f} us, read of its bytes {read:.1f} us", flush=True)
    assert score < factor * read


@pytest.mark.parametrize("C,F,factor", [(3, 16, 2.5), (7, 64, 4.0)])
def test_short_rows_of_a_few_classes(C, F, factor):
    _score_against_read(C, F, 300_000, nbg.W_F32, factor)


def test_many_classes():
    _score_against_read(200, 1000, 30_000, nbg.W_BF16, 7.0)


def test_training_reads_the_last_row_once():
    """The row that ends the buffer is read byte by byte; where it is alone in its batch
    (1,000 files) the batch's empty places must not read it again."""
    C, F = 7, 1000
    calls = []
    for n in (1000, 1008):
        x = torch.ones((n, F), dtype=torch.uint8, device=DEV)
        y = (torch.arange(n, device=DEV) % C).to(torch.int32)
        m = nbg.Model(C, F, "bernoulli")
        ws = nbg.train_workspace(m, n)
        calls.append(lambda m=m, x=x, y=y, ws=ws: nbg.train(m, x, y, workspace=ws, asynchronous=True))
    alone, beside = _us(*calls)
    print(f"[time] training {alone:.1f} us, with a fuller last batch {beside:.1f} us", flush=True)
    assert alone < 1.15 * beside
