"""Workspace slots: more calls in flight than there are slots, of every kind whose last launch says so in its own way, on three streams at
once and from three threads, each stream held up first so that the slots do run out; each result against the same call by itself."""
import threading

import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star
from gpu_util import rand_stream

pytestmark = pytest.mark.gpu

HP = dict(lr=0.1, momentum_coef=0.9, weight_decay=1e-4, wmode="stale")
# kind, rows, dtype, updates, elements, options
CALLS = [("norms", 8, "f32", 16, 300_007, {}), ("update", 16, "bf16", 40, 70_001, {}), ("update", 5, "f32", 9, 65_536, {"queue_threshold": 1}),
         ("plain", 3, "f32", 5, 1_200_000, {"queue_threshold": 1}), ("plain", 16, "f32", 5, 1_200_000, {"queue_threshold": 1}),
         ("plain", 2, "f32", 1, 900_000, {"queue_threshold": 1}), ("plain", 4, "f32", 90, 50_000, {"kernel": star.KERNEL_SEQ}),
         ("plain", 12, "f32", 5, 3000, {"queue_threshold": 1}), ("norms", 12, "bf16", 300, 40_000, {"direct_norms": True}),
         ("gram", 12, "f32", 0, 100_000, {}), ("gram", 24, "bf16", 0, 1 << 20, {}), ("reduce", 6, "f32", 3, 200_001, {"norms": True}),
         ("reduce", 6, "f32", 3, 200_001, {}), ("reduce", 16, "f32", 2, 900_000, {"queue_threshold": 1}), ("reduce", 9, "bf16", 40, 5000, {})]


def _make(i, seed):
    kind, W, dtype, U, P, kw = CALLS[i]
    gen = torch.Generator(device="cuda").manual_seed(100 * i + seed)
    rows = [(torch.randn(P, generator=gen, device="cuda") * 1e-2).to(torch.float32 if dtype == "f32" else torch.bfloat16) for _ in range(W)]
    us = star.UpdateStream(*rand_stream(np.random.default_rng(i), W, max(U, 1), stale=4))
    n = torch.full((max(U, 1),), -1.0, device="cuda")
    p, v = (torch.randn(P, generator=gen, device="cuda") for _ in range(2))
    kw = dict(kw)
    if kind == "gram":
        out = torch.empty(W, W, dtype=torch.float64, device="cuda")
        return lambda s: star.star_group_gram(rows, out, stream=s, **kw), [out]
    if kind == "norms":
        return lambda s: star.star_group_norms(rows, us, n, wmode="stale", stream=s, **kw), [n]
    if kind == "reduce":
        norms = n if kw.pop("norms", False) else None
        out = [torch.empty(P, device="cuda") for _ in range(U)]
        return lambda s: star.star_group_reduce(out, rows, us, wmode="stale", norms_out=norms, stream=s, **kw), out + [n]
    return lambda s: star.star_group_update(p, v, rows, us, norms_out=n if kind == "update" else None, stream=s, **HP, **kw), [p, v, n]


def test_more_calls_than_slots_on_three_streams():
    want = []
    for i in range(len(CALLS)):
        call, out = _make(i, 0)
        call(None)
        torch.cuda.synchronize()
        want.append([x.clone() for x in out])
    streams = [torch.cuda.Stream() for _ in range(3)]
    for repeat in range(6):
        made = [(int(i), *_make(int(i), 0)) for i in np.random.default_rng(repeat).permutation(len(CALLS))]
        torch.cuda.synchronize()
        for k, (i, call, out) in enumerate(made):
            call(streams[(k + repeat) % 3])
        torch.cuda.synchronize()
        for i, call, out in made:
            for a, b in zip(out, want[i]):
                if a.dtype == torch.float64:   # tiles from the queue: sums in double, their order is not fixed
                    assert torch.allclose(a, b, rtol=1e-12, atol=1e-12 * float(b.abs().max()))
                else:
                    assert torch.equal(a, b), CALLS[i]


def _wanted():
    want = []
    for i in range(len(CALLS)):
        call, out = _make(i, 0)
        call(None)
        torch.cuda.synchronize()
        want.append([x.clone() for x in out])
    return want


def _check(made, want):
    for i, call, out in made:
        for a, b in zip(out, want[i]):
            if a.dtype == torch.float64:   # tiles from the queue: sums in double, their order is not fixed
                assert torch.allclose(a, b, rtol=1e-12, atol=1e-12 * float(b.abs().max()))
            else:
                assert torch.equal(a, b), CALLS[i]


class _Delay:
    """Some 50 ms of ordinary work on a stream, so that what follows it stays in flight while the host goes on."""
    def __init__(self):
        self.a = torch.randn(8192, 8192, device="cuda")
        self.out = [torch.empty_like(self.a) for _ in range(3)]

    def on(self, stream, k):
        ended = torch.cuda.Event()
        with torch.cuda.stream(stream):
            for _ in range(5):
                torch.mm(self.a, self.a, out=self.out[k])
            ended.record(stream)
        return ended


def test_slots_run_out_on_three_streams():
    want, delay = _wanted(), _Delay()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for repeat in range(4):
        order = np.random.default_rng(repeat).permutation(len(CALLS))
        made = [(int(i), *_make(int(i), 0)) for _ in range(3) for i in order]   # three rounds without a synchronisation
        torch.cuda.synchronize()
        ended = [delay.on(s, k) for k, s in enumerate(streams)]
        for k, (i, call, out) in enumerate(made):
            call(streams[(k + repeat) % 3])
            if k == 7:   # so many calls at the least are in flight, and every slot there is with them
                assert not any(e.query() for e in ended)
        # the ninth that takes a slot has waited for the first one's
        assert ended[repeat % 3].query()
        torch.cuda.synchronize()
        _check(made, want)


def test_slots_run_out_from_three_threads():
    want, delay = _wanted(), _Delay()
    streams = [torch.cuda.Stream() for _ in range(3)]
    made = [[(int(i), *_make(int(i), 0)) for i in np.random.default_rng(t).permutation(len(CALLS))] for t in range(3)]
    errors = []

    def work(t):
        try:
            torch.cuda.set_device(0)
            for i, call, out in made[t]:
                call(streams[t])
        except Exception as e:   # noqa: BLE001 (handed to the main thread)
            errors.append(e)

    torch.cuda.synchronize()
    ended = [delay.on(s, k) for k, s in enumerate(streams)]
    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert any(e.query() for e in ended)   # 45 calls, eight slots
    torch.cuda.synchronize()
    for t in range(3):
        _check(made[t], want)
