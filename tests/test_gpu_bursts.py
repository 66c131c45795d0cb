"""Updates whose results are written in bursts: the lengths where the tiles of a workgroup are none, one, a remainder, more than its LDS
holds; against the kernels with a fixed assignment, whose arithmetic is the same to the bit, and 64 bits."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star
from gpu_util import rand_stream

pytestmark = pytest.mark.gpu

HP = dict(lr=0.1, momentum_coef=0.9, weight_decay=1e-4, wmode="stale")
GUARD = 64


def _guarded(n, offset, gen, dtype=torch.float32, std=0.02):
    """A buffer of n elements from place `offset` on inside a larger one, which is returned as well."""
    whole = (torch.randn(n + offset + GUARD, generator=gen, device="cuda") * std).to(dtype)
    return whole, whole[offset:offset + n]


def _call(W, P, dtype, offset, out, threshold, U=12, norms=None):
    gen = torch.Generator(device="cuda").manual_seed(W + P)
    rows = [_guarded(P, offset, gen, torch.float32 if dtype == "f32" else torch.bfloat16, 1e-2)[1] for _ in range(W)]
    (pw, p), (vw, v) = _guarded(P, offset, gen), _guarded(P, offset, gen, std=1e-2)
    start = p.double().clone(), v.double().clone()
    offs, mem, st = rand_stream(np.random.default_rng(W), W, U, stale=4)
    us = star.UpdateStream(offs, mem, st)
    whole = [pw, vw]
    if out is None:
        star.star_group_update(p, v, rows, us, norms_out=norms, queue_threshold=threshold, **HP)
    else:
        sw, s = _guarded(P, offset, gen, out)
        whole.append(sw)
        star.star_group_update_publish(p, v, rows, us, s, norms_out=norms, queue_threshold=threshold, **HP)
    torch.cuda.synchronize()
    return whole, (p, v, rows, us, start)


# threshold None: what the library chooses for the length (each the shortest of its row count); 1: the queue whatever the length
@pytest.mark.parametrize("W,dtype,P,threshold,offset,out", [
    (10, "f32", 1, 1, 0, None), (12, "f32", 1023, 1, 0, torch.bfloat16), (16, "f32", 1025, 1, 3, None), (32, "f32", 256 * 1024 + 5, 1, 0, None),
    (11, "f32", 600_001, 1, 1, torch.float32), (20, "f32", 511 * 1024, 1, 0, None), (28, "f32", 511 * 1024 + 1, 1, 7, torch.bfloat16),
    (10, "f32", 6_000_003, 1, 0, torch.float32), (24, "f32", (7 << 19) + 1, None, 0, None), (16, "f32", 7 << 20, None, 5, None),
    (12, "f32", 11_000_001, None, 0, None), (10, "f32", 13_000_000, None, 2, torch.bfloat16),
    (12, "bf16", 5, 1, 0, None), (16, "bf16", 70_001, 1, 1, torch.bfloat16), (32, "bf16", 512 * 1024 + 3, 1, 0, None),
    (24, "bf16", 16_000_003, None, 3, torch.bfloat16), (16, "bf16", 21_000_001, None, 0, None), (20, "bf16", 6_000_513, 1, 0, torch.float32),
    (13, "bf16", 26_000_003, None, 6, None)])
def test_update_in_bursts(W, dtype, P, threshold, offset, out):
    us = _call(W, 1, dtype, 0, None, 1)[1][3]
    choice = dict(lr=0.1, momentum_coef=0.9, wmode="stale")
    assert star.star_plan_choice(P, W, dtype, us, queue_threshold=threshold, **choice)["queue_order"] == 1
    assert star.star_plan_choice(P, W, dtype, us, queue_threshold=1 << 62, **choice)["queue_order"] == 0
    got, (p, v, rows, us, (p0, v0)) = _call(W, P, dtype, offset, out, threshold)
    fixed = _call(W, P, dtype, offset, out, 1 << 62)[0]
    assert all(_same_bits(a, b) for a, b in zip(got, fixed))   # whole buffers: nothing beside the shard is written either
    M, B = star.star_plan_affine(W, us, **HP)
    ep, ev = M[0, 0] * p0 + M[0, 1] * v0, M[1, 0] * p0 + M[1, 1] * v0
    for w in range(W):
        ep.add_(rows[w].double(), alpha=float(B[0, w]))
        ev.add_(rows[w].double(), alpha=float(B[1, w]))
    # a chain of W + 2 fp32 multiply-adds of terms of the result's size
    for x, e in ((p, ep), (v, ev)):
        assert float(((x.double() - e).abs() / (e.abs() + e.square().mean().sqrt())).max()) <= 3e-6


def _same_bits(a, b):
    as_int = torch.int16 if a.dtype == torch.bfloat16 else torch.int32
    return torch.equal(a.view(as_int), b.view(as_int))


# threshold None: the shortest shards of a row count and, with up to 11 bf16 rows, the longest
@pytest.mark.parametrize("W,dtype,P,threshold,offset,out", [
    (14, "f32", 4099, 1, 0, None), (16, "f32", 256 * 1024 + 5, 1, 1, torch.bfloat16), (20, "f32", 511 * 1024 + 1, 1, 0, torch.float32),
    (18, "f32", 5_000_001, 1, 3, None), (16, "f32", 16 << 20, None, 5, None), (15, "f32", (16 << 20) + 1025, None, 0, torch.bfloat16),
    (12, "bf16", 5001, 1, 0, None), (16, "bf16", 5_000_003, None, 1, torch.bfloat16), (7, "bf16", 5_000_003, None, 0, None),
    (11, "bf16", 12 << 20, None, 0, torch.float32), (13, "bf16", 15_000_003, None, 6, None), (24, "bf16", 17_000_001, None, 0, None),
    (32, "bf16", 512 * 1024 + 3, 1, 2, None), (28, "bf16", 3_000_513, 1, 0, torch.float32)])
def test_update_with_norms_in_bursts(W, dtype, P, threshold, offset, out):
    n, m = torch.full((12,), -1.0, device="cuda"), torch.full((12,), -1.0, device="cuda")
    got, (p, v, rows, us, _) = _call(W, P, dtype, offset, out, threshold, norms=n)
    choice = star.star_plan_choice(P, W, dtype, us, lr=0.1, momentum_coef=0.9, wmode="stale", want_norms=True)
    assert choice["kernel"] == star.KERNEL_AFFINE_MFMA
    fixed = _call(W, P, dtype, offset, out, 1 << 62, norms=m)[0]
    assert all(_same_bits(a, b) for a, b in zip(got, fixed))
    # the same sums tile by tile, in double from there on: only their order differs
    assert float(((n - m) / m).abs().max()) <= 2.0 ** -23
    r = torch.stack([x.double() for x in rows])
    C = torch.zeros(us.U, W, dtype=torch.float64)
    for u in range(us.U):
        for k in range(us.offsets[u], us.offsets[u + 1]):
            C[u, us.members[k]] = 1.0 / ((us.offsets[u + 1] - us.offsets[u]) * (1.0 + us.staleness[k]))
    want = sum((C.cuda() @ part).square().sum(1) for part in r.split(1 << 22, dim=1)).sqrt()
    assert float(((n.double() - want) / want).abs().max()) <= 1e-6   # (rows that are not anti-correlated, see star.h)


# threshold None: the shortest shard of a row count; 1: the queue whatever the length
@pytest.mark.parametrize("W,dtype,P,threshold,offset,out", [
    (6, "f32", 1, 1, 0, "f32"), (8, "f32", 1027, 1, 1, "f32"), (16, "f32", 511 * 1024 + 3, 1, 0, "f32"), (7, "f32", 11_000_003, 1, 3, "f32"),
    (6, "f32", 14 << 20, None, 0, "f32"), (8, "f32", (8 << 20) + 5, None, 5, "f32"), (11, "f32", 7_340_035, None, 0, "f32"),
    (12, "f32", 3 << 20, None, 2, "f32"), (24, "f32", 3_200_001, None, 0, "f32"), (12, "f32", 6001, 1, 1, "bf16"),
    (13, "f32", (14 << 20) + 7, None, 0, "bf16"), (20, "f32", 4 << 20, None, 3, "bf16"), (12, "bf16", 5, 1, 0, "f32"),
    (12, "bf16", (16 << 20) + 1, None, 1, "f32"), (14, "bf16", 8 << 20, None, 0, "f32"), (32, "bf16", 7_900_001, None, 0, "f32"),
    (28, "bf16", 262_147, 1, 1, "bf16"), (32, "bf16", 7_900_001, None, 5, "bf16")])
def test_aggregate_in_bursts(W, dtype, P, threshold, offset, out):
    gen = torch.Generator(device="cuda").manual_seed(W + P)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}
    rows = [_guarded(P, offset, gen, dt[dtype], 1e-2)[1] for _ in range(W)]
    members = np.random.default_rng(W).permutation(W)[:max(1, W - 2)].astype(np.int32)   # two rows that are in no group
    members = np.concatenate([members, np.arange(W, dtype=np.int32)])
    us = [star.UpdateStream(np.array([0, n], np.int32), m, np.arange(n, dtype=np.int32) % 3)
          for n, m in ((len(members) - W, members[:-W]), (W, members[-W:]))]
    for stream in us:
        got = []
        for t in (threshold, 1 << 62):
            gen.manual_seed(7)
            whole, o = _guarded(P, offset, gen, dt[out])
            star.star_group_reduce([o], rows, stream, wmode="stale", queue_threshold=t)
            torch.cuda.synchronize()
            got.append(whole)
        assert _same_bits(*got)
        y = len(stream.members)
        want = sum(rows[int(w)].double() / (y * (1.0 + int(s))) for w, s in zip(stream.members, stream.staleness))
        have = got[0][offset:offset + P].double()
        # a chain of W fp32 multiply-adds, and half a unit of the last place of a bf16 result
        bound = 3e-6 if out == "f32" else 2.0 ** -8
        assert float(((have - want).abs() / (want.abs() + want.square().mean().sqrt())).max()) <= bound


@pytest.mark.parametrize("W,P", [(12, 6001), (16, 600_013)])
@pytest.mark.parametrize("step", [1, 3])
def test_bursts_of_buffers_off_by_different_amounts(W, P, step):
    """Rows, state, copy and aggregate each off by their own number of elements, so that no advance aligns them all: the bursts store 8 and 16
    bytes at places that are 4 (fp32) or 2 (bf16) byte aligned, and nothing beside the shard."""
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}
    us = star.UpdateStream(*rand_stream(np.random.default_rng(W), W, 5, stale=4))
    one = star.UpdateStream([0, W], np.arange(W, dtype=np.int32))
    for dtype in ("f32", "bf16"):
        for out in ("f32", "bf16"):
            got = []
            for threshold in (1, 1 << 62):
                gen = torch.Generator(device="cuda").manual_seed(W + P)
                rows = [_guarded(P, 1 + step * w, gen, dt[dtype], 1e-2)[1] for w in range(W)]
                (pw, p), (vw, v) = _guarded(P, 2, gen), _guarded(P, 5, gen, std=1e-2)
                (sw, s), (ow, o) = _guarded(P, 3, gen, dt[out]), _guarded(P, 7, gen, dt[out])
                star.star_group_update_publish(p, v, rows, us, s, queue_threshold=threshold, **HP)
                n = torch.zeros(5, device="cuda")
                star.star_group_update_publish(p, v, rows, us, s, norms_out=n, queue_threshold=threshold, **HP)
                star.star_group_reduce([o], rows, one, queue_threshold=threshold)
                torch.cuda.synchronize()
                got.append((pw, vw, sw, ow))
            assert all(_same_bits(a, b) for a, b in zip(*got)), (dtype, out)


def _norms64(W, rows, us):
    r = torch.stack([x.double() for x in rows])
    C = torch.zeros(us.U, W, dtype=torch.float64)
    for u in range(us.U):
        for k in range(us.offsets[u], us.offsets[u + 1]):
            C[u, us.members[k]] = 1.0 / ((us.offsets[u + 1] - us.offsets[u]) * (1.0 + us.staleness[k]))
    return sum((C.cuda() @ part).square().sum(1) for part in r.split(1 << 22, dim=1)).sqrt()


# 8 and 9 fp32 rows on long shards: one workgroup per unit that writes as it goes; the shortest such shard, the one below, remainders
@pytest.mark.parametrize("W,P,offset,out", [(8, 16 << 20, 0, None), (9, (16 << 20) - 1024, 0, None), (9, (16 << 20) + 1, 0, torch.bfloat16),
                                            (9, (17 << 20) + 1023, 3, None), (8, (16 << 20) + 517, 1, torch.float32)])
def test_update_with_norms_by_one_workgroup_a_unit(W, P, offset, out):
    n = torch.full((12,), -1.0, device="cuda")
    got, (p, v, rows, us, _) = _call(W, P, "f32", offset, out, None, norms=n)
    choice = star.star_plan_choice(P, W, "f32", us, lr=0.1, momentum_coef=0.9, wmode="stale", want_norms=True)
    assert choice["kernel"] == star.KERNEL_AFFINE_MFMA
    assert star.star_plan_bursts(P, W, "f32", us, lr=0.1, momentum_coef=0.9, wmode="stale", want_norms=True) == 0
    plain = _call(W, P, "f32", offset, out, 1 << 62)[0]   # without norms: the same arithmetic in another kernel
    assert all(_same_bits(a, b) for a, b in zip(got, plain))
    want = _norms64(W, rows, us)
    assert float(((n.double() - want) / want).abs().max()) <= 1e-6


# The same just above a limit at an odd place: of P elements, what is left behind an advance of up to 63 to whole cache lines still writes in
# bursts (an aggregation's length counts behind the advance, an update's before it).
@pytest.mark.parametrize("what,W,dtype,P,offset,out", [
    ("update", 16, "f32", (7 << 20) + 69, 5, None), ("norms", 16, "f32", (16 << 20) + 69, 5, None), ("reduce", 8, "f32", (8 << 20) + 69, 5, "f32"),
    ("reduce", 12, "f32", (3 << 20) + 64, 2, "f32"), ("reduce", 20, "f32", (4 << 20) + 64, 3, "bf16"), ("reduce", 12, "bf16", (16 << 20) + 65, 1, "f32")])
def test_bursts_just_above_a_limit_at_an_odd_place(what, W, dtype, P, offset, out):
    one, us = star.UpdateStream([0, W], np.arange(W, dtype=np.int32)), star.UpdateStream(*rand_stream(np.random.default_rng(W), W, 12, stale=4))
    choice = dict(lr=0.1, momentum_coef=0.9, wmode="stale", want_norms=what == "norms")
    tiles = ([star.star_plan_reduce_bursts(n, W, out, dtype, one, wmode="stale") for n in (P - 63, P - 70)] if what == "reduce"
             else [star.star_plan_bursts(n, W, dtype, us, **choice) for n in (P - 63, P - 70)])
    assert tiles[0] > 0 and tiles[1] == 0
    {"update": test_update_in_bursts, "norms": test_update_with_norms_in_bursts, "reduce": test_aggregate_in_bursts}[what](
        W, dtype, P, None, offset, out)


# What the tests above compare with the fixed assignment is written in bursts (whole cache lines: without an advance).
def test_cases_above_are_written_in_bursts():
    def cases_of(test):
        return [m for m in test.pytestmark if m.name == "parametrize"][0].args[1]
    for norms, test in ((False, test_update_in_bursts), (True, test_update_with_norms_in_bursts)):
        for W, dtype, P, threshold, _, _ in cases_of(test):
            us = star.UpdateStream(*rand_stream(np.random.default_rng(W), W, 12, stale=4))
            choice = dict(lr=0.1, momentum_coef=0.9, wmode="stale", want_norms=norms)
            assert star.star_plan_bursts(P, W, dtype, us, queue_threshold=threshold, **choice) > 0
            assert star.star_plan_bursts(P, W, dtype, us, queue_threshold=1 << 62, **choice) == 0
    for W, dtype, P, threshold, _, out in cases_of(test_aggregate_in_bursts):
        one = star.UpdateStream([0, W], np.arange(W, dtype=np.int32))
        assert star.star_plan_reduce_bursts(P, W, out, dtype, one, wmode="stale", queue_threshold=threshold) > 0
        assert star.star_plan_reduce_bursts(P, W, out, dtype, one, wmode="stale", queue_threshold=1 << 62) == 0


def test_bursts_beside_work_that_holds_units():
    """A launch that writes in bursts takes the whole LDS of every unit; here other kernels hold some or all of it when it starts, on a stream
    of their own: matrix products on the whole device, one on few units for long, a softmax of many short workgroups."""
    W, P = 16, 17_000_003
    gen = torch.Generator(device="cuda").manual_seed(1)
    rows = [torch.randn(P, generator=gen, device="cuda") * 1e-2 for _ in range(W)]
    p0, v0 = (torch.randn(P, generator=gen, device="cuda") for _ in range(2))
    us = star.UpdateStream(*rand_stream(np.random.default_rng(W), W, 12, stale=4))
    one = star.UpdateStream([0, W], np.arange(W, dtype=np.int32))
    assert star.star_plan_bursts(P, W, "f32", us, **HP) > 0 and star.star_plan_bursts(P, W, "f32", us, want_norms=True, **HP) > 0
    assert star.star_plan_reduce_bursts(P, W, "f32", "f32", one) > 0
    wide, small = torch.randn(4096, 4096, device="cuda"), torch.randn(256, 1 << 18, device="cuda", dtype=torch.bfloat16)
    tall, many = small.t().contiguous(), torch.randn(16384, 4096, device="cuda")

    def calls(stream):
        p, v, n, o = p0.clone(), v0.clone(), torch.zeros(12, device="cuda"), torch.empty(P, device="cuda")
        torch.cuda.current_stream().synchronize()
        star.star_group_update(p, v, rows, us, stream=stream, **HP)
        star.star_group_update(p, v, rows, us, norms_out=n, stream=stream, **HP)
        star.star_group_reduce([o], rows, one, stream=stream)
        return p, v, o, n

    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    want = calls(mine)
    torch.cuda.synchronize()
    for work in (lambda: torch.mm(wide, wide), lambda: torch.mm(small, tall), lambda: torch.softmax(many, 1)):
        with torch.cuda.stream(other):
            for _ in range(20):
                work()
        got = calls(mine)
        torch.cuda.synchronize()
        assert all(_same_bits(a, b) for a, b in zip(got[:3], want[:3]))
        assert float(((got[3] - want[3]) / want[3]).abs().max()) <= 2.0 ** -23   # (tiles from the queue: the order of the sums)
