"""Performance cases of the group-synchronous update: what a parameter server asks of the library, call by call.

Every case is one call of a public entry point on one shard.  ``listed()`` names twelve of them, ``draw`` gives
more from the same ranges, ``prepare`` makes the buffers a server has in hand before the call (parameters, momentum,
the workers' gradient rows marshalled once, the queued update stream), ``run`` is the call, ``exact`` the definition
evaluated literally in 64 bits.

Fields of a case
  op        "update", "publish" (update that also writes the send copy), "norms", "reduce" (aggregation), "gram"
  P, W      elements of the shard, workers;  dtype  "f32" | "bf16" gradient rows
  U         queued updates (groups, for the aggregation);  lo, hi  group sizes, uniform in lo..hi; ``alternate``:
            even updates take all W workers, odd ones ``lo``;  cycle: sizes cycle lo, 2 lo, .. hi
  wmode     "mean" | "stale" (staleness 0..stale) | "explicit" (coefficients of both signs)
  norms     per-group norms wanted;  direct  the caller asks for norms from direct sums
  out       dtype of the published copy or of the aggregated rows
  offset    first element of the shard inside larger flat buffers: a server that owns the elements from an odd
            index on is handed pointers that are not 16-byte aligned
  noalloc   the entry point that allocates nothing (serving loop on preallocated memory)
  gstd, lr, mu, wd, heavy   spread of the gradients, hyper-parameters, one worker's row times ten
"""
import math

import numpy as np
import torch

import paper_2512_09685_amd as star

_BASE = {"op": "update", "dtype": "f32", "U": 1, "lo": 1, "hi": 1, "alternate": False, "cycle": False, "wmode": "mean",
         "stale": 0, "norms": False, "direct": False, "out": "f32", "offset": 0, "noalloc": False, "gstd": 1e-3,
         "lr": 0.01, "mu": 0.9, "wd": 1e-4, "heavy": False}


def _case(**kw):
    return dict(_BASE, **kw)


def listed():
    return [
        # the smallest job: four workers, ten queued updates on a one-million-element shard; a call is one launch
        _case(name="tiny", P=1_048_576, W=4, U=10, lo=2, hi=2, gstd=1e-2, lr=0.1),
        # a small model's shard of odd length with the gradient-norm signal: launches and their gaps
        _case(name="small_norms", P=300_007, W=8, U=16, lo=1, hi=8, wmode="stale", stale=4, norms=True, lr=0.1),
        # an image model's shard, static x-order of changing x, no norms
        _case(name="resnet50", P=25_557_032, W=8, U=64, lo=2, hi=8, cycle=True, lr=0.1, wd=5e-5),
        # a language model's shard, dynamic x-order with staleness weights and the norm signal
        _case(name="bert_base", P=110_000_000, W=16, U=64, lo=1, hi=16, wmode="stale", stale=4, norms=True, heavy=True),
        # 32 workers that report in bf16, full groups alternating with groups of four
        _case(name="vgg16", P=138_357_544, W=32, dtype="bf16", U=128, lo=4, hi=32, alternate=True, wd=0.0),
        # the largest shard: one of its streamed batches of 64 updates, bf16 reports, norms
        _case(name="bert_large", P=340_000_000, W=16, dtype="bf16", U=64, lo=2, hi=16, wmode="stale", stale=8, norms=True,
              gstd=5e-4),
        # ASGD: every report applied on arrival, from the serving loop's entry point, its norm returned
        _case(name="report", P=25_557_032, W=8, U=1, norms=True, noalloc=True, lr=0.1),
        # one of three servers that share a model by elements: its slice starts at an odd element of the flat buffers,
        # and the updated slice goes back to the workers in bf16
        _case(name="slice_publish", op="publish", P=46_119_181, W=8, dtype="bf16", U=32, lo=1, hi=8, wmode="stale", stale=4,
              norms=True, out="bf16", offset=1),
        # 24 workers that report in fp32, norms over a long stream
        _case(name="wide_norms", P=25_557_032, W=24, U=48, lo=1, hi=24, wmode="stale", stale=4, norms=True),
        # a parent of the all-reduce ring or a node of the communication tree: the mean of eight reports, no update
        _case(name="aggregate", op="reduce", P=25_557_032, W=8, lo=8, hi=8),
        # noise-scale estimate: Gram matrix of sixteen bf16 reports
        _case(name="gram", op="gram", P=25_557_032, W=16, dtype="bf16"),
        # the norm signal alone where reports may be anti-correlated: the caller asks for direct sums
        _case(name="direct_norms", op="norms", P=25_557_032, W=8, U=32, lo=1, hi=8, norms=True, direct=True),
    ]


def draw(rng):
    """One more call of the same kinds.  Shards from 200 thousand to 150 million elements, 1 to 32 workers, 1 to 128
    updates; a quarter of the shards start at an odd place; lengths shortened where the call would cost more than the
    largest listed one."""
    op = rng.choice(["update"] * 6 + ["publish", "norms", "norms", "reduce", "reduce", "gram"])
    W = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 8, 10, 12, 13, 16, 16, 17, 20, 22, 24, 27, 32, 32])
    dtype = rng.choice(["f32", "bf16"])
    P = int(math.exp(rng.uniform(math.log(2e5), math.log(1.5e8))))
    U = 1 if rng.random() < 0.15 else int(round(math.exp(rng.uniform(math.log(2), math.log(128)))))
    c = dict(op=op, W=W, dtype=dtype, wmode="mean")
    if op == "gram":
        c.update(U=1, lo=W, hi=W, norms=False)
    else:
        if op == "reduce":
            U = rng.choice([1, 1, 1, 2, 4, 8])
        c["hi"] = rng.randint(1, W)
        c["lo"] = rng.randint(1, c["hi"])
        c["U"] = U
        c["norms"] = op == "norms" or rng.random() < (0.25 if op == "reduce" else 0.6)
        c["wmode"] = rng.choice(["mean", "stale", "stale"])
        if c["wmode"] == "stale":
            c["stale"] = rng.randint(1, 8)
        if op in ("update", "publish", "norms"):
            x = rng.random()
            if x < 0.08:
                c["wmode"] = "explicit"
            elif x < 0.16 and c["norms"]:
                c["direct"] = True
        if op == "update" and not c.get("direct") and rng.random() < 0.15:
            c["noalloc"] = True
        if op in ("publish", "reduce"):
            c["out"] = rng.choice(["f32", "bf16"])
    c["lr"] = rng.choice([0.1, 0.01])
    c["offset"] = rng.choice([0, 0, 0, rng.randint(1, 7)])
    c["P"] = P
    c = _case(**c)
    most = 8e9 if not c["offset"] else 4e9
    c["P"] = min(P, int(most / (work(c)["bytes"] / P)))
    if c["direct"] or c["wmode"] == "explicit":   # these walk the stream element by element
        c["P"] = min(c["P"], int(8e9 / (c["U"] * (0.5 * (c["lo"] + c["hi"]) + 4))))
    return c


def _rows_used(case):
    if case["op"] == "gram":
        return case["W"]
    if case["alternate"]:
        return case["W"]
    mean = 0.5 * (case["lo"] + case["hi"])
    return case["W"] * (1.0 - (1.0 - mean / case["W"]) ** case["U"])   # expected: groups are drawn


def work(case):
    P, rows = case["P"], _rows_used(case)
    nbytes = rows * (4 if case["dtype"] == "f32" else 2)
    out = 4 if case["out"] == "f32" else 2
    flops = 0.0
    if case["op"] in ("update", "publish"):
        nbytes += 16   # params and momentum, read and written
        flops += 2 * (2 * rows + 4)
    if case["op"] == "publish":
        nbytes += out
    if case["op"] == "reduce":
        nbytes += out * case["U"]
        flops += 2 * 0.5 * (case["lo"] + case["hi"]) * case["U"]
    if case["op"] == "gram":
        flops += rows * (rows + 1)
    elif case["norms"]:
        flops += min(rows * (rows + 1), 2 * case["U"] * (0.5 * (case["lo"] + case["hi"]) + 1))
    return {"bytes": nbytes * P, "flops": flops * P}


def tolerance(case):
    # fp32 sums of at most a few dozen terms (state and aggregates: up to 1.1e-7 from the 64-bit result; norms and Gram matrix
    # the same).  A value rounded to bf16 flips to its neighbour, 2^-8 away, where the fp32 sums before the rounding
    # differ across a tie: about one in 1e4 values.
    if case["op"] in ("publish", "reduce") and case["out"] == "bf16":
        return {"rel": 2e-4, "max": 1.6e-2}
    return {"rel": 5e-7, "max": 5e-6}


# ------------------------------------------------------------------------------------------------ inputs
def _stream(case, seed):
    r = np.random.default_rng([int(seed), 2])
    W, U = case["W"], case["U"]
    sizes = []
    cyc = []
    y = case["lo"]
    while y < case["hi"]:
        cyc.append(y)
        y *= 2
    cyc.append(case["hi"])
    for u in range(U):
        if case["alternate"]:
            sizes.append(W if u % 2 == 0 else case["lo"])
        elif case["cycle"]:
            sizes.append(cyc[u % len(cyc)])
        else:
            sizes.append(int(r.integers(case["lo"], case["hi"] + 1)))
    offsets = np.zeros(U + 1, np.int32)
    offsets[1:] = np.cumsum(sizes)
    members = np.concatenate([r.permutation(W)[:y] for y in sizes]).astype(np.int32)
    staleness = coeff = None
    if case["wmode"] == "stale":
        staleness = r.integers(0, case["stale"] + 1, size=len(members)).astype(np.int32)
    if case["wmode"] == "explicit":
        coeff = (r.standard_normal(len(members)) / np.repeat(sizes, sizes)).astype(np.float32)
    return offsets, members, staleness, coeff


def _normal(case, gen, std, dtype):
    n = case["P"] + case["offset"]
    x = torch.randn(n, generator=gen, device="cuda", dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    return x.mul_(std)[case["offset"]:]


def _tensors(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    heavy = int(np.random.default_rng([int(seed), 5]).integers(case["W"])) if case["heavy"] else -1
    rows = [_normal(case, gen, case["gstd"] * (10.0 if w == heavy else 1.0), case["dtype"]) for w in range(case["W"])]
    t = {"rows": rows}
    if case["op"] in ("update", "publish"):
        t["params"] = _normal(case, gen, 0.02, "f32")
        t["momentum"] = _normal(case, gen, case["gstd"], "f32")
    return t


def _empty(case, dtype):
    return torch.empty(case["P"] + case["offset"], device="cuda",
                       dtype=torch.float32 if dtype == "f32" else torch.bfloat16)[case["offset"]:]


def prepare(case, seed):
    s = dict(_tensors(case, seed), case=case)
    s["rows"] = star.GradRows(s["rows"])
    if case["op"] == "gram":
        s["gram"] = torch.empty(case["W"], case["W"], dtype=torch.float64, device="cuda")
        return s
    s["updates"] = star.UpdateStream(*_stream(case, seed))
    if case["norms"]:
        s["norms"] = torch.empty(case["U"], dtype=torch.float32, device="cuda")
    if case["op"] == "publish":
        s["send"] = _empty(case, case["out"])
    if case["op"] == "reduce":
        s["out"] = star.GradRows([_empty(case, case["out"]) for _ in range(case["U"])])
    return s


def run(s):
    c = s["case"]
    norms = s.get("norms")
    if c["op"] == "gram":
        star.star_group_gram(s["rows"], s["gram"])
        return s["gram"]
    if c["op"] == "norms":
        star.star_group_norms(s["rows"], s["updates"], norms, wmode=c["wmode"], direct_norms=c["direct"])
        return norms
    if c["op"] == "reduce":
        star.star_group_reduce(s["out"], s["rows"], s["updates"], wmode=c["wmode"], norms_out=norms)
        return {"out": list(s["out"]), "norms": norms}
    hp = dict(lr=c["lr"], momentum_coef=c["mu"], weight_decay=c["wd"], wmode=c["wmode"], norms_out=norms)
    if c["op"] == "publish":
        star.star_group_update_publish(s["params"], s["momentum"], s["rows"], s["updates"], s["send"],
                                       direct_norms=c["direct"], **hp)
    elif c["noalloc"]:
        star.star_group_update_noalloc(s["params"], s["momentum"], s["rows"], s["updates"], **hp)
    else:
        star.star_group_update(s["params"], s["momentum"], s["rows"], s["updates"], direct_norms=c["direct"], **hp)
    return {"params": s["params"], "momentum": s["momentum"], "norms": norms, "send": s.get("send")}


# ------------------------------------------------------------------------------------------------ the definition
def exact(case, seed):
    """The definition in 64 bits, element slice by element slice: for every update the weighted sum of its members,
    weight decay, momentum, step (the published copy and the aggregated rows before any rounding to bf16)."""
    t = _tensors(case, seed)
    P, W, U = case["P"], case["W"], case["U"]
    if case["op"] == "gram":
        gram = torch.zeros(W, W, dtype=torch.float64, device="cuda")
        for lo in range(0, P, 1 << 21):
            g = torch.stack([r[lo:lo + (1 << 21)].double() for r in t["rows"]])
            for a in range(W):
                gram[a] += (g * g[a]).sum(1)
        return gram
    offsets, members, staleness, coeff = _stream(case, seed)
    C = np.zeros((U, W))
    for u in range(U):
        y = int(offsets[u + 1] - offsets[u])
        for m in range(offsets[u], offsets[u + 1]):
            if coeff is not None:
                C[u, members[m]] = float(coeff[m])
            else:
                C[u, members[m]] = 1.0 / (y * (1.0 + (0 if staleness is None else float(staleness[m]))))
    lr, mu, wd = (float(np.float32(case[k])) for k in ("lr", "mu", "wd"))
    update = case["op"] in ("update", "publish")
    sums = [torch.zeros((), dtype=torch.float64, device="cuda") for _ in range(U)]
    if update:
        p_out, v_out = torch.empty(P, dtype=torch.float64, device="cuda"), torch.empty(P, dtype=torch.float64, device="cuda")
    if case["op"] == "reduce":
        out = [torch.empty(P, dtype=torch.float64, device="cuda") for _ in range(U)]
    for lo in range(0, P, 1 << 24):
        hi = min(P, lo + (1 << 24))
        g = [r[lo:hi].double() for r in t["rows"]]
        if update:
            p, v = t["params"][lo:hi].double(), t["momentum"][lo:hi].double()
        for u in range(U):
            gbar = torch.zeros(hi - lo, dtype=torch.float64, device="cuda")
            for w in range(W):
                if C[u, w] != 0.0:
                    gbar.add_(g[w], alpha=C[u, w])
            if case["norms"]:
                sums[u] += gbar.square().sum()
            if case["op"] == "reduce":
                out[u][lo:hi] = gbar
            if update:
                gbar.add_(p, alpha=wd)
                v.mul_(mu).add_(gbar)
                p.add_(v, alpha=-lr)
        if update:
            p_out[lo:hi], v_out[lo:hi] = p, v
    norms = torch.stack(sums).sqrt() if case["norms"] else None
    if case["op"] == "norms":
        return norms
    if case["op"] == "reduce":
        return {"out": out, "norms": norms}
    return {"params": p_out, "momentum": v_out, "norms": norms, "send": p_out if case["op"] == "publish" else None}
