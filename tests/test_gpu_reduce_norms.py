"""Aggregation with norms where the number of workgroups per compute unit changes (row count, groups, 4 and 16 Mi elements on 256
units), against a 64-bit evaluation on the device."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star
from gpu_util import opts, rand_stream, tile_order  # noqa: F401 (tile_order: autouse fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,dtype,U,P", [(5, "f32", 3, 4097), (7, "f32", 1, (4 << 20) - 1), (8, "f32", 1, (4 << 20) + 1025),
                                         (12, "f32", 2, (4 << 20) + 3), (9, "bf16", 1, (16 << 20) + 1), (10, "bf16", 1, 16 << 20),
                                         (13, "bf16", 3, 300001), (24, "bf16", 5, 5000), (20, "bf16", 6, 1024 * 1025), (28, "bf16", 7, 70001),
                                         (4, "f32", 1, (4 << 20) + 1), (16, "bf16", 6, (4 << 20) + 1), (24, "bf16", 4, (4 << 20) - 1),
                                         (16, "bf16", 7, 16 << 20), (28, "bf16", 8, (16 << 20) + 3)])
def test_reduce_with_norms(W, dtype, U, P):
    rng = np.random.default_rng(W * 100 + U)
    gen = torch.Generator(device="cuda").manual_seed(P)
    rows = [torch.randn(P, generator=gen, device="cuda", dtype=torch.float32 if dtype == "f32" else torch.bfloat16) for _ in range(W)]
    offs, mem, st = rand_stream(rng, W, U, stale=3)
    out = [torch.empty(P, device="cuda") for _ in range(U)]
    n = torch.full((U,), -1.0, device="cuda")
    star.star_group_reduce(out, rows, star.UpdateStream(offs, mem, st), wmode="stale", norms_out=n, **opts())
    torch.cuda.synchronize()
    for u in range(U):
        ids, s = mem[offs[u]:offs[u + 1]], st[offs[u]:offs[u + 1]]
        ref = sum(rows[w].double() / (len(ids) * (1.0 + float(x))) for w, x in zip(ids, s))
        # at most 28 fp32 multiply-adds with rounded coefficients: 29 half-ulps of the terms, far less on average
        assert float((out[u].double() - ref).abs().max()) <= 1e-6 * float(ref.abs().max())
        assert abs(float(n[u]) - float(ref.norm())) <= 5e-7 * float(ref.norm())
