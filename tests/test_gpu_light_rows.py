"""Norms of few rows at the shard lengths where the number of workgroups of the vector-register Gram kernel changes (1 and 3 Mi
elements on 256 compute units; one tile and less than a tile per workgroup), against the oracle."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star
from oracle import star_oracle as so
from gpu_util import opts, rand_rows, rand_stream, tile_order, to_dev_rows  # noqa: F401 (tile_order: autouse fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,dtype,P", [(1, "f32", (1 << 20) + 1023), (1, "bf16", (1 << 20) - 1), (4, "f32", (3 << 20) + 1025),
                                       (2, "bf16", (3 << 20) - 3), (6, "f32", 5000), (8, "f32", (1 << 20) + 7)])
def test_norms_of_few_rows(W, dtype, P):
    rng = np.random.default_rng(W + P)
    rows = rand_rows(rng, W, P, dtype)
    offs, mem, st = rand_stream(rng, W, 12, stale=4)
    us = star.UpdateStream(offs, mem, st)
    dev = to_dev_rows(rows)
    hp = dict(lr=0.1, momentum_coef=0.9, weight_decay=1e-4, wmode="stale")
    p0 = (rng.standard_normal(P) * 0.02).astype(np.float32)
    ep, ev, en = so.group_update(p0, np.zeros_like(p0), rows, offs, mem, staleness=st, want_norms=True, **hp)
    p, v, n = torch.from_numpy(p0).cuda(), torch.zeros(P, device="cuda"), torch.full((12,), -1.0, device="cuda")
    star.star_group_update(p, v, dev, us, norms_out=n, **opts(), **hp)
    alone = torch.full((12,), -1.0, device="cuda")
    star.star_group_norms(dev, us, alone, wmode="stale", **opts())
    torch.cuda.synchronize()
    # norms: the rounding of the result (6e-8) and of the products' sums, which cancel between the members' roundings
    assert np.max(np.abs(n.cpu().numpy() - en) / en) <= 1e-6 and np.max(np.abs(alone.cpu().numpy() - en) / en) <= 1e-6
    assert so.max_rel_err(p.cpu().numpy(), ep) <= 1e-6 and so.max_rel_err(v.cpu().numpy(), ev) <= 3e-6


@pytest.mark.parametrize("W,P", [(1, (4 << 20) + 1023), (2, 4 << 20), (3, (16 << 20) + 5), (4, (4 << 20) - 1), (8, (4 << 20) + 1025)])
def test_one_report_with_its_norm(W, P):
    """A single update of fp32 rows where its workgroups per unit change (4 and 16 Mi elements), against 64 bits."""
    gen = torch.Generator(device="cuda").manual_seed(W)
    rows = [torch.randn(P, generator=gen, device="cuda") * 1e-2 for _ in range(W)]
    p0, v0 = torch.randn(P, generator=gen, device="cuda") * 0.02, torch.randn(P, generator=gen, device="cuda") * 1e-2
    us = star.UpdateStream(np.array([0, W], np.int32), np.arange(W, dtype=np.int32))
    p, v, n = p0.clone(), v0.clone(), torch.full((1,), -1.0, device="cuda")
    star.star_group_update(p, v, rows, us, norms_out=n, lr=0.1, momentum_coef=0.9, weight_decay=1e-4, **opts())
    torch.cuda.synchronize()
    gbar = sum(r.double() for r in rows) / W
    lr, mu, wd = (float(np.float32(x)) for x in (0.1, 0.9, 1e-4))
    ev = mu * v0.double() + gbar + wd * p0.double()
    ep = p0.double() - lr * ev
    # up to eleven fp32 roundings of terms of the result's size
    assert abs(float(n) - float(gbar.norm())) <= 5e-7 * float(gbar.norm())
    for got, ref in ((p, ep), (v, ev)):
        assert float(((got.double() - ref).abs() / (ref.abs() + ref.square().mean().sqrt())).max()) <= 1e-6
