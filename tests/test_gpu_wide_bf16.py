"""17 to 32 bf16 rows on the matrix cores, at the shard lengths where the workgroups per unit and the split of the tiles change
(4 Mi elements with an update on 256 compute units; norms alone: fewer tiles than workgroups, and one more), against the oracle."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star
from oracle import star_oracle as so
from gpu_util import opts, rand_rows, rand_stream, tile_order, to_dev_rows  # noqa: F401 (tile_order: autouse fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,P", [(17, 4097), (20, 255 * 1024 + 1), (24, 257 * 1024), (32, 256 * 1024 - 1)])
def test_norms_alone(W, P):
    rng = np.random.default_rng(W)
    rows = rand_rows(rng, W, P, "bf16")
    offs, mem, _ = rand_stream(rng, W, 20)
    n = torch.full((20,), -1.0, device="cuda")
    star.star_group_norms(to_dev_rows(rows), star.UpdateStream(offs, mem), n, **opts())
    ref = so.group_norms(rows, offs, mem)
    assert np.max(np.abs(n.cpu().numpy() - ref) / ref) <= 1e-6   # as every norm of non-negative weights


@pytest.mark.parametrize("W", [19, 20, 32])
@pytest.mark.parametrize("P", [4 << 20, (4 << 20) + 1025])
def test_update_around_the_limit(W, P):
    rng = np.random.default_rng(W + P)
    gen = torch.Generator(device="cuda").manual_seed(W)
    dev = [torch.randn(P, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(1e-2) for _ in range(W)]
    offs, mem, _ = rand_stream(rng, W, 12)
    us = star.UpdateStream(offs, mem)
    p0 = torch.randn(P, generator=gen, device="cuda") * 0.02
    p, v, n = p0.clone(), torch.zeros(P, device="cuda"), torch.full((12,), -1.0, device="cuda")
    star.star_group_update(p, v, dev, us, norms_out=n, lr=0.1, momentum_coef=0.9, weight_decay=1e-4, **opts())
    torch.cuda.synchronize()
    # the state on a slice at each end and one across the middle, the norms over the whole shard
    G = [r.double() for r in dev]
    for u in range(12):
        ids = mem[offs[u]:offs[u + 1]]
        gbar = sum(G[w] for w in ids) / len(ids)
        assert abs(float(n[u]) - float(gbar.norm())) <= 1e-6 * float(gbar.norm())
    for lo in (0, P // 2 - 700, P - 1500):
        cut = [r[lo:lo + 1500].cpu().view(torch.int16).numpy().view(np.uint16).copy() for r in dev]
        ep, ev, _ = so.group_update(p0[lo:lo + 1500].cpu().numpy(), np.zeros(1500, np.float32), cut, offs, mem, lr=0.1,
                                    momentum_coef=0.9, weight_decay=1e-4)
        assert so.max_rel_err(p[lo:lo + 1500].cpu().numpy(), ep) <= 1e-6
        assert so.max_rel_err(v[lo:lo + 1500].cpu().numpy(), ev) <= 3e-6
