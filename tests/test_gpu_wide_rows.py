"""17 to 32 fp32 rows on the matrix cores (row groups of four up to 24, 16x16 blocks beyond): Gram matrix and norms against
the oracle at the lengths where a tile, a wave or a chunk is cut, and a non-finite value that only its own groups may see."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star
from oracle import star_oracle as so
from gpu_util import opts, rand_rows, rand_stream, tile_order, to_dev_rows  # noqa: F401 (tile_order: autouse fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [17, 20, 21, 24, 25, 28, 29, 32])
@pytest.mark.parametrize("P,off", [(1024, 0), (1027, 1), (4 * 64 + 3, 0), (270001, 0)])
def test_gram_of_wide_fp32_rows(W, P, off):
    rng = np.random.default_rng(W * 31 + P)
    rows = rand_rows(rng, W, P + off, "f32")
    ref = so.gram([r[off:].copy() for r in rows])
    dev = [r[off:] for r in to_dev_rows(rows)]
    out = torch.full((W, W), -1.0, dtype=torch.float64, device="cuda")
    star.star_group_gram(dev, out, **opts())
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.array_equal(got, got.T)
    # up to 256 products are added in fp32 (each rounded to 2^-24 of the running sum) before the sums go on in double: a few
    # hundred elements make one such chain, whose roundings add up like sqrt(256) 2^-24 = 9.5e-7
    err = float(np.max(np.abs(got - ref) / np.sqrt(np.outer(np.diag(ref), np.diag(ref)))))
    print(f"gram W={W} P={P}+{off}: err {err:.3g}", flush=True)
    assert err <= 1e-6
    if P < 4096:
        return
    offs, mem, _ = rand_stream(rng, W, 40)
    us = star.UpdateStream(offs, mem)
    n = torch.full((40,), -1.0, device="cuda")
    star.star_group_norms(dev, us, n, **opts())
    ref_n = so.group_norms([r[off:].copy() for r in rows], offs, mem)
    assert np.max(np.abs(n.cpu().numpy() - ref_n) / ref_n) <= 1e-6
    dev[W - 1][P // 3] = float("nan")
    star.star_group_norms(dev, us, n, **opts())
    member = np.array([W - 1 in mem[offs[u]:offs[u + 1]] for u in range(40)])
    assert np.array_equal(~np.isfinite(n.cpu().numpy()), member)


@pytest.mark.parametrize("W", [17, 20, 24, 28])
@pytest.mark.parametrize("P", [300007, 1 << 20])
def test_gram_of_a_short_shard_is_the_same_every_run(W, P):
    """A short shard's tiles are split evenly, so the sums are formed in one order: the same bits in double on every run.  Every
    256 elements, a wave's share of a tile, have a scale of their own, so that an addition in double rounds and an order shows."""
    gen = torch.Generator(device="cuda").manual_seed(W)
    scale = torch.exp2(-torch.randint(0, 19, ((P + 255) // 256,), device="cuda", generator=gen).float()).repeat_interleave(256)[:P]
    rows = [torch.randn(P, device="cuda", generator=gen) * scale for _ in range(W)]
    first = None
    for _ in range(6):
        out = torch.empty(W, W, dtype=torch.float64, device="cuda")
        star.star_group_gram(rows, out, **opts())
        got = out.cpu().numpy()
        first = got if first is None else first
        assert np.array_equal(got, first)


@pytest.mark.parametrize("W,U,y", [(17, 4, 8), (20, 8, 10), (24, 5, 18), (32, 6, 12)])
def test_direct_norms_beside_the_update_of_wide_fp32_rows(W, U, y):
    """Direct norms on request in the pass of the collapsed update: state and norms against the oracle, with a pair of rows that
    almost cancel, whose norm the Gram matrix would lose."""
    rng = np.random.default_rng(W * 7 + U)
    P = 70003
    rows = rand_rows(rng, W, P, "f32")
    rows[1] = -rows[0] + (rng.standard_normal(P) * 1e-4).astype(np.float32)
    groups = [[0, 1]] + [list(rng.permutation(W)[:y]) for _ in range(U - 1)]
    offs = np.cumsum([0] + [len(g) for g in groups]).astype(np.int32)
    mem = np.concatenate(groups).astype(np.int32)
    us = star.UpdateStream(offs, mem)
    hp = dict(lr=0.1, momentum_coef=0.9, weight_decay=1e-4)
    used = len(set(mem.tolist()))
    c = star.star_plan_choice(P, W, "f32", us, want_norms=True, direct_norms=True, **hp)
    assert c["launches"] == 1 and c["kernel"] == star.KERNEL_SEQ and c["rows_used"] == used
    p0 = (rng.standard_normal(P) * 0.02).astype(np.float32)
    v0 = (rng.standard_normal(P) * 1e-2).astype(np.float32)
    ep, ev, en = so.group_update(p0, v0, rows, offs, mem, want_norms=True, **hp)
    p, v, n = torch.from_numpy(p0).cuda(), torch.from_numpy(v0).cuda(), torch.full((U,), -1.0, device="cuda")
    star.star_group_update(p, v, to_dev_rows(rows), us, norms_out=n, direct_norms=True, **opts(), **hp)
    torch.cuda.synchronize()
    assert np.max(np.abs(n.cpu().numpy() - en) / en) <= 1e-6
    assert so.max_rel_err(p.cpu().numpy(), ep) <= 1e-6 and so.max_rel_err(v.cpu().numpy(), ev) <= 1e-6
