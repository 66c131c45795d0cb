"""Direct norm sums without an update (the kernel behind direct_norms, signed coefficients and very short shards) against
the oracle: shard lengths around its tiles (4096, 2048 and 1024 elements by row count), every register form, streams
around the 240 updates of one launch, rows off by one element, and a non-finite value that only its own groups may see."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star
from oracle import star_oracle as so
from gpu_util import opts, rand_rows, rand_stream, tile_order, to_dev_rows  # noqa: F401 (tile_order: autouse fixture)

pytestmark = pytest.mark.gpu

# Norms against 64 bits: the coefficients and the result are rounded to fp32 (6e-8 each), a group sum of y terms carries
# at most y roundings of 6e-8 that average out over the elements, and four squares are added in fp32 (double beyond).
TOL = 3e-7


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("W,U,P,off", [(1, 1, 1, 0), (1, 2, 4096, 0), (3, 5, 16383, 0), (4, 7, 16385, 1), (5, 240, 8192, 0),
                                       (8, 32, 300007, 0), (9, 241, 6145, 3), (16, 3, 2 * 2048 * 300 + 5, 1), (17, 9, 5000, 0),
                                       (24, 2, 1024 * 41 - 1, 0), (32, 33, 70007, 1)])
def test_direct_norms(dtype, W, U, P, off):
    rng = np.random.default_rng(W * 1000 + U)
    rows = rand_rows(rng, W, P + off, dtype)
    offs, mem, st = rand_stream(rng, W, U, stale=3)
    dev = [r[off:] for r in to_dev_rows(rows)]
    ref = so.group_norms([r[off:].copy() for r in rows], offs, mem, staleness=st, wmode="stale")
    us = star.UpdateStream(offs, mem, st)
    n = torch.full((U,), -1.0, device="cuda")
    star.star_group_norms(dev, us, n, wmode="stale", direct_norms=True, **opts())
    torch.cuda.synchronize()
    err = float(np.max(np.abs(n.cpu().numpy() - ref) / ref))
    print(f"direct norms W={W} U={U} P={P}+{off} {dtype}: err {err:.3g}", flush=True)
    assert err <= TOL
    # the rows of one group cancel exactly: its norm is zero, not a rounding of the rows' size
    if W >= 2 and dtype == "f32":
        dev[1].copy_(-dev[0])
        z = torch.full((1,), -1.0, device="cuda")
        star.star_group_norms(dev, star.UpdateStream(np.array([0, 2], np.int32), np.array([0, 1], np.int32)), z,
                              direct_norms=True, **opts())
        assert float(z.cpu()) == 0.0
    # a non-finite value of one worker reaches the norms of its groups and no others
    dev[0][P // 2] = float("inf")
    star.star_group_norms(dev, us, n, wmode="stale", direct_norms=True, **opts())
    member = np.array([0 in mem[offs[u]:offs[u + 1]] for u in range(U)])
    assert np.array_equal(~np.isfinite(n.cpu().numpy()), member)


@pytest.mark.parametrize("W,U", [(1, 1), (4, 3), (8, 2), (16, 5), (32, 4)])
def test_direct_norms_of_large_elements(W, U):
    """Only four squares are ever added in fp32: elements of 9e18 (squares of 8.1e37, four of them 3.2e38) still have a finite norm."""
    P = 70001
    rows = [torch.full((P,), 9e18, device="cuda") for _ in range(W)]
    n = torch.full((U,), -1.0, device="cuda")
    us = star.UpdateStream(np.arange(U + 1, dtype=np.int32), np.arange(U, dtype=np.int32) % W)
    star.star_group_norms(rows, us, n, direct_norms=True, **opts())
    ref = float(np.float32(9e18)) * P ** 0.5
    # every partial sum is a whole multiple of one square: the roundings of the square's sum (3 of 6e-8, halved by the root) and the result's
    assert np.max(np.abs(n.cpu().numpy().astype(np.float64) - ref)) <= 2e-7 * ref


@pytest.mark.parametrize("W,U,P", [(1, 3, 1), (2, 9, 4096 * 3 + 1), (4, 13, 4096 * 200), (6, 61, 2048 * 20 - 3), (8, 33, 2048 * 64 + 5),
                                   (16, 32, 2048 * 128 + 1), (20, 8, 2048 * 127), (28, 12, 7), (32, 130, 2048 * 5 + 3)])
def test_direct_norms_shared_out_updates(W, U, P):
    """Shards of fewer tiles than compute units, where the updates are shared out over workgroups in fours: whole shares, short
    last shares, more shares than fours."""
    rng = np.random.default_rng(W + U)
    rows = rand_rows(rng, W, P, "f32")
    offs, mem, st = rand_stream(rng, W, U, stale=3)
    ref = so.group_norms(rows, offs, mem, staleness=st, wmode="stale")
    n = torch.full((U,), -1.0, device="cuda")
    star.star_group_norms(to_dev_rows(rows), star.UpdateStream(offs, mem, st), n, wmode="stale", direct_norms=True, **opts())
    err = float(np.max(np.abs(n.cpu().numpy() - ref) / ref))
    print(f"direct norms W={W} U={U} P={P}: err {err:.3g}", flush=True)
    # a shard of a few elements has nothing to average over: up to 33 roundings of the coefficients, products and sums
    assert err <= (TOL if P > 1000 else 1e-6)
