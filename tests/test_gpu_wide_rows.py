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
