"""Direct norm sums on the matrix cores (norm_mma_kernel) at the edges of its tiles, blocks and launches: rows that are no
multiple of four, updates around 16 and beyond one workgroup's 64, shards that end inside a lane's load, odd starts, and rows
with infinities and NaN, which a dense product would spread over groups they are no members of."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star

pytestmark = pytest.mark.gpu

MI = 1 << 20
SHAPES = [(3, 64, MI + 5, 0), (4, 48, MI + 1, 3), (5, 17, 2 * MI - 1, 0), (8, 16, MI, 1), (8, 240, MI + 4095, 0),
          (13, 33, MI + 2047, 7), (16, 65, MI + 7, 0), (20, 32, MI + 3, 2), (24, 64, MI + 63, 0), (32, 16, MI + 1025, 5),
          (32, 128, MI + 2, 0), (8, 32, (1 << 17) + 1, 5), (16, 48, (1 << 19) + 3, 63)]


def _call(W, U, P, offset, dtype, spoil=()):
    rng = np.random.default_rng([W, U, P])
    sizes = rng.integers(max(1, W // 2), W + 1, size=U)
    sizes[0] = 1
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    members = np.concatenate([[W - 1]] + [rng.permutation(W)[:y] for y in sizes[1:]]).astype(np.int32)
    C = torch.zeros(U, W, dtype=torch.float64, device="cuda")
    for u in range(U):
        C[u, members[offs[u]:offs[u + 1]]] = 1.0 / sizes[u]
    gen = torch.Generator(device="cuda").manual_seed(W * 1000 + U)
    rows = [(torch.randn(P + offset, generator=gen, device="cuda") * 1e-3).to(dtype)[offset:] for _ in range(W)]
    for w, j, x in spoil:
        rows[w][j] = x
    out = torch.full((U,), -1.0, device="cuda")
    star.star_group_norms(star.GradRows(rows), star.UpdateStream(offs, members), out, direct_norms=True)
    return out, C, rows


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("W,U,P,offset", SHAPES)
def test_direct_norms(W, U, P, offset, dtype):
    out, C, rows = _call(W, U, P, offset, dtype)
    sums = torch.zeros(U, dtype=torch.float64, device="cuda")
    for lo in range(0, P, MI // 4):
        g = torch.stack([r[lo:lo + MI // 4].double() for r in rows])
        sums += (C @ g).square().sum(1)
    # W roundings in a sum of W products, four squares, the root and its rounding
    torch.testing.assert_close(out.double(), sums.sqrt(), rtol=(W + 6) * 2.0 ** -24, atol=0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("W,U,P,offset", SHAPES[1:8])
def test_non_finite_rows_reach_the_groups_they_are_members_of(W, U, P, offset, dtype):
    inf = float("inf")
    plain, C, _ = _call(W, U, P, offset, dtype)
    out, _, _ = _call(W, U, P, offset, dtype, [(0, P // 3, inf), (1, P - 1, float("nan")), (2, 0, -inf), (2, P // 2, inf)])
    has = [(C[:, w] != 0) for w in range(W)]
    nan, clean = has[1], ~(has[0] | has[1] | has[2])
    assert clean.any() and nan.any()
    assert torch.isnan(out[nan]).all()
    assert torch.isinf(out[(has[0] | has[2]) & ~nan]).all()
    # the same sums with some zeros added, by whichever of the two kernels
    torch.testing.assert_close(out[clean], plain[clean], rtol=2.0 ** -22, atol=0)


def test_shard_with_a_row_of_nan():
    """A worker that diverged: every tile holds NaN."""
    W, U, P = 8, 32, MI + 11
    plain, C, rows = _call(W, U, P, 0, torch.float32)
    bad, _, _ = _call(W, U, P, 0, torch.float32, [(3, slice(None), float("nan"))])
    has = C[:, 3] != 0
    assert torch.isnan(bad[has]).all() and (~has).any()
    torch.testing.assert_close(bad[~has], plain[~has], rtol=2.0 ** -22, atol=0)
