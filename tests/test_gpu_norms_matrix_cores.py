"""Direct norm sums on the matrix cores (norm_mma_kernel) at the edges of its tiles, blocks and launches: rows that are no
multiple of four, updates around 16 and beyond one workgroup's 64, the shortest shards it takes, shards that end inside a lane's
load, odd starts, groups that nearly cancel, and rows with infinities and NaN, which a dense product would spread over groups they are no
members of.  Every case asks the library which kernel it would take."""
import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star

pytestmark = pytest.mark.gpu

MI = 1 << 20
F, B = torch.float32, torch.bfloat16
# Norms against 64 bits: the coefficients and the result are rounded to fp32 (6e-8 each), a group sum of y terms carries at most y
# roundings of 6e-8 that average out over the elements, and four squares are added in fp32 (double beyond).
TOL = 3e-7


def _head(offset, dtype):
    """Elements before the first whole cache line of rows that start `offset` elements into an aligned buffer."""
    return -offset % (128 // dtype.itemsize)


def _on_matrix_cores(us, W, P, offset, dtype, **kw):
    return star.star_plan_choice(P - _head(offset, dtype), W, "f32" if dtype == F else "bf16", us, update=False, want_norms=True,
                                 direct_norms=True, **kw)["norms_on_matrix_cores"]


def _stream(W, U, least, seed):
    """Groups of `least` to W workers; the first is the last worker alone."""
    rng = np.random.default_rng(seed)
    sizes = rng.integers(least, W + 1, size=U)
    sizes[0] = 1
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    members = np.concatenate([[W - 1]] + [rng.permutation(W)[:y] for y in sizes[1:]]).astype(np.int32)
    C = torch.zeros(U, W, dtype=torch.float64, device="cuda")
    for u in range(U):
        C[u, members[offs[u]:offs[u + 1]]] = 1.0 / sizes[u]
    return star.UpdateStream(offs, members), C


def _rows(W, U, P, offset, dtype):
    gen = torch.Generator(device="cuda").manual_seed(W * 1000 + U)
    return [(torch.randn(P + offset, generator=gen, device="cuda") * 1e-3).to(dtype)[offset:] for _ in range(W)]


def _norms(rows, us, **kw):
    out = torch.full((us.U,), -1.0, device="cuda")
    star.star_group_norms(star.GradRows(rows), us, out, direct_norms=True, **kw)
    return out


def _exact(C, rows):
    sums = torch.zeros(C.shape[0], dtype=torch.float64, device="cuda")
    for lo in range(0, rows[0].shape[0], MI // 4):
        g = torch.stack([r[lo:lo + MI // 4].double() for r in rows])
        sums += (C @ g).square().sum(1)
    return sums.sqrt()


# the last field: whether the matrix cores take it.  The shortest shards are a few elements above and one below their limits.
SHAPES = [(3, 2, 64, MI + 5, 0, F, 1), (3, 2, 64, MI + 5, 0, B, 1), (4, 3, 48, MI + 7, 3, F, 1), (4, 3, 48, MI + 61 + 1, 3, B, 1),
          (5, 4, 96, 2 * MI - 1, 0, F, 1), (6, 3, 17, 2 * MI - 1, 0, B, 1), (7, 4, 32, MI - 1, 2, F, 1), (8, 4, 16, MI, 1, F, 1),
          (8, 4, 16, MI, 1, B, 1), (8, 4, 240, MI + 4095, 0, F, 1), (8, 4, 240, MI + 4095, 0, B, 1), (9, 6, 31, MI + 2, 0, F, 1),
          (13, 8, 47, MI + 2047, 7, F, 1), (13, 6, 33, MI + 2047, 7, B, 1), (16, 8, 65, MI + 7, 0, F, 1), (16, 8, 65, MI + 7, 0, B, 1),
          (20, 10, 32, MI + 3, 2, F, 1), (20, 10, 32, MI + 3, 2, B, 1), (24, 12, 64, MI + 63, 0, F, 1), (24, 12, 64, MI + 63, 0, B, 1),
          (32, 16, 17, MI + 1025, 5, F, 1), (32, 16, 16, MI + 1025, 5, B, 1), (32, 16, 128, MI + 2, 0, F, 1),
          (32, 16, 128, MI + 2, 0, B, 1),
          (8, 4, 32, (1 << 17) + 27 + 3, 5, F, 1), (8, 4, 32, (1 << 17) + 27 - 1, 5, F, 0), (8, 4, 32, (1 << 19) + 59 + 1, 5, B, 1),
          (8, 4, 32, (1 << 19) + 59 - 1, 5, B, 0), (16, 8, 48, (1 << 19) + 1 + 2, 63, B, 1), (4, 3, 64, (1 << 18) + 5, 0, F, 1),
          (4, 3, 64, (1 << 18) - 1, 0, F, 0)]


@pytest.mark.parametrize("W,least,U,P,offset,dtype,matrix", SHAPES)
def test_direct_norms(W, least, U, P, offset, dtype, matrix):
    us, C = _stream(W, U, least, [W, U, P])
    assert _on_matrix_cores(us, W, P, offset, dtype) == matrix
    rows = _rows(W, U, P, offset, dtype)
    torch.testing.assert_close(_norms(rows, us).double(), _exact(C, rows), rtol=TOL, atol=0)


@pytest.mark.parametrize("dtype", [F, B])
@pytest.mark.parametrize("W,U", [(4, 64), (8, 32), (13, 64), (16, 64), (32, 128)])
def test_groups_that_nearly_cancel(W, U, dtype):
    """What direct sums are asked for.  Rows that are one vector up to a hundredth, in groups whose coefficients add up to zero: kappa of
    1e4 and more.  An element of gbar carries roundings of its products, at most W 2^-24 sqrt(kappa) of its size, 1e-3, which
    are independent of its sign and average out over 1 Mi elements to 1e-6 (seen: 2.4e-7)."""
    gen = torch.Generator(device="cuda").manual_seed(W + U)
    base = torch.randn(MI, generator=gen, device="cuda") * 1e-3
    rows = [(base + 1e-5 * torch.randn(MI, generator=gen, device="cuda")).to(dtype) for _ in range(W)]
    rng = np.random.default_rng(3)
    offs, members, coeff = [0], [], []
    for _ in range(U):
        k = int(rng.integers(max(1, W // 4), W // 2 + 1))
        c = rng.uniform(0.1, 1.0, k).astype(np.float32)
        members += list(rng.permutation(W)[:2 * k])
        coeff += list(c) + list(-c[rng.permutation(k)])
        offs.append(len(members))
    C = torch.zeros(U, W, dtype=torch.float64)
    for u in range(U):
        for m in range(offs[u], offs[u + 1]):
            C[u, members[m]] = float(coeff[m])
    C = C.cuda()
    us = star.UpdateStream(offs, members, None, coeff)
    assert _on_matrix_cores(us, W, MI, 0, dtype, wmode="explicit") == 1
    want = _exact(C, rows)
    size = torch.stack([r.double().norm() for r in rows])
    assert float(((C.abs() @ size) / want).square().min()) > 1e4
    torch.testing.assert_close(_norms(rows, us, wmode="explicit").double(), want, rtol=1e-6, atol=0)


@pytest.mark.parametrize("dtype", [F, B])
@pytest.mark.parametrize("W,least,U,P,offset", [(4, 2, 64, MI + 63, 3), (8, 4, 16, MI, 1), (8, 4, 240, MI + 4095, 0), (13, 8, 47, MI + 2047, 7),
                                                (16, 8, 65, MI + 7, 0), (20, 10, 32, MI + 3, 2), (24, 12, 64, MI + 63, 0)])
def test_non_finite_rows_reach_the_groups_they_are_members_of(W, least, U, P, offset, dtype):
    inf = float("inf")
    us, C = _stream(W, U, least, [W, U, P])
    assert _on_matrix_cores(us, W, P, offset, dtype) == 1
    rows = _rows(W, U, P, offset, dtype)
    plain = _norms(rows, us)
    for w, j, x in [(0, P // 3, inf), (1, P - 1, float("nan")), (2, 0, -inf), (2, P // 2, inf)]:
        rows[w][j] = x
    out = _norms(rows, us)
    has = [(C[:, w] != 0) for w in range(W)]
    nan, clean = has[1], ~(has[0] | has[1] | has[2])
    assert clean.any() and nan.any()
    assert torch.isnan(out[nan]).all()
    assert torch.isinf(out[(has[0] | has[2]) & ~nan]).all()
    # the same sums with some zeros added
    torch.testing.assert_close(out[clean], plain[clean], rtol=2.0 ** -22, atol=0)


def test_shard_with_a_row_of_nan():
    """A worker that diverged: every tile holds NaN."""
    W, U, P = 8, 32, MI + 11
    us, C = _stream(W, U, W // 2, [W, U, P])
    rows = _rows(W, U, P, 0, F)
    plain = _norms(rows, us)
    rows[3].fill_(float("nan"))
    bad = _norms(rows, us)
    has = C[:, 3] != 0
    assert torch.isnan(bad[has]).all() and (~has).any()
    torch.testing.assert_close(bad[~has], plain[~has], rtol=2.0 ** -22, atol=0)


KINDS = ["finite", "+inf", "-inf", "both", "some +inf", "some -inf", "some of both", "first and last", "some NaN", "NaN"]


def _spoil(row, kind, rng):
    inf, P = float("inf"), row.shape[0]
    some = None if rng is None else torch.from_numpy(rng.integers(0, P, size=40)).cuda()
    if kind in ("+inf", "-inf", "NaN"):
        row.fill_(float(kind))
    elif kind == "both":
        row.fill_(inf)
        row[::2] = -inf
    elif kind == "first and last":
        row[0], row[-1] = inf, -inf
    elif kind != "finite":
        row[some] = float("nan") if kind == "some NaN" else (-inf if kind == "some -inf" else inf)
        if kind == "some of both":
            row[some[::2]] = -inf


@pytest.mark.parametrize("dtype", [F, B])
@pytest.mark.parametrize("W,U,P,offset", [(4, 64, MI + 70, 3), (8, 32, MI, 0), (8, 128, MI + 62, 1), (13, 64, MI + 2047, 7),
                                          (24, 48, MI + 69, 2), (32, 64, MI + 6, 0)])
def test_infinities_and_nan_of_every_kind(W, U, P, offset, dtype):
    """Norms are NaN and infinite exactly where the definition is, sum by sum: a NaN, an infinity times a coefficient of zero, infinities
    of both signs at one element; and infinite otherwise."""
    us0, _ = _stream(W, U, max(1, W // 2), [W, U, P])
    plain = _rows(W, U, P, offset, dtype)
    for seed in range(6):
        rng = np.random.default_rng([W, U, seed])
        kinds = rng.choice(KINDS[:8] if seed < 4 else KINDS, size=W, p=None if seed else [0.44] + 7 * [0.08])
        coeff = rng.choice([-1.0, -0.5, 0.25, 1.0] if seed % 2 else [0.25, 0.5, 1.0], size=len(us0.members)).astype(np.float32)
        if seed == 3:
            coeff[rng.random(len(coeff)) < 0.05] = 0.0
        us = star.UpdateStream(us0.offsets, us0.members, None, coeff)
        assert _on_matrix_cores(us, W, P, offset, dtype, wmode="explicit") == 1
        rows = [r.clone() for r in plain] if not offset else [torch.cat([r.new_zeros(offset), r])[offset:] for r in plain]
        for r, kind in zip(rows, kinds):
            _spoil(r, kind, rng)
        out = _norms(rows, us, wmode="explicit")
        for u in range(U):
            gbar = torch.zeros(P, dtype=torch.float64, device="cuda")
            for m in range(us.offsets[u], us.offsets[u + 1]):
                gbar += float(coeff[m]) * rows[us.members[m]].double()
            want = float(gbar.square().sum().sqrt())
            got = float(out[u])
            assert got == pytest.approx(want, rel=TOL, nan_ok=True), (seed, u, [kinds[w] for w in us.members[us.offsets[u]:us.offsets[u + 1]]])


def _microseconds(call):
    best = float("inf")
    for _ in range(3):
        call()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 200)
    return best


@pytest.mark.parametrize("dtype", [F, B])
@pytest.mark.parametrize("kinds", [["+inf"], ["both"], ["+inf", "+inf"], ["+inf", "NaN"], 8 * ["+inf"]])
def test_workers_that_diverged_do_not_slow_the_call_down(kinds, dtype):
    """Every tile holds infinities then.  The search for them and their removal cost up to half as much again as the call; looked at
    element by element, tile after tile, it was 6 to 20 times."""
    W, U, P = 8, 32, 8 * MI
    us, _ = _stream(W, U, 1, [W, U, P])
    rows = _rows(W, U, P, 0, dtype)
    g, out = star.GradRows(rows), torch.empty(U, device="cuda")
    call = lambda: star.star_group_norms(g, us, out, direct_norms=True)
    clean = _microseconds(call)
    for r, kind in zip(rows, kinds):
        _spoil(r, kind, None)
    bad = _microseconds(call)
    print(f"{kinds} {dtype}: {clean:.1f} -> {bad:.1f} us", flush=True)
    assert bad < 3 * clean


@pytest.mark.parametrize("dtype", [F, B])
@pytest.mark.parametrize("W", [1, 2, 4, 5, 8, 12, 24])
def test_norms_are_not_biased(W, dtype):
    """The mean of the signed error over many updates.  A norm is rounded to fp32, 2.5e-8 rms, which over 720 updates averages out to
    1e-9; the roundings within the sums differ from update to update, a few 1e-9 each (the table is fp32 on both sides)."""
    U, P, err = 240, MI + 64, []
    for seed in range(3):
        rng = np.random.default_rng([W, seed])
        sizes = rng.integers(1, W + 1, size=U)
        offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        members = np.concatenate([rng.permutation(W)[:y] for y in sizes]).astype(np.int32)
        coeff = rng.standard_normal(len(members)).astype(np.float32)
        C = np.zeros((U, W))
        for u in range(U):
            C[u, members[offs[u]:offs[u + 1]]] = coeff[offs[u]:offs[u + 1]]
        us = star.UpdateStream(offs, members, None, coeff)
        if dtype == B:
            assert _on_matrix_cores(us, W, P, 0, dtype, wmode="explicit") == 1
        rows = _rows(W, seed, P, 0, dtype)
        err.append(_norms(rows, us, wmode="explicit").double() / _exact(torch.tensor(C, device="cuda"), rows) - 1)
    assert abs(float(torch.cat(err).mean())) < 5e-9
