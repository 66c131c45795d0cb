"""Norms of up to 8 rows on a short shard: Gram sums and norms in one finishing launch (gram_finish_kernel).  The workgroup that
arrives last forms the norms and puts the ticket back, so calls are repeated: back to back, on two streams, from the entry point
that works in the fixed array, and as replays of a captured graph."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2512_09685_amd as star

pytestmark = pytest.mark.gpu

HP = dict(lr=0.1, momentum_coef=0.9, weight_decay=1e-4, wmode="stale")


def _inputs(W, U, P, seed=0):
    rng = np.random.default_rng([W, U, P, seed])
    sizes = rng.integers(1, W + 1, size=U)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    members = np.concatenate([rng.permutation(W)[:y] for y in sizes]).astype(np.int32)
    stale = rng.integers(0, 5, size=len(members)).astype(np.int32)
    C = torch.zeros(U, W, dtype=torch.float64)
    for u in range(U):
        for m in range(offs[u], offs[u + 1]):
            C[u, members[m]] = 1.0 / (sizes[u] * (1.0 + stale[m]))
    gen = torch.Generator(device="cuda").manual_seed(seed + U)
    rows = [torch.randn(P, generator=gen, device="cuda") * 1e-3 for _ in range(W)]
    want = (C.cuda() @ torch.stack(rows).double()).square().sum(1).sqrt()
    p, v = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    return star.GradRows(rows), star.UpdateStream(offs, members, stale), p, v, C.cuda(), want


def _finishing(W, us, P, dtype="f32", **kw):
    return star.star_plan_choice(P, W, dtype, us, want_norms=True, wmode="stale", **kw)["finishing_launches"]


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("W,U,P,launches", [(1, 16, 4096, 1), (2, 64, 4099, 1), (3, 33, 300007, 1), (5, 16, 70001, 1),
                                            (7, 64, 1 << 20, 1), (8, 17, 2 << 20, 1), (8, 17, (2 << 20) + 1, 2), (8, 128, 8191, 1),
                                            (8, 129, 8191, 2), (9, 17, 8191, 2)])
def test_norms(W, U, P, launches, noalloc):
    g, us, p, v, C, want = _inputs(W, U, P)
    assert _finishing(W, us, P, lr=0.1, momentum_coef=0.9) == launches
    call = star.star_group_update_noalloc if noalloc else star.star_group_update
    for _ in range(3):
        out = torch.full((U,), -1.0, device="cuda")
        call(p, v, g, us, norms_out=out, **HP)
        # n^2 = c^T Gamma c: entries of fp32 chains of at most 256 products, c >= 0 and rows that are nearly orthogonal
        torch.testing.assert_close(out.double(), want, rtol=1e-6, atol=0)
    g[0][P // 2] = float("nan")
    out = torch.full((U,), -1.0, device="cuda")
    call(p, v, g, us, norms_out=out, **HP)
    has = C[:, 0] != 0
    assert torch.isnan(out[has]).all()
    torch.testing.assert_close(out[~has].double(), want[~has], rtol=1e-6, atol=0)


@pytest.mark.parametrize("W,U,P,dtype", [(1, 1, 4096, "f32"), (1, 128, 300007, "f32"), (8, 64, 70001, "f32"), (8, 16, 2 << 20, "f32"),
                                         (1, 24, 300007, "bf16"), (2, 128, 1 << 20, "bf16")])
def test_norms_without_an_update(W, U, P, dtype):
    g, us, _, _, C, want = _inputs(W, U, P)
    if dtype == "bf16":
        g = star.GradRows([r.bfloat16() for r in g])
        want = (C @ torch.stack([r.double() for r in g])).square().sum(1).sqrt()
    assert _finishing(W, us, P, dtype, update=False) == 1
    for _ in range(3):
        out = torch.full((U,), -1.0, device="cuda")
        star.star_group_norms(g, us, out, wmode="stale")
        torch.testing.assert_close(out.double(), want, rtol=1e-6, atol=0)


def test_two_streams():
    cases = [_inputs(8, 16, 300007, 1), _inputs(4, 40, 123457, 2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    outs = []
    for k in range(40):
        g, us, p, v, _, want = cases[k % 2]
        with torch.cuda.stream(streams[k % 2]):
            out = torch.full((us.U,), -1.0, device="cuda")
            star.star_group_update(p, v, g, us, norms_out=out, **HP)
            outs.append((out, want))
    torch.cuda.synchronize()
    for out, want in outs:
        torch.testing.assert_close(out.double(), want, rtol=1e-6, atol=0)


def test_captured():
    g, us, p, v, _, want = _inputs(6, 24, 200003, 3)
    out = torch.empty(us.U, device="cuda")
    call = lambda: star.star_group_update_noalloc(p, v, g, us, norms_out=out, **HP)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(4):
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        torch.testing.assert_close(out.double(), want, rtol=1e-6, atol=0)
        out.fill_(-1.0)
        call()   # the program's own call between the replays
        torch.cuda.synchronize()
        torch.testing.assert_close(out.double(), want, rtol=1e-6, atol=0)


def test_ticket_left_out_of_step():
    """Calls of the entry point without allocation that overlap race on the fixed array, but may not spoil the ones after them: whatever the
    ticket holds (64 bytes into the array) when a call begins, its norms are right."""
    g, us, p, v, _, want = _inputs(4, 24, 70001, 4)
    assert _finishing(4, us, 70001, lr=0.1, momentum_coef=0.9) == 1
    base = ctypes.c_void_p()
    assert getattr(star.load_library(), "_ZN4star15scratch_addressEPPv")(ctypes.byref(base)) == 0
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    for left in (1000, 1, 0):
        torch.cuda.synchronize()
        ticket = ctypes.c_uint32(left)
        assert hip.hipMemcpy(base.value + 64, ctypes.byref(ticket), 4, 1) == 0   # host to device
        out = torch.full((us.U,), -1.0, device="cuda")
        star.star_group_update_noalloc(p, v, g, us, norms_out=out, **HP)
        torch.testing.assert_close(out.double(), want, rtol=1e-6, atol=0)
