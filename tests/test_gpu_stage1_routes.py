"""Stage 1 at the edges of its routes and tiles: the index must be the stable top-k of the device's own scores (larger
score first, lower key on ties), whatever kernels an L, a k and a type lead through, and idx_t its transpose."""
from __future__ import annotations

import ctypes

import pytest
import torch

import paper_2502_07590_amd as dsv

pytestmark = pytest.mark.gpu


def _inputs(H, L, d, r, dtype, ties, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    if ties:   # integer scores: most thresholds are tied
        draw = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda").to(td)
        return draw(1, H, L, d), draw(1, H, L, d), draw(H, d, r), draw(H, d, r)
    draw = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return draw(1, H, L, d).to(td), draw(1, H, L, d).to(td), (draw(H, d, r) / d ** 0.5).to(td), (draw(H, d, r) / d ** 0.5).to(td)


def _check(p, Q, K, Wq, Wk):
    idx, idx_t, col = dsv.lowrank_topk_t(p, Q, K, Wq, Wk)
    assert torch.equal(idx, dsv.lowrank_topk(p, Q, K, Wq, Wk))
    want_t, want_col = dsv.idx_transpose(p, idx)
    assert torch.equal(idx_t, want_t) and torch.equal(col, want_col)
    Qlr, Klr = dsv.lowrank_project(p, Q, K, Wq, Wk)
    off = 0
    for h, k in enumerate(p.k_per_head):
        S = dsv.lowrank_scores_rows(p, Qlr, Klr, 0, h, torch.arange(p.L, dtype=torch.int32, device="cuda"))
        best = torch.sort(S, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values.to(torch.int32)
        assert torch.equal(idx[off:off + p.L * k].reshape(p.L, k), best), f"head {h}"
        off += p.L * k


# one kernel up to 2048 keys (512, 1024, 2048: 1, 2, 4 score tiles per wave), the radix passes above (and, in bf16 below rank 64, from
# 257 blocks of 32 queries and more than 1024 keys on)
@pytest.mark.parametrize("L,ks", [(1, [1, 1]), (33, [33, 1]), (512, [100, 511]), (513, [7, 64]), (1025, [1025, 200]), (2048, [1, 300]),
                                  (1025, [1025, 200] * 4), (2049, [150, 2048])])
@pytest.mark.parametrize("dtype,d,r", [("f32", 64, 16), ("bf16", 128, 32), ("bf16", 64, 64)])
@pytest.mark.parametrize("ties", [False, True])
def test_short_sequences(L, ks, dtype, d, r, ties):
    Q, K, Wq, Wk = _inputs(len(ks), L, d, r, dtype, ties, L + r)
    _check(dsv.Problem(1, len(ks), L, d, r, dtype, ks, 0.1), Q, K, Wq, Wk)


def _all_indices(p, grp, Q, K, Wq, Wk):
    return (dsv.lowrank_topk(p, Q, K, Wq, Wk), *dsv.lowrank_topk_t(p, Q, K, Wq, Wk), *dsv.lowrank_topk_grouped(p, grp, Q, K, Wq, Wk))


def _launches(call):
    """Nodes of the graph that capturing the call gives: its kernel launches."""
    graph, n = torch.cuda.CUDAGraph(keep_graph=True), ctypes.c_size_t(0)
    with torch.cuda.graph(graph):
        call()
    assert ctypes.CDLL("libamdhip64.so").hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("grid,ks", [((1, 1, 2), [1, 2]), ((1, 5, 10), [49, 3]), ((8, 8, 8), [100, 511]), ((3, 19, 9), [7, 64]),
                                     ((4, 16, 32), [1, 300])])
@pytest.mark.parametrize("dtype,d,r", [("f32", 64, 16), ("bf16", 128, 32)])
@pytest.mark.parametrize("ties", [False, True])
def test_the_radix_search_is_to_be_had_for_short_sequences(grid, ks, dtype, d, r, ties):
    """Mode 1 is the radix search at every length.  Where the automatic mode takes one kernel after the projection, the four
    passes and the emission give the same bits; the launches that a capture records show that they ran."""
    L = grid[0] * grid[1] * grid[2]
    Q, K, Wq, Wk = _inputs(2, L, d, r, dtype, ties, L + r)
    p, grp = dsv.Problem(1, 2, L, d, r, dtype, ks, 0.1), dsv.Grouping(grid, (1, 1, 2 if grid[2] % 2 == 0 else grid[2]))
    one, launches_one = _all_indices(p, grp, Q, K, Wq, Wk), _launches(lambda: dsv.lowrank_topk(p, Q, K, Wq, Wk))
    assert dsv.threshold_search(1) == 0
    try:
        radix, launches = _all_indices(p, grp, Q, K, Wq, Wk), _launches(lambda: dsv.lowrank_topk(p, Q, K, Wq, Wk))
    finally:
        dsv.threshold_search(0)
    assert launches == launches_one + 4 == 6
    for a, b in zip(one, radix):
        assert torch.equal(a, b)


# above 2048 keys: radix passes, from 16384 on the windowed search
@pytest.mark.parametrize("H,L,ks,r,ties", [(1, 2080, [2080], 16, False), (2, 5001, [5, 900], 64, True), (1, 16411, [1500], 16, False),
                                           (3, 22000, [1100, 2, 5000], 16, False)])
def test_longer_sequences(H, L, ks, r, ties):
    Q, K, Wq, Wk = _inputs(H, L, 64, r, "bf16", ties, L)
    _check(dsv.Problem(1, H, L, 64, r, "bf16", ks, 0.1), Q, K, Wq, Wk)


# the emission by blocks and by waves, on either side of the line between them: query tiles against the length, the type and
# the rank, and for short rows of bf16 half as many again
@pytest.mark.parametrize("dtype,H,L,k,r", [("f32", 6, 2080, 130, 16), ("f32", 7, 2080, 130, 16), ("f32", 3, 2080, 40, 64), ("f32", 4, 2080, 40, 64),
                                           ("f32", 4, 2080, 2080, 32), ("bf16", 6, 2080, 9, 64), ("bf16", 7, 2080, 1040, 64),
                                           ("bf16", 31, 2080, 65, 32), ("bf16", 32, 2080, 65, 32), ("bf16", 9, 8192, 256, 16), ("bf16", 9, 8192, 257, 16)])
@pytest.mark.parametrize("ties", [False, True])
def test_emission(dtype, H, L, k, r, ties):
    Q, K, Wq, Wk = _inputs(H, L, 64, r, dtype, ties, H + r)
    _check(dsv.Problem(1, H, L, 64, r, dtype, [k] * H, 0.1), Q, K, Wq, Wk)


# emission in batches of up to 32 key tiles (16 query tiles for the lists) by four waves in turn: one tile over a round, over two, an odd
# number of tiles; every score twice, so that queries in two take one of two ties, whose places lie batches apart
@pytest.mark.parametrize("dtype,H,L,ks,r", [("bf16", 8, 4097, [256] * 8, 16), ("bf16", 5, 8193, [2000, 8193, 3, 511, 130], 32), ("bf16", 2, 16385, [1025, 77], 16),
                                            ("bf16", 4, 4160, [260, 1, 4159, 1000], 64), ("f32", 4, 3007, [189, 3000, 2, 750], 32)])
def test_emission_in_batches(dtype, H, L, ks, r):
    Q, K, Wq, Wk = _inputs(H, L, 64, r, dtype, False, L + r)
    _check(dsv.Problem(1, H, L, 64, r, dtype, ks, 0.1), Q, K, Wq, Wk)
    K[:, :, L - L // 2:] = K[:, :, :L // 2]
    _check(dsv.Problem(1, H, L, 64, r, dtype, ks, 0.1), Q, K, Wq, Wk)


# lists of up to 48 query tiles are written by owners, 16 tiles at a time, and of up to 32 counted by all waves: one tile, a few, 15 to 17, 32 and 33, 48 and 49
@pytest.mark.parametrize("dtype,r", [("bf16", 16), ("bf16", 64), ("f32", 32)])
@pytest.mark.parametrize("L", [31, 97, 160, 480, 512, 513, 1024, 1025, 1536, 1537])
@pytest.mark.parametrize("ties", [False, True])
def test_lists_of_few_queries(dtype, r, L, ties):
    ks = [1, L, max(1, L // 3)]
    Q, K, Wq, Wk = _inputs(3, L, 64, r, dtype, ties, L + r)
    _check(dsv.Problem(1, 3, L, 64, r, dtype, ks, 0.1), Q, K, Wq, Wk)


def test_smooth_inputs_keep_the_windowed_search():
    """Keys that vary slowly along the token grid, whose width the sample's stride divides: the scrambled sample brackets
    the thresholds, and the result is the radix search's."""
    L, k = 16384, 1024
    g = torch.Generator(device="cuda").manual_seed(1)
    t = torch.arange(L, device="cuda", dtype=torch.float32)
    wave = torch.stack([torch.cos(2 * torch.pi * t / period + phase) for period in (64.0, 32.0, 4096.0, 1500.0)
                        for phase in (0.0, 1.0, 2.0, 3.0)], 1)
    mix = torch.randn(16, 64, generator=g, device="cuda")
    Q, K = ((wave @ mix + 0.1 * torch.randn(L, 64, generator=g, device="cuda")).bfloat16()[None, None].contiguous() for _ in range(2))
    Wq, Wk = ((torch.randn(1, 64, 16, generator=g, device="cuda") / 8).bfloat16() for _ in range(2))
    _check(dsv.Problem(1, 1, L, 64, 16, "bf16", [k], 0.1), Q, K, Wq, Wk)


# 64 tokens per wave, 256 per block; 4 outputs per lane below 32768 tokens, 16 or 32 from there on
@pytest.mark.parametrize("L", [1, 65, 321, 16385])
@pytest.mark.parametrize("dtype,d,r", [("f32", 64, 16), ("f32", 128, 64), ("bf16", 128, 32), ("bf16", 64, 64), ("bf16", 128, 16)])
def test_projection(L, dtype, d, r):
    Q, K, Wq, Wk = _inputs(2, L, d, r, dtype, False, L + d)
    p = dsv.Problem(1, 2, L, d, r, dtype, [1, 1], 0.1)
    for X, W, got in zip((Q, K), (Wq, Wk), dsv.lowrank_project(p, Q, K, Wq, Wk)):
        want = X.double() @ W.double()
        # a chain of d fp32 multiply-adds, rounded to the storage type once
        bound = d * 2.0 ** -24 * (X.double().abs() @ W.double().abs()) + want.abs() * (2.0 ** -8 if dtype == "bf16" else 0.0)
        assert ((got.double() - want).abs() <= bound).all()
