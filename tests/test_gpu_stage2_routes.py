"""Stage 2 across its routes -- a wave per row, a lane group per row, key ranges; a wave per key, query ranges -- at sizes on
either side of the rules, and where a wave's lane groups get no or few keys, against dense attention in 64 bits."""
from __future__ import annotations

import pytest
import torch

import paper_2502_07590_amd as dsv

pytestmark = pytest.mark.gpu


def _rows(L, k, g):
    edge = (torch.arange(k + 1, device="cuda") * L) // k
    width = edge[1:] - edge[:-1]
    idx = edge[:-1] + (torch.rand(L, k, generator=g, device="cuda") * width).long().clamp_max(width - 1)
    return idx.to(torch.int32)


def _dense(q, k, v, do, rows, scale):
    out = [torch.empty_like(q), q.new_empty(q.shape[0]), torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)]
    for a in range(0, q.shape[0], 2048):
        s = slice(a, min(a + 2048, q.shape[0]))
        keep = torch.zeros(rows[s].shape[0], k.shape[0], dtype=torch.bool, device="cuda").scatter_(1, rows[s].long(), True)
        x = (q[s] @ k.T * scale).masked_fill(~keep, -torch.inf)
        out[1][s] = torch.logsumexp(x, 1)
        p = (x - out[1][s][:, None]).exp()
        out[0][s] = p @ v
        dp = do[s] @ v.T
        ds = p * (dp - (p * dp).sum(1, keepdim=True))
        out[2][s] = ds @ k * scale
        out[3] += ds.T @ q[s] * scale
        out[4] += p.T @ do[s]
    return out


# Forward and dq step: a wave per row up to 6500 keys, a lane group per row at 8192 (and 16400, dq), ranges above -- eight in the
# forward and for the lists (above 6500 keys), in the dq step two, four and eight; without the flag waves and groups only.
@pytest.mark.parametrize("dtype,d,L,ks", [("f32", 64, 1, [1]), ("bf16", 128, 5, [5, 1, 2]), ("f32", 128, 70, [3, 70]), ("bf16", 64, 1030, [1, 33, 400]),
                                          ("bf16", 128, 2100, [300, 257]), ("bf16", 128, 4300, [40, 260, 100]), ("f32", 64, 6500, [256, 17]),
                                          ("bf16", 128, 16400, [768]), ("bf16", 128, 8192, [100, 60, 30, 31]), ("f32", 128, 6000, [900, 20]),
                                          ("f32", 64, 8200, [900] * 15 + [901]), ("f32", 64, 16400, [900, 1000, 700, 910])])
@pytest.mark.parametrize("in_order", [True, False])
def test_every_route_matches_dense_attention(dtype, d, L, ks, in_order):
    H = len(ks)
    g = torch.Generator(device="cuda").manual_seed(L + d)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dO = (torch.randn(1, H, L, d, generator=g, device="cuda").to(td) for _ in range(4))
    heads = [_rows(L, k, g) for k in ks]
    flat = torch.cat([(x if in_order else x.flip(1)).reshape(-1) for x in heads])
    p = dsv.Problem(1, H, L, d, 16, dtype, ks, d ** -0.5, sorted_index=in_order)
    O, lse = dsv.sparse_attn_fwd(p, Q, K, V, flat)
    grads = dsv.sparse_attn_bwd(p, Q, K, V, flat, O, lse, dO)
    idx_t, col = dsv.idx_transpose(p, flat)
    parts = dsv.sparse_attn_bwd_t(p, Q, K, V, flat, idx_t, col, O, lse, dO)
    # the bounds of the parity tests against the oracle: 2e-2 (bf16) and 1e-4 (fp32), a few output ulps where values are large
    floor, ulps = (2e-2, 2.0 ** -7) if dtype == "bf16" else (1e-4, 2.0 ** -20)
    for h in range(H):
        want = _dense(*(x[0, h].double() for x in (Q, K, V, dO)), heads[h], d ** -0.5)
        got = [O[0, h], lse[0, h]] + [x[0, h] for x in grads]
        for x, y in zip(got, want):
            assert ((x.double() - y).abs() <= torch.clamp_min(y.abs() * ulps, floor)).all()
        for x, y in zip([x[0, h] for x in parts], want[2:]):
            assert ((x.double() - y).abs() <= torch.clamp_min(y.abs() * ulps, floor)).all()


def _error(got, want):
    return float((got.double() - want).norm() / want.norm())


# Rows walked in one piece -- dense tiles, a wave per row, a lane group per row -- add nothing to the rounding of the output:
# one bf16 word per probability would make the error 1.09 times as large here.  fp32 rows: 341 sums in one chain leave 4.4e-7
# to 4.6e-7, folded ones 3.1e-7 to 3.4e-7; 1000 in eight ranges 3.8e-7 to 4.0e-7.
@pytest.mark.parametrize("dtype,d,H,L,k", [("bf16", 128, 12, 2048, 400), ("bf16", 64, 12, 2048, 500), ("bf16", 128, 1, 3000, 100), ("bf16", 64, 1, 2100, 300), ("bf16", 64, 2, 3000, 70),
                                           ("bf16", 128, 4, 8192, 273), ("bf16", 64, 4, 16384, 300),
                                           ("f32", 64, 4, 8192, 341), ("f32", 128, 4, 4300, 100), ("f32", 64, 4, 12000, 1000), ("f32", 128, 1, 3000, 300)])
def test_forward_error_is_that_of_its_rounding(dtype, d, H, L, k):
    g = torch.Generator(device="cuda").manual_seed(L)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V = (torch.randn(1, H, L, d, generator=g, device="cuda").to(td) for _ in range(3))
    rows = _rows(L, k, g)
    p = dsv.Problem(1, H, L, d, 16, dtype, [k] * H, 2 * d ** -0.5, sorted_index=True)
    O, _ = dsv.sparse_attn_fwd(p, Q, K, V, rows.reshape(-1).repeat(H))
    at = torch.arange(0, L, max(1, L // 500), device="cuda")
    for h in range(H):
        s = torch.gather(Q[0, h].double()[at] @ K[0, h].double().T * p.scale, 1, rows[at].long()).softmax(1)
        want = torch.stack([s[i] @ V[0, h].double()[rows[at[i]].long()] for i in range(len(at))])
        bound = 1.02 * _error(want.to(td), want) if dtype == "bf16" else 4.2e-7
        assert _error(O[0, h][at], want) <= bound


@pytest.mark.parametrize("cube", [(1, 2, 2), (2, 2, 2), (2, 4, 4)])
@pytest.mark.parametrize("in_order", [True, False])
def test_grouped_forward_error_is_that_of_its_rounding(cube, in_order):
    grid, k = (4, 32, 32), 500
    L, G = 4096, cube[0] * cube[1] * cube[2]
    g = torch.Generator(device="cuda").manual_seed(G)
    Q, K, V = (torch.randn(1, 1, L, 128, generator=g, device="cuda").bfloat16() for _ in range(3))
    rows = _rows(L, k, g)[:L // G]
    p = dsv.Problem(1, 1, L, 128, 16, "bf16", [k], 2 * 128 ** -0.5, sorted_index=in_order)
    O, _ = dsv.sparse_attn_fwd_grouped(p, dsv.Grouping(grid, cube), Q, K, V, rows.reshape(-1))
    tokens = torch.arange(L, device="cuda").reshape(*[n for a, b in zip(grid, cube) for n in (a // b, b)]).permute(0, 2, 4, 1, 3, 5).reshape(-1, G)
    q, kk, v = (x[0, 0].double() for x in (Q, K, V))
    want = torch.empty(L, 128, dtype=torch.float64, device="cuda")
    for i, t in enumerate(tokens):
        j = rows[i].long()
        want[t] = (q[t] @ kk[j].T * p.scale).softmax(1) @ v[j]
    assert _error(O[0, 0], want) <= 1.02 * _error(want.bfloat16(), want)
