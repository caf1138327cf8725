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


# bf16, d = 128: blocked from 16384 keys of k >= 768 on; lane groups from 12800 rows on; query ranges above 1 MB and k > 256
@pytest.mark.parametrize("dtype,d,L,ks", [("f32", 64, 1, [1]), ("bf16", 128, 5, [5, 1, 2]), ("f32", 128, 70, [3, 70]), ("bf16", 64, 1030, [1, 33, 400]),
                                          ("bf16", 128, 2100, [300, 257]), ("bf16", 128, 4300, [40, 260, 100]), ("f32", 64, 6500, [256, 17]),
                                          ("bf16", 128, 16400, [768])])
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
