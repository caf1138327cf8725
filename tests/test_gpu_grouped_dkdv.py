"""dK and dV of the grouped backward at the edges of its tiles (16 keys, 32 queries per step, 1024 groups per window, ranges
of 8192 queries), against the per-query backward of the same selection with the group's row given to every member."""
from __future__ import annotations

import math

import pytest
import torch

import paper_2502_07590_amd as dsv

pytestmark = pytest.mark.gpu


# keys that neighbours share, that they do not, one head of each; cubes of 1, 2, 3, 8, 12 and 32 queries; more than one window of groups;
# keys nobody selects.  Up to the first comment eight ranges (six for 17 keys), the small ones by unions whatever the keys; then one
# range (8192 keys at most, 4096 blocks of 64 rows), two (2048 blocks) and four (16384 keys, 1024 blocks), by unions where
# neighbours share keys (and where a row keeps one in ten), by the per-query sweep where they do not.
@pytest.mark.parametrize("grid,cube,ks", [((1, 1, 17), (1, 1, 1), [5]), ((3, 5, 7), (3, 1, 1), [1, 40]), ((2, 6, 30), (2, 1, 1), [77]),
                                          ((4, 48, 48), (1, 3, 4), [300, 64]), ((8, 32, 48), (2, 2, 2), [700]), ((4, 72, 72), (2, 1, 1), [90]),
                                          ((8, 64, 72), (2, 4, 4), [500]),
                                          ((4, 16, 16), (1, 2, 2), [40] * 256),  # one range
                                          ((8, 27, 38), (2, 1, 1), [100] * 16), ((4, 16, 16), (2, 2, 2), [100] * 128),  # two
                                          ((2, 96, 86), (1, 2, 2), [200, 160, 180, 40]),  # four
                                          # and 5e7 pairs, the form head by head: eight ranges, and one
                                          ((8, 32, 32), (2, 2, 2), [4096, 60, 2048, 60]), ((4, 16, 16), (1, 2, 2), [200] * 256)])
@pytest.mark.parametrize("near", [(True, True), (False, False), (True, False)])
def test_grouped_gradients_of_keys_and_values(grid, cube, ks, near):
    L, G, H = math.prod(grid), math.prod(cube), len(ks)
    (F, Hh, Ww), (gf, gh, gw) = grid, cube
    g = torch.Generator(device="cuda").manual_seed(L)
    Q, K, V, dO = (torch.randn(1, H, L, 128, generator=g, device="cuda").bfloat16() for _ in range(4))
    tokens = torch.arange(L, device="cuda").reshape(F // gf, gf, Hh // gh, gh, Ww // gw, gw).permute(0, 2, 4, 1, 3, 5).reshape(-1, G)
    idx_g, idx, lists, cols = [], [], [], []
    for h, k in enumerate(ks):
        # evenly spread, or one after the other, from a start of the group's own, never the last 7 keys (L > 8): distinct, lists of uneven length
        n = max(L - 7, k)
        first = (torch.rand(L // G, 1, generator=g, device="cuda") ** 2 * n).long()
        rows = ((first + torch.arange(k, device="cuda")[None] * (1 if near[h % 2] else n // k)) % n).sort(1).values
        rows = rows.to(torch.int32)
        full = torch.empty(L, k, dtype=torch.int32, device="cuda")
        full[tokens.reshape(-1)] = rows.repeat_interleave(G, 0)
        order = torch.sort(rows.reshape(-1), stable=True).indices
        col = torch.zeros(L + 1, dtype=torch.int64, device="cuda")
        col[1:] = torch.bincount(rows.reshape(-1), minlength=L).cumsum(0)
        idx_g.append(rows.reshape(-1)); idx.append(full.reshape(-1)); lists.append((order // k).to(torch.int32)); cols.append(col)
    p = dsv.Problem(1, H, L, 128, 16, "bf16", ks, 128 ** -0.5, sorted_index=True)
    grp = dsv.Grouping(grid, cube)
    O, lse = dsv.sparse_attn_fwd(p, Q, K, V, torch.cat(idx))
    want = dsv.sparse_attn_bwd(p, Q, K, V, torch.cat(idx), O, lse, dO)
    got = dsv.sparse_attn_bwd_grouped(p, grp, Q, K, V, torch.cat(idx_g), torch.cat(lists), torch.stack(cols), O, lse, dO)
    # both are fp32 sums rounded to bf16 once: the parity bound of the tests against the oracle
    for a, b in zip(got, want):
        a, b = a.float(), b.float()
        assert ((a - b).abs() <= torch.clamp_min(b.abs() * 2.0 ** -7, 2e-2)).all()


# a gradient row that is not finite belongs to the keys that its group keeps, and to no others; eight ranges, and one
@pytest.mark.parametrize("grid,bad,H", [((4, 16, 16), float("inf"), 1), ((4, 48, 48), float("nan"), 1), ((4, 16, 16), float("nan"), 256)])
def test_gradient_rows_that_are_not_finite(grid, bad, H):
    L, k, cube = math.prod(grid), 200, (2, 2, 2)
    g = torch.Generator(device="cuda").manual_seed(L)
    Q, K, V, dO = (torch.randn(1, H, L, 128, generator=g, device="cuda").bfloat16() for _ in range(4))
    ids = torch.arange(L, device="cuda").reshape(grid[0] // 2, 2, grid[1] // 2, 2, grid[2] // 2, 2).permute(0, 2, 4, 1, 3, 5).reshape(-1, 8)
    rows = torch.rand(L // 8, L, generator=g, device="cuda").topk(k, 1).indices.sort(1).values.to(torch.int32)
    order = torch.sort(rows.reshape(-1), stable=True).indices
    col = torch.zeros(L + 1, dtype=torch.int64, device="cuda")
    col[1:] = torch.bincount(rows.reshape(-1), minlength=L).cumsum(0)
    full = torch.empty(L, k, dtype=torch.int32, device="cuda")
    full[ids.reshape(-1)] = rows.repeat_interleave(8, 0)
    p = dsv.Problem(1, H, L, 128, 16, "bf16", [k] * H, 128 ** -0.5, sorted_index=True)
    grp = dsv.Grouping(grid, cube)
    O, lse = dsv.sparse_attn_fwd(p, Q, K, V, full.reshape(-1).repeat(H))
    args = (rows.reshape(-1).repeat(H), (order // k).to(torch.int32).repeat(H), col.repeat(H, 1), O, lse)
    clean = dsv.sparse_attn_bwd_grouped(p, grp, Q, K, V, *args, dO)
    group = 5
    dO[0, H - 1, ids[group, 3]] = bad
    got = dsv.sparse_attn_bwd_grouped(p, grp, Q, K, V, *args, dO)
    keeps = torch.zeros(L, dtype=torch.bool, device="cuda")
    keeps[rows[group].long()] = True
    for a, b in zip(got[1:], clean[1:]):
        assert not a[0, H - 1, keeps].isfinite().all(-1).any() and a[0, H - 1, ~keeps].isfinite().all()
        assert torch.equal(a[0, :H - 1], b[0, :H - 1])
        a, b = a[0, H - 1, ~keeps].float(), b[0, H - 1, ~keeps].float()
        assert ((a - b).abs() <= torch.clamp_min(b.abs() * 2.0 ** -7, 2e-2)).all()  # sums of another order: the bound above
