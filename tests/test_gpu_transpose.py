"""The key-major form of an index (dsv_idx_transpose) against a stable sort of its pairs, and the backward that sorts
rows given in any order, at the edges of the blocks (512 keys x 1024 queries) and of the routes."""
from __future__ import annotations

import pytest
import torch

import paper_2502_07590_amd as dsv

pytestmark = pytest.mark.gpu


def _rows(L, k, seed, ascending):
    """int32 [L, k] on the device: one key from each of k equal strata (distinct), turned round in every row."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    edge = (torch.arange(k + 1, device="cuda") * L) // k
    width = edge[1:] - edge[:-1]
    idx = edge[:-1] + (torch.rand(L, k, generator=g, device="cuda") * width).long().clamp_max(width - 1)
    if not ascending:
        turn = torch.randint(0, k, (L, 1), generator=g, device="cuda")
        idx = torch.gather(idx, 1, (torch.arange(k, device="cuda")[None] + turn) % k)
    return idx.to(torch.int32)


def _expected(rows, L):
    keys = rows.reshape(-1)
    order = torch.sort(keys, stable=True).indices
    col = torch.zeros(L + 1, dtype=torch.int64, device="cuda")
    col[1:] = torch.bincount(keys, minlength=L).cumsum(0)
    return (order // rows.shape[1]).to(torch.int32), col


# L = 2000, k = 1: the entry sort (rows keep under 1/768 of the keys); L = 140000: the bit matrix goes piece by piece
@pytest.mark.parametrize("L,ks", [(1, [1]), (31, [7, 31]), (512, [40, 512]), (513, [100]), (1023, [64, 3]), (1024, [128]), (1025, [300, 1, 77]),
                                  (2000, [1]), (5121, [700, 33]), (140000, [600])])
@pytest.mark.parametrize("ascending", [True, False])
def test_transpose_is_a_stable_sort_of_the_pairs(L, ks, ascending):
    heads = [_rows(L, k, 10 * h + L, ascending) for h, k in enumerate(ks)]
    p = dsv.Problem(1, len(ks), L, 64, 16, "bf16", ks, 0.1)
    idx_t, col = dsv.idx_transpose(p, torch.cat([x.reshape(-1) for x in heads]))
    off = 0
    for h, rows in enumerate(heads):
        want, ptr = _expected(rows, L)
        assert torch.equal(col[h], ptr)
        assert torch.equal(idx_t[off:off + rows.numel()], want)
        off += rows.numel()


# bitmaps of four, three, two rows and one per block (up to 130560 keys, up to 174592, up to 261632, above); rows that begin at no multiple of 16 bytes,
# of up to 256 entries and more
@pytest.mark.parametrize("L,k", [(8192, 61), (16384, 1023), (131072, 171), (150001, 198), (200003, 263), (200003, 1031), (300007, 391)])
def test_bitmaps_of_rows(L, k):
    rows = _rows(L, k, L, True)
    p = dsv.Problem(1, 1, L, 64, 16, "bf16", [k], 0.1)
    idx_t, col = dsv.idx_transpose(p, rows.reshape(-1))
    want, ptr = _expected(rows, L)
    assert torch.equal(col[0], ptr) and torch.equal(idx_t, want)


# rows of 512 bytes of K and V: a head passes 3 MB above 6144 keys; from there rows in any order are sorted first, up to 524288
# keys (a row's bitmap: 64 KB of LDS)
@pytest.mark.parametrize("dtype,L,d,ks", [("bf16", 6145, 128, [300, 1]), ("f32", 6200, 64, [6200]), ("bf16", 20011, 64, [777]),
                                          ("bf16", 516097, 64, [5]), ("bf16", 524288, 64, [5])])
def test_backward_of_rows_in_any_order_equals_that_of_the_sorted_rows(dtype, L, d, ks):
    g = torch.Generator(device="cuda").manual_seed(L)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dO = (torch.randn(1, len(ks), L, d, generator=g, device="cuda").to(td) for _ in range(4))
    heads = [_rows(L, k, h, False) for h, k in enumerate(ks)]
    mixed = torch.cat([x.reshape(-1) for x in heads])
    ascending = torch.cat([x.sort(dim=1).values.reshape(-1) for x in heads])
    any_order = dsv.Problem(1, len(ks), L, d, 16, dtype, ks, d ** -0.5)
    in_order = dsv.Problem(1, len(ks), L, d, 16, dtype, ks, d ** -0.5, sorted_index=True)
    O, lse = dsv.sparse_attn_fwd(in_order, Q, K, V, ascending)
    got = dsv.sparse_attn_bwd(any_order, Q, K, V, mixed, O, lse, dO)
    want = dsv.sparse_attn_bwd(in_order, Q, K, V, ascending, O, lse, dO)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
