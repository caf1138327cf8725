"""The forward over dense tiles with a mask, next to gathered heads in one call, at the edges of its tiles (128 queries,
64 keys), on rows that leave whole tiles out, and where the mask goes piece by piece; against attention in 64 bits."""
from __future__ import annotations

import pytest
import torch

import paper_2502_07590_amd as dsv

pytestmark = pytest.mark.gpu


def _check(p, Q, K, V, heads, at):
    O, lse = dsv.sparse_attn_fwd(p, Q, K, V, torch.cat([x.reshape(-1) for x in heads]))
    for bh, rows in enumerate(heads):
        b, h = divmod(bh, p.H)
        q, k, v = Q[b, h].double()[at], K[b, h].double(), V[b, h].double()
        s = torch.gather(q @ k.T * p.scale, 1, rows[at].long())
        want = torch.logsumexp(s, 1)
        prob = (s - want[:, None]).exp()
        out = torch.stack([prob[i] @ v[rows[at[i]].long()] for i in range(len(at))])
        # the parity bounds of the tests against the oracle
        assert ((O[b, h][at].double() - out).abs() <= torch.clamp_min(out.abs() * 2.0 ** -7, 2e-2)).all()
        assert ((lse[b, h][at].double() - want).abs() <= torch.clamp_min(want.abs() * 2.0 ** -20, 1e-4)).all()


def _rows(L, k, g, near=False):
    if near:   # a run of k keys round the query's own place: most tiles hold nothing for it
        first = (torch.arange(L, device="cuda") - k // 2).clamp(0, L - k)
        return (first[:, None] + torch.arange(k, device="cuda")[None]).to(torch.int32)
    edge = (torch.arange(k + 1, device="cuda") * L) // k
    width = edge[1:] - edge[:-1]
    return (edge[:-1] + (torch.rand(L, k, generator=g, device="cuda") * width).long().clamp_max(width - 1)).to(torch.int32)


# 12 heads fill the chip: those that keep L / 5 run over tiles, those that keep 9 are gathered
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,L,near", [(1, 2047, False), (2, 2177, False), (1, 4159, True), (1, 4096, False)])
def test_dense_and_gathered_heads(d, B, L, near):
    g = torch.Generator(device="cuda").manual_seed(L + d)
    ks = [L // 5, 9, L // 4, L // 5, L, 9, L // 3, L // 5, L // 4, L // 5, L // 4, L // 3]
    Q, K, V = (3 * torch.randn(B, 12, L, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    p = dsv.Problem(B, 12, L, d, 16, "bf16", ks, d ** -0.5, sorted_index=True)
    assert dsv.sparse_attn_fwd_workspace(p) > 0
    heads = [_rows(L, k, g, near) for _ in range(B) for k in ks]
    _check(p, Q, K, V, heads, torch.cat([torch.arange(0, L, 61, device="cuda"), torch.arange(L - 70, L, device="cuda")]))


def _queries_per_block(p, rows):
    """Of the launch that takes `rows` rows of all heads over tiles: 128 or 256 on sparse products, 0 on dense ones."""
    heads = [k for k in p.k_per_head if k >= dsv.dense_min_k(p, "fwd_sweep")] if dsv.dense_min_k(p, "fwd_sweep") else []
    if sum(heads) * 14 > p.L * len(heads) or len(heads) * -(-rows // 128) <= 256:
        return 0
    blocks = len(heads) * -(-rows // 256)
    return 256 if blocks * 100 >= -(-blocks // 256) * 256 * 85 else 128


# the form on sparse products, in blocks of 128 queries and of 256 (one a CU, nearly all of them), the last one whole and not, one key in 16 on
# the mean, so that groups with a third pair come; rows of neighbours leave whole tiles out and crowd others
@pytest.mark.parametrize("d,H,L,near,block", [(128, 24, 2111, False, 128), (128, 24, 2304, False, 128), (128, 24, 2304, True, 128), (128, 33, 1985, False, 256),
                                              (128, 26, 2337, True, 128), (64, 24, 4001, False, 128), (64, 16, 4096, False, 256), (64, 24, 4127, True, 128),
                                              (128, 25, 2337, False, 256), (128, 25, 2337, True, 256), (128, 25, 2559, False, 256), (64, 16, 4001, False, 256),
                                              (64, 16, 4001, True, 256)])
def test_heads_that_keep_few_pairs_of_a_tile(d, H, L, near, block):
    g = torch.Generator(device="cuda").manual_seed(3 * L + d)
    ks = [L // 16] * (H - 3) + [L // 9, L // 20, L // 13]
    Q, K, V = (3 * torch.randn(1, H, L, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    p = dsv.Problem(1, H, L, d, 16, "bf16", ks, d ** -0.5, sorted_index=True)
    assert 0 < dsv.dense_min_k(p, "fwd_sweep") <= L // 16 and _queries_per_block(p, L) == block
    heads = [_rows(L, k, g, near) for k in ks]
    _check(p, Q, K, V, heads, torch.cat([torch.arange(0, L, 97, device="cuda"), torch.arange(L - 40, L, device="cuda")]))


def test_a_call_without_scratch_gathers_where_gathers_need_none():
    L, d, ks = 2111, 128, [100] * 24  # one key in 21: over tiles for sparse products only
    g = torch.Generator(device="cuda").manual_seed(1)
    Q, K, V = (torch.randn(1, 24, L, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    p = dsv.Problem(1, 24, L, d, 16, "bf16", ks, d ** -0.5, sorted_index=True)
    idx = torch.cat([_rows(L, k, g).reshape(-1) for k in ks])
    assert dsv.sparse_attn_fwd_workspace(p) > 0
    want, want_lse = dsv.sparse_attn_fwd(p, Q, K, V, idx)
    O, lse = torch.empty_like(Q), torch.empty_like(want_lse)
    lib, stream = dsv.load_library(), torch.cuda.current_stream().cuda_stream
    assert lib.dsv_sparse_attn_fwd(p.c, *(t.data_ptr() for t in (Q, K, V, idx, O, lse)), None, 0, stream) == 0
    # both round an output to bf16 once, their sums differ by 2^-16 of sum p |v| and less
    assert ((O.float() - want.float()).abs() <= 2.0 ** -7 * want.float().abs() + 2.0 ** -9).all() and torch.allclose(lse, want_lse, atol=1e-4)


# a mask in as many rows at a time as the scratch holds: all of them beside the partial results of d = 128; pieces at d = 64, the last one no whole block,
# on dense and on sparse products
@pytest.mark.parametrize("d,L,k,pieces,block", [(128, 98309, 6000, 1, 128), (64, 98309, 20000, 2, 0), (64, 150001, 9375, 3, 128)])
def test_mask_in_pieces(d, L, k, pieces, block):
    g = torch.Generator(device="cuda").manual_seed(7)
    Q, K, V = (torch.randn(1, 1, L, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    p = dsv.Problem(1, 1, L, d, 16, "bf16", [k], d ** -0.5, sorted_index=True)
    words = -(-L // 512) * 16  # of a row; neither length leaves space between rows
    assert words % 256
    rows = min(dsv.sparse_attn_fwd_workspace(p) // (4 * words) // 128 * 128, L)
    assert dsv.dense_min_k(p, "fwd_sweep") > 0 and -(-L // rows) == pieces
    assert _queries_per_block(p, L - (pieces - 1) * rows) == block  # the last piece
    ends = [torch.arange(max(r - 20, 0), min(r + 20, L), device="cuda") for r in range(0, L, rows)] + [torch.arange(L - 20, L, device="cuda")]
    _check(p, Q, K, V, [_rows(L, k, g)], torch.cat(ends + [torch.randint(0, L, (100,), generator=g, device="cuda")]))


# one launch whose masks hold more than 2^32 words: the rows past that, the last ones of the second head
def test_masks_of_more_than_16_gigabytes():
    H, L, d = 2, 262144, 128
    k = L // 20
    g = torch.Generator(device="cuda").manual_seed(11)
    Q, K, V = (torch.randn(1, H, L, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    p = dsv.Problem(1, H, L, d, 16, "bf16", [k] * H, d ** -0.5, sorted_index=True)
    assert 0 < dsv.dense_min_k(p, "fwd_sweep") <= k
    words = H * L * (L // 32)  # without the space between rows
    assert words >= 2 ** 32 and dsv.sparse_attn_fwd_workspace(p) > 4 * words
    rows = _rows(L, k, g, near=True)
    _check(p, Q, K, V, [rows] * H, torch.cat([torch.arange(0, L, 4099, device="cuda"), torch.arange(L - 60, L, device="cuda")]))


# a value row that is not finite belongs to the queries that keep its key, and to no others
@pytest.mark.parametrize("d,bad", [(64, float("inf")), (128, float("nan"))])
def test_rows_that_are_not_finite(d, bad):
    _rows_that_are_not_finite(d, bad, 12, 2113, 400)


@pytest.mark.parametrize("d,H,L,bad,block", [(64, 24, 4096, float("nan"), 128), (128, 24, 2304, float("inf"), 128), (64, 16, 4001, float("inf"), 256),
                                             (128, 25, 2437, float("nan"), 256)])
def test_rows_that_are_not_finite_on_sparse_products(d, H, L, bad, block):
    _rows_that_are_not_finite(d, bad, H, L, L // 15, block)


def _rows_that_are_not_finite(d, bad, H, L, k, block=0):
    g = torch.Generator(device="cuda").manual_seed(d)
    Q, K, V = (torch.randn(1, H, L, d, generator=g, device="cuda").bfloat16() for _ in range(3))
    V[0, :, 700] = bad
    K[0, :, 1500] = bad
    rows = _rows(L, k, g, near=True)
    idx = torch.cat([rows.reshape(-1)] * H)
    p = dsv.Problem(1, H, L, d, 16, "bf16", [k] * H, d ** -0.5, sorted_index=True)
    assert dsv.sparse_attn_fwd_workspace(p) > 0 and _queries_per_block(p, L) == block
    O, _ = dsv.sparse_attn_fwd(p, Q, K, V, idx)
    V[0, :, 700], K[0, :, 1500] = 0, 0
    keeps = ((rows == 700) | (rows == 1500)).any(1)
    assert not O[0][:, keeps].isfinite().all(-1).any() and O[0][:, ~keeps].isfinite().all()
    want, _ = dsv.sparse_attn_fwd(p, Q, K, V, idx)
    # queries whose tiles held the row are formed once more, with probabilities of 24 instead of 8 bits: the two differ by
    # 2^-9 sum p |v| < 2^-9 max |v| and the roundings of both outputs
    a, b = O[0][:, ~keeps].float(), want[0][:, ~keeps].float()
    assert ((a - b).abs() <= 2.0 ** -9 * V.float().abs().max() + 2.0 ** -8 * b.abs()).all()
