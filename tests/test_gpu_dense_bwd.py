"""Backward over dense tiles with a selection mask: heads that keep enough of their keys, against the same sums in fp64."""
import pytest
import torch

import paper_2502_07590_amd as dsv

pytestmark = pytest.mark.gpu


def problem(L, d, ks, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    H = len(ks)
    Q, K, V, dO = (torch.randn(1, H, L, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    rows, lists, ptrs = [], [], []
    for h, k in enumerate(ks):
        # a slope over the keys, so that some lists are several times as long as others
        score = torch.rand(L, L, generator=g, device="cuda") + torch.linspace(0, 0.2, L, device="cuda")
        row = score.topk(k, dim=1).indices.sort(dim=1).values.to(torch.int32)
        rows.append(row)
        keys = row.reshape(-1)
        lists.append((torch.sort(keys, stable=True).indices // k).to(torch.int32))
        ptr = torch.zeros(L + 1, dtype=torch.int64, device="cuda")
        ptr[1:] = torch.bincount(keys, minlength=L).cumsum(0)
        ptrs.append(ptr)
    p = dsv.Problem(1, H, L, d, 16, "bf16", ks, 2.0 / d ** 0.5, sorted_index=True)
    return p, Q, K, V, dO, rows, torch.cat(lists), torch.stack(ptrs)


def reference(p, Q, K, V, dO, rows, h):
    q, k, v, g = (t[0, h].double() for t in (Q, K, V, dO))
    keep = torch.zeros(p.L, p.L, dtype=torch.bool, device="cuda").scatter_(1, rows[h].long(), True)
    s = (q @ k.T * p.scale).masked_fill(~keep, float("-inf"))
    lse = torch.logsumexp(s, dim=1)
    w = torch.exp(s - lse[:, None])
    dp = (g @ v.T).masked_fill(~keep, 0.0)
    ds = w * (dp - (w * dp).sum(1, keepdim=True))
    return w @ v, lse, ds @ k * p.scale, ds.T @ q * p.scale, w.T @ g, keep


def backward(p, Q, K, V, dO, rows, lists, ptrs, refs):
    O = torch.stack([r[0] for r in refs])[None].to(torch.bfloat16)
    lse = torch.stack([r[1] for r in refs])[None].float()
    # heads that keep an eighth of their keys and more run over dense tiles in both steps, sparse ones gather in the dkdv step
    # (in the dq step their tiles can be cheaper than a launch of their own)
    least = [dsv.dense_min_k(p, step) for step in ("dq_sweep", "dkdv_sweep")]
    for k in p.k_per_head:
        assert (k >= least[0] > 0 and k >= least[1] > 0) if 8 * k >= p.L else k < least[1], (k, least)
    return dsv.sparse_attn_bwd_t(p, Q, K, V, torch.cat([r.reshape(-1) for r in rows]), lists, ptrs, O, lse, dO)


# L around tiles of 32, blocks of 128 and ranges; groups of four with one to four pairs (k = L); heads by gathers beside dense ones
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,ks", [(2977, (2977,)), (2048, (1024, 512, 1500)), (2081, (1900, 60, 1700, 1)), (4100, (2050, 1640))])
def test_backward_over_dense_tiles(L, d, ks):
    p, Q, K, V, dO, rows, lists, ptrs = problem(L, d, list(ks))
    refs = [reference(p, Q, K, V, dO, rows, h) for h in range(len(ks))]
    got = backward(p, Q, K, V, dO, rows, lists, ptrs, refs)
    for name, t, at in zip(("dQ", "dK", "dV"), got, (2, 3, 4)):
        for h, ref in enumerate(refs):
            want, err = ref[at], t[0, h].double() - ref[at]
            # the rounding of the output is 2^-9 of an element at most; the weights' 16 bits and fp32 sums stay far below it,
            # except where a row's terms nearly cancel (a part of the typical row is allowed for that).  k = 1: dQ and dK are zero, and
            # fp32 leaves 2^-20 of dP (below 50) there, times a row of norm 8 to 11 and the scale of 0.25 to 0.18: below 1.4e-4
            size = want.norm(dim=1)
            assert (err.norm(dim=1) <= 2 ** -8 * size + 2 ** -10 * size.mean() + 1.4e-4).all(), (name, h)


@pytest.mark.parametrize("L,d,ks", [(2048, 128, [1200, 1000]), (3000, 64, [1800, 1500])])
@pytest.mark.parametrize("where", ["Q", "K", "V", "dO"])
def test_rows_that_are_not_finite_reach_only_those_that_select_them(L, d, ks, where):
    """Every sum of a dense tile has zero weights on rows that were not selected, and zero times no number is none."""
    p, Q, K, V, dO, rows, lists, ptrs = problem(L, d, ks)
    refs = [reference(p, Q, K, V, dO, rows, h) for h in range(2)]
    r = [777, 1027, L - 1]  # one row at the end of a tile, two beside finite ones
    for bad, x in zip(r, (float("inf"), float("nan"), float("-inf"))):
        dict(Q=Q, K=K, V=V, dO=dO)[where][0, :, bad, 5] = x
    dQ, dK, dV = backward(p, Q, K, V, dO, rows, lists, ptrs, refs)
    for h, ref in enumerate(refs):
        keep = ref[5]
        mine = torch.ones(L, dtype=torch.bool, device="cuda")
        mine[r] = False
        if where in ("K", "V"):  # queries that select one of these keys, through Delta all keys of such queries; dV has no V in it
            hit = keep[:, r].any(1)
            fine = [~hit, ~keep[hit].any(0), mine if where == "K" else mine | True]
        else:                    # these queries themselves, and the keys that they select
            fine = [mine, ~keep[r].any(0), ~keep[r].any(0)]
        for name, got, want, ok in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref[2:5], fine):
            if name == "dK" and where in ("K", "V") and not ok.any():
                continue
            assert ok.any()
            assert torch.isfinite(got[0, h][ok]).all(), (name, h)
            assert (got[0, h].double() - want)[ok].norm() / want[ok].norm() < 4e-3, (name, h)  # twice the rounding of the output
        broken = dQ[0, h][~fine[0]]
        assert not torch.isfinite(broken).all(1).any()


# K and V rows of 3.2 MB: rows sorted first; 0.4 MB and 1 MB: not (dkdv over dense tiles all the same, and by gathers beside them)
@pytest.mark.parametrize("L,d,ks", [(6201, 128, [150, 1300, 1000]), (1500, 64, [1400] * 6), (4100, 64, [2050, 40, 1640])])
def test_whole_backward_is_that_of_its_steps(L, d, ks):
    """The whole backward, which builds the lists itself, bit for bit against the steps on the same lists, with the flag and on
    rows in any order without it; and the latter against ascending rows."""
    p, Q, K, V, dO, rows, lists, ptrs = problem(L, d, ks)
    refs = [reference(p, Q, K, V, dO, rows, h)[:2] for h in range(len(ks))]
    want = backward(p, Q, K, V, dO, rows, lists, ptrs, refs)
    O = torch.stack([r[0] for r in refs])[None].to(torch.bfloat16)
    lse = torch.stack([r[1] for r in refs])[None].float()
    idx = torch.cat([r.reshape(-1) for r in rows])
    for _ in range(2):
        for a, b in zip(dsv.sparse_attn_bwd(p, Q, K, V, idx, O, lse, dO), want):
            assert torch.equal(a, b)
    loose = dsv.Problem(1, len(ks), L, d, 16, "bf16", ks, p.scale)
    turned = torch.cat([r.flip(1).reshape(-1) for r in rows])
    got = dsv.sparse_attn_bwd(loose, Q, K, V, turned, O, lse, dO)
    for a, b in zip(got, want):
        assert (a - b).double().norm() / b.double().norm() < 2 ** -8  # two results within half a unit each
    if L * 4 * d <= 3 << 20:
        dQ, delta = dsv.sparse_attn_bwd_dq(loose, Q, K, V, turned, O, lse, dO)
        want = [dQ, *dsv.sparse_attn_bwd_dkdv(p, Q, K, V, lists, ptrs, lse, delta, dO)]
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_a_call_without_scratch_gathers_where_gathers_need_none():
    """L = 2048, d = 64: nothing is cut in ranges, so a null workspace is accepted, and one that holds no partial results."""
    L, d, ks = 2048, 64, [1024, 512, 1500]
    p, Q, K, V, dO, rows, lists, ptrs = problem(L, d, ks)
    refs = [reference(p, Q, K, V, dO, rows, h) for h in range(3)]
    want = backward(p, Q, K, V, dO, rows, lists, ptrs, refs)
    O = torch.stack([r[0] for r in refs])[None].to(torch.bfloat16)
    lse = torch.stack([r[1] for r in refs])[None].float()
    idx = torch.cat([r.reshape(-1) for r in rows])
    lib, stream = dsv.load_library(), torch.cuda.current_stream().cuda_stream
    assert dsv.sparse_attn_bwd_dq_workspace(p) > 0
    dQ, dK, dV = (torch.empty_like(Q) for _ in range(3))
    delta = torch.empty_like(lse)
    at = [t.data_ptr() for t in (Q, K, V, idx, O, lse, dO, dQ, delta)]
    assert lib.dsv_sparse_attn_bwd_dq(p.c, *at, None, 0, stream) == 0
    at = [t.data_ptr() for t in (Q, K, V, lists, ptrs, lse, delta, dO, dK, dV)]
    assert lib.dsv_sparse_attn_bwd_dkdv(p.c, *at, None, 0, stream) == 0
    # Delta alone, then the whole backward with all but the steps' scratch
    small = torch.empty(-(-3 * L * 4 // 256) * 256, dtype=torch.uint8, device="cuda")
    whole = torch.empty(dsv.sparse_attn_bwd_workspace(p) - dsv.sparse_attn_bwd_dq_workspace(p), dtype=torch.uint8, device="cuda")
    calls = [(dQ, dK, dV), dsv.sparse_attn_bwd_t(p, Q, K, V, idx, lists, ptrs, O, lse, dO, workspace=small),
             dsv.sparse_attn_bwd(p, Q, K, V, idx, O, lse, dO, workspace=whole)]
    for got in calls:
        for a, b in zip(got, want):
            assert (a - b).double().norm() / b.double().norm() < 2 ** -8  # two results within half a unit each
        for a, b in zip(got, calls[0]):
            assert torch.equal(a, b)  # the same gathers
    with pytest.raises(dsv.DsvError):
        dsv.sparse_attn_bwd_t(p, Q, K, V, idx, lists, ptrs, O, lse, dO, workspace=small[:-256])


def test_masks_of_several_heads_at_a_time():
    """12 heads of 16384: masks of 402 MB go through scratch three heads at a time; of 6 heads they are whole.  The same bits."""
    L, d, H, k = 16384, 64, 12, 2048
    p, Q, K, V, dO, rows, lists, ptrs = problem(L, d, [k] * H)
    refs = [reference(p, Q, K, V, dO, rows, h)[:2] for h in range(H)]
    got = backward(p, Q, K, V, dO, rows, lists, ptrs, refs)
    for a in (0, 6):
        s = slice(a, a + 6)
        half = dsv.Problem(1, 6, L, d, 16, "bf16", [k] * 6, p.scale, sorted_index=True)
        want = backward(half, *(t[:, s].contiguous() for t in (Q, K, V, dO)), rows[s], lists[a * L * k:(a + 6) * L * k], ptrs[s], refs[s])
        for x, y in zip(got, want):
            assert torch.equal(x[:, s], y)
    for t, want in zip(got, reference(p, Q, K, V, dO, rows, 4)[2:5]):
        assert (t[0, 4].double() - want).norm() / want.norm() < 4e-3  # twice the rounding of the output


@pytest.mark.parametrize("scale", [1e-31, 2e-30])
def test_scales_on_either_side_of_the_least_one(scale):
    """The key-major tiles start from lse / scale: not below 1e-30.  All keys weigh the same here."""
    L, d, ks = 2048, 128, [1200, 1000]
    p, Q, K, V, dO, rows, lists, ptrs = problem(L, d, ks)
    tiny = dsv.Problem(1, 2, L, d, 16, "bf16", ks, scale, sorted_index=True)
    assert (dsv.dense_min_k(tiny, "dkdv_sweep") > 0) == (scale > 1e-30)
    refs = [reference(tiny, Q, K, V, dO, rows, h) for h in range(2)]
    O = torch.stack([r[0] for r in refs])[None].to(torch.bfloat16)
    lse = torch.stack([r[1] for r in refs])[None].float()
    got = dsv.sparse_attn_bwd_t(tiny, Q, K, V, torch.cat([r.reshape(-1) for r in rows]), lists, ptrs, O, lse, dO)
    for t, at in zip(got, (2, 3, 4)):
        for h, ref in enumerate(refs):
            assert (t[0, h].double() - ref[at]).norm() / ref[at].norm() < 4e-3  # twice the rounding of the output
