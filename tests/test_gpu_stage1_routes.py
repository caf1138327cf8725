"""Stage 1 at the edges of its routes and tiles: the index must be the stable top-k of the device's own scores (larger
score first, lower key on ties), whatever kernels an L, a k and a type lead through, and idx_t its transpose."""
from __future__ import annotations

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


# one kernel up to 2048 keys (512, 1024, 2048: 1, 2, 4 score tiles per wave), the radix passes above
@pytest.mark.parametrize("L,ks", [(1, [1, 1]), (33, [33, 1]), (512, [100, 511]), (513, [7, 64]), (1025, [1025, 200]), (2048, [1, 300]),
                                  (2049, [150, 2048])])
@pytest.mark.parametrize("dtype,d,r", [("f32", 64, 16), ("bf16", 128, 32), ("bf16", 64, 64)])
@pytest.mark.parametrize("ties", [False, True])
def test_short_sequences(L, ks, dtype, d, r, ties):
    Q, K, Wq, Wk = _inputs(2, L, d, r, dtype, ties, L + r)
    _check(dsv.Problem(1, 2, L, d, r, dtype, ks, 0.1), Q, K, Wq, Wk)
