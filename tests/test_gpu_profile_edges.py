"""dsv_profile_sparsity where its counters and searches have edges: few keys, keys past the last whole tile, equal scores,
one key that holds the whole mass; counts against the definition in 64 bits, and the same from run to run."""
from __future__ import annotations

import pytest
import torch

import paper_2502_07590_amd as dsv

pytestmark = pytest.mark.gpu


def _counts(q, k, scale, mass):
    p = torch.softmax(q.double() @ k.double().T * scale, 1).sort(1, descending=True).values
    return ((p.cumsum(1) < mass).sum(1) + 1).clamp_max(k.shape[0]), p


@pytest.mark.parametrize("L,n", [(1, 1), (31, 5), (33, 33), (512, 31), (1000, 32), (4097, 65)])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("scale_mul", [0.0, 1.0, 40.0])   # all keys alike; ordinary; one key takes all
def test_counts_at_the_edges(L, n, dtype, d, scale_mul):
    g = torch.Generator(device="cuda").manual_seed(L + n)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K = (torch.randn(1, 2, L, d, generator=g, device="cuda").to(td) for _ in range(2))
    rows = torch.randperm(L, generator=g, device="cuda")[:n].to(torch.int32)
    p = dsv.Problem(1, 2, L, d, 16, dtype, [1, 1], scale_mul / d ** 0.5)
    sparsity, counts = dsv.profile_sparsity(p, Q, K, rows, mass=0.9)
    again = dsv.profile_sparsity(p, Q, K, rows, mass=0.9)
    assert torch.equal(counts, again[1]) and torch.equal(sparsity, again[0])
    for h in range(2):
        want, prob = _counts(Q[0, h][rows.long()], K[0, h], p.scale, 0.9)
        off = counts[h].long() - want
        # fp32 scores and normaliser: the cumulative mass is right to about 4e-6 (d * 2^-24 in the exponent, summed), so a
        # count may be off by the keys that such a mass holds where it crosses 0.9
        edge = torch.gather(prob, 1, (want[:, None] - 1)).squeeze(1)
        assert (off.abs() <= torch.ceil(8e-6 * max(1.0, scale_mul) / edge).clamp_min(1)).all()
        assert torch.isclose(sparsity[h].double(), (1 - counts[h].double() / L).mean(), atol=1e-6)


# the crossing bin: some keys (ranked in LDS), more than 512 nearly alike (divided again), more than 512 of one score
@pytest.mark.parametrize("noise", [None, 1e-3, 0.0])
def test_counts_in_crowded_bins(noise):
    L, d, n = 6000, 64, 40
    g = torch.Generator(device="cuda").manual_seed(3)
    Q = torch.randn(1, 1, L, d, generator=g, device="cuda")
    K = torch.randn(1, 1, L, d, generator=g, device="cuda")
    if noise is not None:
        K[0, 0, 100:5500] = K[0, 0, 100] + noise * torch.randn(5400, d, generator=g, device="cuda")
    rows = torch.randperm(L, generator=g, device="cuda")[:n].to(torch.int32)
    p = dsv.Problem(1, 1, L, d, 16, "f32", [1], 0.2)
    _, counts = dsv.profile_sparsity(p, Q, K, rows, mass=0.9)
    want, prob = _counts(Q[0, 0][rows.long()], K[0, 0], p.scale, 0.9)
    edge = torch.gather(prob, 1, (want[:, None] - 1)).squeeze(1)
    assert ((counts[0].long() - want).abs() <= torch.ceil(8e-6 / edge).clamp_min(1)).all()  # as above


# targets below one unit of the counters (2^-38), and of a few units: the most probable key holds that much; without ties, one
@pytest.mark.parametrize("mass", [1e-30, 1e-12, 3.6e-12, 1e-11])
@pytest.mark.parametrize("dtype,d,L", [("bf16", 128, 1000), ("f32", 64, 33), ("f32", 128, 4097)])
def test_a_tiny_mass_needs_one_key(mass, dtype, d, L):
    n = 33
    g = torch.Generator(device="cuda").manual_seed(L)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K = (torch.randn(1, 2, L, d, generator=g, device="cuda").to(td) for _ in range(2))
    rows = torch.randperm(L, generator=g, device="cuda")[:n].to(torch.int32)
    p = dsv.Problem(1, 2, L, d, 16, dtype, [1, 1], 1.0 / d ** 0.5)
    sparsity, counts = dsv.profile_sparsity(p, Q, K, rows, mass=mass)
    assert (counts == 1).all()
    assert torch.allclose(sparsity.double(), torch.full((2,), 1 - 1 / L, dtype=torch.float64, device="cuda"), atol=1e-6)


# a target next to 1, most of the keys alike and hardly probable: where the fp32 sum of all probabilities is short of the
# target, every key counts
def test_a_mass_next_to_one_counts_no_key_twice():
    L, d, n, mass = 6000, 64, 64, 1 - 2.0 ** -24
    g = torch.Generator(device="cuda").manual_seed(5)
    u = torch.nn.functional.normalize(torch.randn(d, generator=g, device="cuda"), dim=0)
    Q = (1 + torch.rand(1, 1, L, 1, generator=g, device="cuda")) * u
    K = torch.randn(1, 1, L, d, generator=g, device="cuda")
    K[0, 0, 100:5500] = -4 * u
    rows = torch.arange(n, dtype=torch.int32, device="cuda")
    p = dsv.Problem(1, 1, L, d, 16, "f32", [1], 1.0)
    _, counts = dsv.profile_sparsity(p, Q, K, rows, mass=mass)
    least, _ = _counts(Q[0, 0, :n], K[0, 0], p.scale, mass - 8e-6)  # the bound on the cumulative mass above
    assert (counts[0] <= L).all() and (counts[0] >= least).all()


# more blocks than one dimension of a grid takes (2^32 work items): the same three heads many times over
def test_many_heads_and_rows():
    B, H, L, d = 21845, 3, 4097, 64
    g = torch.Generator(device="cuda").manual_seed(5)
    K = torch.randn(1, H, L, d, generator=g, device="cuda").bfloat16()
    rows = torch.randperm(L, generator=g, device="cuda").to(torch.int32)
    want, want_counts = dsv.profile_sparsity(dsv.Problem(1, H, L, d, 16, "bf16", [1] * H, 0.3), K, K, rows)
    K = K.repeat(B, 1, 1, 1)
    sparsity, counts = dsv.profile_sparsity(dsv.Problem(B, H, L, d, 16, "bf16", [1] * H, 0.3), K, K, rows)
    assert (counts.view(B, H, L) == want_counts.view(1, H, L)).all() and (sparsity.view(B, H) == want.view(1, H)).all()
