"""Which heads run a backward step over dense tiles: host arithmetic, queried through dsv_dense_min_k."""
import pytest

import paper_2502_07590_amd as dsv

STEPS = ("dq_sweep", "dkdv_sweep")


def least(L, ks, d=128, dtype="bf16", scale=None, sorted_index=True, B=1):
    p = dsv.Problem(B, len(ks), L, d, 16, dtype, ks, 2.0 / d ** 0.5 if scale is None else scale, sorted_index=sorted_index)
    return [dsv.dense_min_k(p, s) for s in STEPS]


def test_dense_tiles_need_ascending_bf16_rows_and_a_scale_to_divide_by():
    ks = [2028, 4056]
    assert least(20280, ks) == [2028, 2028]
    assert least(20280, ks, sorted_index=False) == [0, 0]
    assert least(20280, ks, dtype="f32") == [0, 0]
    # the key-major tiles start from lse / scale
    for scale in (0.0, -0.1, 1e-31, float("nan")):
        assert least(20280, ks, scale=scale) == [0, 0], scale
    assert least(20280, ks, scale=2e-30) == [2028, 2028]
    p = dsv.Problem(1, 2, 20280, 128, 16, "bf16", ks, 0.1, sorted_index=True)
    lib = dsv.load_library()
    assert lib.dsv_dense_min_k(p.c, -1) == 0 and lib.dsv_dense_min_k(p.c, 3) == 0 and lib.dsv_dense_min_k(None, 1) == 0


@pytest.mark.parametrize("L,ks,want", [(32768, [2048] * 4, [2048, 0]), (20280, [507, 1014, 2028, 4056], [2028, 2028]), (131072, [8192], [8192, 0]),
                                       (524288, [16384] * 2, [0, 0])])
def test_heads_of_long_sequences(L, ks, want):
    assert least(L, ks) == want
