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


# us by gathers and over dense tiles, measured: the rule takes dense tiles where they are faster
@pytest.mark.parametrize("d,H,L,k,gathers,dense", [
    (128, 24, 1500, 187, 150, 231), (128, 12, 3000, 250, 185, 271), (128, 24, 2048, 256, 248, 341), (128, 12, 4096, 341, 332, 429),
    (128, 24, 4096, 341, 673, 821), (64, 24, 3000, 375, 292, 345), (64, 12, 3000, 375, 146, 159), (128, 6, 6000, 500, 354, 385),
    (128, 6, 21861, 1452, 4403, 3672), (128, 4, 2048, 512, 85, 58), (128, 2, 3000, 750, 95, 61), (128, 1, 8192, 1024, 164, 114), (64, 2, 4096, 1024, 90, 58),
    (128, 4, 6000, 750, 352, 263), (64, 12, 8192, 1024, 1032, 860), (128, 3, 24000, 1500, 2268, 1995), (128, 3, 24000, 1000, 1502, 1777)])
def test_dq_of_short_and_long_sequences(d, H, L, k, gathers, dense):
    assert (least(L, [k] * H, d=d)[0] > 0) == (dense < gathers)
