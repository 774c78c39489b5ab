"""Host-side contract of the planner (no GPU): which shapes and entries it accepts, and what a workspace's size and
layout may depend on."""
import ctypes

import pytest

OK, INVALID, UNSUPPORTED = 0, 1, 2


@pytest.fixture()
def S():
    from paper_1504_07028_amd import segsalsa as S
    import os
    S.lib()
    S.segsalsa_tuning_clear()
    yield S
    S.segsalsa_tuning_clear()
    if os.path.exists(S.DEFAULT_TUNING_CACHE):
        S.segsalsa_tuning_load(S.DEFAULT_TUNING_CACHE)


# Entries near the LDS limit with four classes per wavefront, on a 145 x 170 image.  Every one fits with two buffers of
# one class sum per wavefront next to the two grown-tile planes: (2 K ER EC + 12 nw 64) s + 5648 <= 163840 bytes.
LIMIT_TILES = [(9, 0, 1, 16, 64), (9, 2, 0, 48, 48), (9, 2, 1, 16, 48), (5, 3, 1, 24, 64), (9, 4, 1, 16, 32),
               (9, 5, 0, 20, 64), (9, 5, 1, 6, 48), (16, 2, 1, 16, 20)]


@pytest.mark.parametrize("K,M,prec,rows,cols", LIMIT_TILES)
def test_tiles_near_the_lds_limit_with_four_classes_per_wavefront(S, K, M, prec, rows, cols):
    size = 8 if prec else 4
    # (the 145 rows and 170 columns are cut into equal tiles of at most rows x cols)
    er, ec = (-(-n // -(-n // t)) + 2 * M + 1 for n, t in ((145, rows), (170, cols)))
    assert (2 * K * er * ec + 12 * -(-K // 4) * 64) * size + 5648 <= 160 * 1024
    S.segsalsa_tuning_set(K, 145, 170, M, prec, dict(tile_rows=rows, tile_cols=cols, classes_per_wave=4))
    plan, tuned = S.segsalsa_tuning_get(K, 145, 170, M, prec)
    assert tuned and plan["classes_per_wave"] == 4
