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


def size_and_tiles(S, K, H, W, M, prec, p, simplex, residual_every=0):
    c = [1.0 / (2 * M + 1)] * (2 * M + 1) ** 2
    pr = S.Problem(K, H, W, M, c, p, 1.0, 1.0, 5, g4_simplex=simplex, residual_every=residual_every)
    images, _ = S.image_table([(K, H, W)], [1.0], [1.0])
    plan, = S.segsalsa_str_batch_plans(images, S.BatchParams(M, c, p, 5, g4_simplex=simplex), prec)
    return S.segsalsa_str_workspace_size(pr, prec), plan["tile_rows"], plan["tile_cols"]


@pytest.mark.parametrize("tile", [None, (4, 8)], ids=["planned", "tuned"])
@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "fp64"])
@pytest.mark.parametrize("K,H,W,M", [(2, 900, 901, 0), (3, 500, 501, 1), (2, 256, 257, 1), (5, 163, 900, 1), (9, 209, 795, 1),
                                     (16, 145, 145, 2), (17, 61, 40, 0), (24, 64, 48, 1), (32, 40, 48, 1),
                                     (13, 60, 90, 3), (11, 81, 44, 4), (6, 70, 61, 5)])
def test_size_and_tiles_depend_on_shape_and_precision_only(S, K, H, W, M, prec, tile):
    """The tiles lay out the state that warm starts continue from, also with another p or reading of g4."""
    if tile:
        S.segsalsa_tuning_set(K, H, W, M, prec, dict(tile_rows=tile[0], tile_cols=tile[1]))
    plain = size_and_tiles(S, K, H, W, M, prec, 1.0, False)
    for p in (1.0, 2.0, float("inf"), 3.0):
        for simplex in (False, True):
            for every in (0, 1):
                assert size_and_tiles(S, K, H, W, M, prec, p, simplex, every) == plain, (p, simplex, every)


@pytest.mark.parametrize("K,M,prec,want", [(64, 0, 1, OK), (16, 5, 1, OK), (64, 4, 0, OK), (16, 4, 0, OK), (32, 1, 1, OK),
                                           (64, 5, 0, UNSUPPORTED), (64, 1, 1, UNSUPPORTED), (17, 2, 1, UNSUPPORTED)])
def test_shapes_accepted_depend_on_no_option(S, K, M, prec, want):
    """Class counts whose smallest tile fits LDS barely or not at all: the same for every p and reading of g4."""
    c = [1.0 / (2 * M + 1)] * (2 * M + 1) ** 2
    n = ctypes.c_size_t(0)
    for p in (1.0, 3.0):
        for g4 in (False, True):
            s = S.Problem(K, 200, 311, M, c, p, 1.0, 1.0, 5, g4_simplex=g4).c_struct()
            assert S.lib().segsalsa_str_workspace_size(ctypes.byref(s), prec, ctypes.byref(n)) == want, (p, g4)


# (K, H, W, M, precision) and the bytes of a workspace that holds p_hat, d1, d3, d4, d2, the partial sums, the spectrum
# and the previous z per class on the planner's tiles: what the per-pixel form of d1 and d4 must not add to.
SIZES = [(2, 64, 64, 0, 0, 328192), (4, 64, 64, 1, 0, 1721344), (5, 24, 37, 1, 1, 1016832), (3, 1500, 1500, 0, 0, 255102464),
         (16, 145, 145, 2, 0, 92176128), (16, 145, 145, 2, 1, 184314880), (64, 64, 64, 4, 0, 489989120),
         (9, 610, 340, 2, 0, 458544896)]


@pytest.mark.parametrize("K,H,W,M,prec,most", SIZES)
def test_workspace_bytes(S, K, H, W, M, prec, most):
    assert size_and_tiles(S, K, H, W, M, prec, 1.0, False)[0] <= most


def noalloc_status(S, K, H, W, M, prec, p, simplex):
    """UNSUPPORTED if the problem does not fit the array, else INVALID for the missing output: nothing is launched."""
    s = S.Problem(K, H, W, M, [1.0 / (2 * M + 1)] * (2 * M + 1) ** 2, p, 1.0, 1.0, 5, g4_simplex=simplex).c_struct()
    return S.lib().segsalsa_str_solve_noalloc(ctypes.byref(s), prec, None, None, None)


# Problems that fit the 256 MiB array, on the planner's tiles or only on the tiles of the smallest workspace.
FITS = [(3, 1500, 1500, 0, 0, False), (4, 900, 901, 0, 1, True), (2, 848, 2031, 0, 1, False), (4, 164, 192, 5, 1, True),
        (16, 123, 170, 4, 0, False), (16, 123, 170, 4, 0, True), (4, 300, 301, 4, 0, False), (16, 415, 340, 1, 0, False),
        (12, 686, 308, 1, 0, False), (5, 610, 340, 1, 1, True), (48, 4096, 33, 0, 0, True)]


@pytest.mark.parametrize("K,H,W,M,prec,simplex", FITS)
def test_problems_at_the_noalloc_limit(S, K, H, W, M, prec, simplex):
    for p in (1.0, 3.0):
        assert noalloc_status(S, K, H, W, M, prec, p, simplex) == INVALID
    assert noalloc_status(S, 16, 1024, 1024, 2, 0, 1.0, simplex) == UNSUPPORTED
