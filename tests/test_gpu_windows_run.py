"""That the window solve runs where it is planned and the three passes where it is not (launches counted per phase: the
window solve counts as the column phase, without row passes), and its builds for fold lists of more than two entries:
both window widths, tiles of one to three rows or columns, lists up to the 2M + 2 entries of one-row tiles.

Tolerance: per round some 32 roundings reach one z, of values of size at most 2; as independent errors of at most
2 x 2^-24 with a standard deviation of 2 x 2^-24 / sqrt(3) each, three rounds give sqrt(96) x 6.9e-8 = 6.7e-7 if all are
of that size.  Most are of half that size or less; five standard deviations at half size are 1.7e-6."""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu, problem_inputs, say

pytestmark = pytest.mark.gpu
ROUNDS = 3
TOL = 1.7e-6


def solve(S, x, c, M, dtype, iters=ROUNDS):
    """z and the launches of the row DFT and the column phase."""
    K, H, W = x.shape
    pr = S.Problem(K, H, W, M, c, 1.0, 0.8, 1.1, iters)
    ws = torch.empty(S.segsalsa_str_workspace_size(pr, S._prec(dtype)), dtype=torch.uint8, device="cuda")
    z = torch.empty((K, H, W), dtype=dtype, device="cuda")
    S.segsalsa_profile_enable(True)
    try:
        S.segsalsa_profile_read(reset=True)
        S.segsalsa_str_solve(pr, x.to(dtype), z, ws)
        torch.cuda.synchronize()
        counts = {k: n for k, (_, n) in S.segsalsa_profile_read(reset=True).items()}
    finally:
        S.segsalsa_profile_enable(False)
    return z.double(), (counts["fold_row_dft"], counts["col_solve"])


def inputs(H, W, K, M, wsum, seed):
    probs, _, _, c = problem_inputs(H, W, K, M, seed=seed)
    return torch.from_numpy(probs.astype(np.float32)).cuda(), c * np.sqrt(wsum / np.sum(c ** 2))


@pytest.mark.parametrize("H,W,K,M,wsum,windows", [
    (1, 7, 2, 0, 1.0, True), (39, 40, 5, 1, 1.0, True), (64, 64, 4, 1, 1.0, True), (97, 131, 6, 3, 1.0, True),
    (64, 40, 16, 2, 0.05, True), (70, 59, 4, 1, 2.1, True), (70, 59, 4, 1, 2.6, False), (64, 64, 4, 1, 300.0, False)])
def test_where_windows_run(H, W, K, M, wsum, windows):
    S = need_gpu()
    say(f"case {H}x{W} K={K} M={M} Wsum={wsum}")
    x, c = inputs(H, W, K, M, wsum, 11)
    z, launches = solve(S, x, c, M, torch.float32)
    ref, launches64 = solve(S, x, c, M, torch.float64)
    assert launches == (0 if windows else ROUNDS, ROUNDS) and launches64 == (ROUNDS, ROUNDS)
    err = float(torch.max(torch.abs(z - ref)))
    say(f"  max |z32 - z64| = {err:.3e}")
    assert err <= (TOL if wsum <= 3 else 1e-5)


# (H, W, K, M, tile): 64-column windows, and 128-column ones (640x640, K = 16: 2048 windows of 64 columns)
NARROW = [(41, 80, 4, 2, (1, 80)), (41, 80, 4, 2, (2, 5)), (30, 47, 3, 5, (1, 8)), (90, 31, 5, 3, (7, 1)),
          (1, 70, 3, 4, (1, 3)), (17, 2, 2, 5, (3, 1)), (640, 640, 16, 2, (3, 3)), (640, 640, 16, 1, (2, 64)),
          (1300, 400, 16, 1, (1, 40))]


@pytest.mark.parametrize("H,W,K,M,tile", NARROW)
def test_narrow_tiles(H, W, K, M, tile):
    S = need_gpu()
    say(f"case {H}x{W} K={K} M={M} tiles {tile}")
    x, c = inputs(H, W, K, M, 1.0, 12)
    ref, _ = solve(S, x, c, M, torch.float64)
    try:
        S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, dict(tile_rows=tile[0], tile_cols=tile[1]))
        z, launches = solve(S, x, c, M, torch.float32)
    finally:
        S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, None)
    assert launches == (0, ROUNDS)
    err = float(torch.max(torch.abs(z - ref)))
    say(f"  max |z32 - z64| = {err:.3e}")
    assert err <= TOL


@pytest.mark.parametrize("H,W,K,M", [(37, 41, 9, 1), (37, 41, 13, 1), (64, 50, 16, 0), (33, 47, 16, 2)])
def test_one_and_two_classes_per_wavefront_to_the_bit(H, W, K, M):
    """Up to 16 classes the class sums are taken class by class, whichever wavefront holds them."""
    S = need_gpu()
    say(f"case {H}x{W} K={K} M={M}")
    x, c = inputs(H, W, K, M, 1.0, 13)
    out = []
    try:
        for kpw in (1, 2):
            S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, dict(tile_rows=8, tile_cols=8, classes_per_wave=kpw))
            out.append(solve(S, x, c, M, torch.float32)[0])
    finally:
        S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, None)
    assert torch.equal(out[0], out[1])
