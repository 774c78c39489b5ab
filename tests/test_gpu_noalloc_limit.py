"""segsalsa_str_solve_noalloc on problems near the size of its array: those that fit it only on other tiles than the
planner's give segsalsa_str_solve's z to rounding, and a warm start there continues whatever options it changes.

Other tiles change the order of the sums of a round: per round some 32 roundings of values of size at most 2 reach one
z, 3 x 32 x 2 u over three rounds (u = 2^-24 in FP32, 2^-53 in FP64) if all were one-sided."""
import pytest
import torch

from gpu_common import need_gpu, problem_inputs, say

pytestmark = pytest.mark.gpu
ROUNDS = 3
TOL = {torch.float32: ROUNDS * 64 * 2.0 ** -24, torch.float64: ROUNDS * 64 * 2.0 ** -53}

CASES = [(123, 170, 16, 4, torch.float32), (415, 340, 16, 1, torch.float32), (1500, 1500, 3, 0, torch.float32),
         (610, 340, 5, 1, torch.float64)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_noalloc_near_the_limit(case):
    S = need_gpu()
    H, W, K, M, dtype = CASES[case]
    simplex = dtype == torch.float64
    say(f"case noalloc {H}x{W} K={K} M={M} simplex={simplex} {dtype}")
    probs, _, _, c = problem_inputs(H, W, K, M, seed=950 + case)
    x = torch.from_numpy(probs).to(device="cuda", dtype=dtype)
    z, zw = torch.full_like(x, float("nan")), torch.empty_like(x)
    prob = lambda warm, p: S.Problem(K, H, W, M, c, p, 0.9, 1.2, ROUNDS, warm_start=warm, g4_simplex=simplex)
    ws = torch.empty(S.segsalsa_str_workspace_size(prob(False, 1.0), S._prec(dtype)), dtype=torch.uint8, device="cuda")
    for warm, p in ((False, 1.0), (True, 3.0)):
        S.segsalsa_str_solve_noalloc(prob(warm, p), None if warm else x, z)
        S.segsalsa_str_solve(prob(warm, p), None if warm else x, zw, ws)
        torch.cuda.synchronize()
        err = float(torch.max(torch.abs(z.double() - zw.double())))
        say(f"  p={p} warm={warm}: max |z_noalloc - z_solve| = {err:.3e}")
        assert err <= (1 + warm) * TOL[dtype]
