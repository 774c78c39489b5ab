"""A warm start may change p and the reading of g4: the state that the workspace holds is laid out by tiles that
depend on neither.  The continued solve agrees with one from the exported state, imported under the new options.

As in the forms of the kept state, the two differ in the build of the first round alone: per round at most some 32
roundings of values of size at most 2 reach one z, 3 x 32 x 2 u over three rounds (u = 2^-24 in FP32, 2^-53 in FP64)
if all were one-sided."""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu, problem_inputs, say

pytestmark = pytest.mark.gpu
ROUNDS = 3
TOL = {torch.float32: ROUNDS * 64 * 2.0 ** -24, torch.float64: ROUNDS * 64 * 2.0 ** -53}

# (H, W, K, M, dtype, (p, simplex) before, after): shapes whose tiles would differ if the planner looked at either
CASES = [(186, 442, 2, 5, torch.float64, (1.0, False), (3.0, False)),
         (186, 442, 2, 5, torch.float64, (3.0, False), (2.0, True)),
         (209, 795, 9, 1, torch.float64, (1.0, False), (1.0, True)),
         (209, 795, 9, 1, torch.float64, (1.0, True), (2.0, False)),
         (7, 9, 48, 5, torch.float32, (1.0, False), (1.5, True))]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_warm_start_with_other_options(case):
    S = need_gpu()
    H, W, K, M, dtype, (p0, s0), (p1, s1) = CASES[case]
    say(f"case {H}x{W} K={K} M={M} {dtype}: p {p0} simplex {s0} -> p {p1} simplex {s1}")
    probs, _, _, c = problem_inputs(H, W, K, M, seed=900 + case)
    x = torch.from_numpy(np.ascontiguousarray(probs)).to(device="cuda", dtype=dtype)
    first = S.Problem(K, H, W, M, c, p0, 0.9, 1.2, ROUNDS, g4_simplex=s0)
    then = S.Problem(K, H, W, M, c, p1, 0.9, 1.2, ROUNDS, warm_start=True, g4_simplex=s1)
    n = S.segsalsa_str_workspace_size(first, S._prec(dtype))
    assert n == S.segsalsa_str_workspace_size(then, S._prec(dtype))
    ws, ws2 = (torch.empty(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    z = torch.empty_like(x)
    S.segsalsa_str_solve(first, x, z, ws)
    f = lambda *s: torch.empty(*s, K, H, W, dtype=dtype, device="cuda")
    d1, d2, d3, d4 = f(), f((2 * M + 1) ** 2, 2), f(), f()
    S.segsalsa_str_state_export(first, ws, d1, d2, d3, d4)
    S.segsalsa_str_state_import(then, ws2, x / x.sum(0, keepdim=True), d1, d2, d3, d4)
    z2 = z.clone()
    S.segsalsa_str_solve(then, None, z, ws)
    S.segsalsa_str_solve(then, None, z2, ws2)
    torch.cuda.synchronize()
    err = float(torch.max(torch.abs(z.double() - z2.double())))
    say(f"  max |continued - imported| = {err:.3e}")
    assert err <= TOL[dtype]
