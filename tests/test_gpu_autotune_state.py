"""The autotuner's candidates run on a state that the call itself initialised, whatever the workspace held before,
and with the simplex g4 too: z_scratch holds the last candidate's z, which is the oracle's after as many rounds.
Every candidate runs one round and then `rounds` timed ones."""
import numpy as np
import pytest
import torch

from gpu_common import check_err, need_gpu, problem_inputs, rounded_input, say, weights_as_seen
from oracle import segsalsa_ref as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("simplex", [False, True], ids=["affine", "simplex"])
@pytest.mark.parametrize("H,W,K,M", [(21, 30, 5, 1), (19, 26, 17, 0)])
def test_candidates_start_from_an_initialised_state(H, W, K, M, simplex, dtype):
    S = need_gpu()
    say(f"case autotune {H}x{W} K={K} M={M} simplex={simplex} {dtype}, workspace of NaN bytes")
    probs, _, _, c = problem_inputs(H, W, K, M, seed=H + K)
    x = torch.from_numpy(probs).to(device="cuda", dtype=dtype)
    rounds = 2
    pr = S.Problem(K, H, W, M, c, 1.0, 0.9, 1.2, 10, g4_simplex=simplex)
    try:
        ws = torch.full((S.segsalsa_str_autotune_workspace_size(pr, S._prec(dtype)),), 0xFF, dtype=torch.uint8,
                        device="cuda")
        z = torch.empty_like(x)
        S.segsalsa_str_autotune(pr, x, z, ws, rounds=rounds)
        torch.cuda.synchronize()
    finally:
        S.segsalsa_tuning_set(K, H, W, M, S._prec(dtype), None)
    ref = R.Problem(weights_as_seen(c, dtype), M, 1.0, 0.9, 1.2, "simplex" if simplex else "affine")
    zo = R.solve(rounded_input(probs, dtype), ref, 1 + rounds)
    check_err(float(np.max(np.abs(z.double().cpu().numpy() - zo))), dtype)
