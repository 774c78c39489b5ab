"""9x9 and 11x11 patches, whose kernel loads each pair of the J-split multipliers a few offsets ahead of its use, with
one, two and four classes per wavefront, plain, with residuals and with the simplex g4, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_common import check_err, need_gpu, problem_inputs, rounded_input, say, weights_as_seen
from oracle import segsalsa_ref as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("kpw", [1, 2, 4])
@pytest.mark.parametrize("variant", ["plain", "residuals", "simplex"])
@pytest.mark.parametrize("H,W,K,M", [(13, 17, 5, 4), (12, 14, 3, 5)])
def test_large_patches_match_oracle(H, W, K, M, variant, kpw, dtype):
    S = need_gpu()
    say(f"case {H}x{W} K={K} M={M} {variant} {kpw} classes per wavefront {dtype}")
    probs, _, _, c = problem_inputs(H, W, K, M, seed=H + W + K)
    x = torch.from_numpy(np.ascontiguousarray(probs)).to(device="cuda", dtype=dtype)
    simplex, iters = variant == "simplex", 3
    pr = S.Problem(K, H, W, M, c, 1.0, 0.8, 1.1, iters, g4_simplex=simplex, residual_every=int(variant == "residuals"))
    try:
        S.segsalsa_tuning_set(K, H, W, M, S._prec(dtype), dict(classes_per_wave=kpw))
        ws = torch.empty(S.segsalsa_str_workspace_size(pr, S._prec(dtype)), dtype=torch.uint8, device="cuda")
        z = torch.empty_like(x)
        S.segsalsa_str_solve(pr, x, z, ws, stats=variant == "residuals")
        torch.cuda.synchronize()
    finally:
        S.segsalsa_tuning_set(K, H, W, M, S._prec(dtype), None)
    ref = R.Problem(weights_as_seen(c, dtype), M, 1.0, 0.8, 1.1, "simplex" if simplex else "affine")
    zo = R.solve(rounded_input(probs, dtype), ref, iters)
    err = float(np.max(np.abs(z.double().cpu().numpy() - zo)))
    say(f"  max |z_gpu - z_oracle| = {err:.3e}")
    check_err(err, dtype)
