"""The FP32 window solve's rounding error is no larger than that of the three passes over the whole image, after one
round and after many, where errors that are the same in every round have added up: root mean square over several
images of the distance to the FP64 solve of the same input, windows against a caller's entry that asks for the
three passes."""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu, problem_inputs, say

pytestmark = pytest.mark.gpu
IMAGES = 6


def solve(S, x, c, M, iters):
    K, H, W = x.shape
    pr = S.Problem(K, H, W, M, c, 1.0, 1.5, 1.5, iters)
    ws = torch.empty(S.segsalsa_str_workspace_size(pr, S._prec(x.dtype)), dtype=torch.uint8, device="cuda")
    z = torch.empty_like(x)
    S.segsalsa_str_solve(pr, x, z, ws)
    torch.cuda.synchronize()
    return z.double()


@pytest.mark.parametrize("iters", [1, 20, 60])
@pytest.mark.parametrize("H,W,K,M", [(64, 64, 4, 1), (64, 64, 8, 2), (110, 60, 11, 0), (50, 64, 5, 1), (81, 44, 3, 3)])
def test_window_rounding_is_below_three_passes(H, W, K, M, iters):
    S = need_gpu()
    err = {"windows": 0.0, "three passes": 0.0}
    c = None
    try:
        for seed in range(IMAGES):
            probs, _, _, c = problem_inputs(H, W, K, M, seed=40 + seed)
            c = c.astype(np.float32).astype(np.float64)
            x = torch.from_numpy(probs.astype(np.float32)).cuda()
            S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, None)
            ref = solve(S, x.double(), c, M, iters)
            for name in err:
                S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, dict(generic_fft=1) if name != "windows" else None)
                e = solve(S, x, c, M, iters) - ref
                err[name] += float(torch.sum(e * e) / torch.sum(ref * ref)) / IMAGES
    finally:
        S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, None)
    say(f"case {H}x{W} K={K} M={M} {iters} rounds: rms error {({k: v ** 0.5 for k, v in err.items()})}")
    assert err["windows"] <= err["three passes"]
