"""The reverse sweep takes everything from the bytes of the workspace that it is given: a copy of them at another
address (a workspace moved to host memory and back, say) gives the same gradients to the bit, whatever has become of
the one that the forward call was given."""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu, problem_inputs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("H,W,K,M,every", [(24, 37, 5, 1, 1), (24, 37, 5, 1, 3), (17, 64, 4, 2, 2)])
def test_backward_on_a_copied_workspace(H, W, K, M, every, dtype):
    S = need_gpu()
    say(f"case {H}x{W} K={K} M={M} checkpoint every {every} {dtype}")
    probs, _, _, c = problem_inputs(H, W, K, M, seed=H + M)
    x = torch.from_numpy(np.ascontiguousarray(probs)).to(device="cuda", dtype=dtype)
    pr = S.Problem(K, H, W, M, c, 1.0, 0.9, 1.2, 7)
    n = S.segsalsa_str_grad_workspace_size(pr, S._prec(dtype), every)
    ws, moved = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    z = torch.empty_like(x)
    S.segsalsa_str_solve_ckpt(pr, every, x, z, ws)
    moved.copy_(ws)
    gz = torch.sin(7.0 * z)

    def backward(w):
        g, gl, gw = torch.empty_like(x), *(torch.empty(k, dtype=torch.float64, device="cuda") for k in (1, len(c)))
        S.segsalsa_str_backward(pr, every, x, gz, g, w, gl, gw)
        torch.cuda.synchronize()
        return g, gl, gw

    want = backward(ws)
    ws.zero_()
    for a, b in zip(want, backward(moved)):
        assert torch.equal(a, b)
    # and the same again: a second sweep over one workspace
    for a, b in zip(want, backward(moved)):
        assert torch.equal(a, b)
