"""Which tuned entries take FP32 solves off the window solve: those that the caller sets with DFT kernels named, also
through a saved cache; not measured ones, nor the entries of caches written when every solve took three passes.  The
launches are counted per phase: the window solve counts as the column phase, without row passes."""
import json

import numpy as np
import pytest
import torch

from gpu_common import need_gpu, problem_inputs, say

pytestmark = pytest.mark.gpu
H, W, K, M, ROUNDS = 40, 64, 4, 1, 3


@pytest.fixture()
def table():
    S = need_gpu()
    import os
    S.segsalsa_tuning_clear()
    yield S
    S.segsalsa_tuning_clear()
    if os.path.exists(S.DEFAULT_TUNING_CACHE):
        S.segsalsa_tuning_load(S.DEFAULT_TUNING_CACHE)


def row_launches(S, scale=1.0):
    """Row DFT launches of a solve of ROUNDS rounds whose weights have Wsum = scale ** 2."""
    probs, _, _, c = problem_inputs(H, W, K, M, seed=3)
    x = torch.from_numpy(probs.astype(np.float32)).cuda()
    pr = S.Problem(K, H, W, M, scale * c, 1.0, 0.9, 1.2, ROUNDS)
    ws = torch.empty(S.segsalsa_str_workspace_size(pr, S.SEGSALSA_FP32), dtype=torch.uint8, device="cuda")
    S.segsalsa_profile_enable(True)
    try:
        S.segsalsa_profile_read(reset=True)
        S.segsalsa_str_solve(pr, x, torch.empty_like(x), ws)
        torch.cuda.synchronize()
        counts = {k: n for k, (_, n) in S.segsalsa_profile_read(reset=True).items()}
    finally:
        S.segsalsa_profile_enable(False)
    assert counts["col_solve"] == ROUNDS and counts["fold_row_dft"] == counts["row_idft"]
    return counts["fold_row_dft"]


@pytest.mark.parametrize("entry", [dict(generic_fft=1), dict(col_dft=1), dict(generic_fft=1, col_dft=1)])
def test_entries_that_name_dft_kernels(table, entry, tmp_path):
    S = table
    say(f"case {H}x{W} K={K} M={M} {entry}")
    assert row_launches(S) == 0
    S.segsalsa_tuning_set(K, H, W, M, S.SEGSALSA_FP32, entry)
    assert row_launches(S) == ROUNDS
    path = tmp_path / "cache.json"
    S.segsalsa_tuning_save(str(path))
    S.segsalsa_tuning_clear()
    assert row_launches(S) == 0
    S.segsalsa_tuning_load(str(path))
    assert row_launches(S) == ROUNDS
    # the same entry as caches held it when there were three passes only
    old = json.loads(path.read_text())
    for e in old["entries"]:
        e.pop("three_pass")
    path.write_text(json.dumps(old))
    S.segsalsa_tuning_clear()
    assert S.segsalsa_tuning_load(str(path)) == (1, 0)
    assert S.segsalsa_tuning_get(K, H, W, M, S.SEGSALSA_FP32)[1]
    assert row_launches(S) == 0
    assert row_launches(S, 1.8) == ROUNDS   # weights beyond the windows': the entry's kernels


def test_measured_entries_do_not_switch_the_windows_off(table):
    """An entry measured for large weights, which take the three passes, whatever kernels it names."""
    S = table
    probs, _, _, c = problem_inputs(H, W, K, M, seed=3)
    x = torch.from_numpy(probs.astype(np.float32)).cuda()
    for scale in (1.8, 20.0):   # Wsum 3.2 and 400, where FP32 takes the column DFT
        pr = S.Problem(K, H, W, M, scale * c, 1.0, 0.9, 1.2, ROUNDS)
        ws = torch.empty(S.segsalsa_str_autotune_workspace_size(pr, S.SEGSALSA_FP32), dtype=torch.uint8, device="cuda")
        best = S.segsalsa_str_autotune(pr, x, torch.empty_like(x), ws, rounds=2)
        torch.cuda.synchronize()
        say(f"  Wsum {scale ** 2}: {best}")
        assert row_launches(S, scale) == ROUNDS
        assert row_launches(S) == 0
