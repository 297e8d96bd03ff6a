"""Which weight gradients share a launch, by the library's own rules called on the host: no layer whose matrices would take 3 % less together, by the time of a round
of 256 tiles that those rules weigh, runs them one by one."""
import ctypes as C

import pytest

from paper_2106_02679_amd import binding as B

SLICES, GROUP_SLICES = (B.lib[n] for n in ("_ZN3lga18gemm_splitk_slicesEiii", "_ZN3lga17gemm_group_slicesEPKiS1_ii"))
STORED, WINS = (B.lib[n] for n in ("_ZN3lga26gemm_takes_stored_operandsEiii", "_ZN3lga22gemm_stored_group_winsEPKiS1_ii"))
STORED.restype = WINS.restype = C.c_bool
STEP, FIXED, MEMORY = 1.25, 16.5, 4.5e6       # us of a round: per 64 k, around them; bytes a us of the slices' partial results


def us(matrices, slices, K):
    tiles = sum(-(-m // 256) * -(-n // 256) for m, n in matrices)
    rounds = -(-tiles * slices // 256) * (K // slices / 64 * STEP + FIXED)
    return rounds + ((slices + 1) * 4 * sum(m * n for m, n in matrices) / MEMORY if slices > 1 else 0.0)


def sizes(matrices):
    return [(C.c_int * len(matrices))(*v) for v in zip(*matrices)]


def stored_matrices(d, ff, tokens):
    """Those that are enough work alone to be read as stored; None where the others share a launch."""
    all_four = [(ff, d), (d, ff), (d, d), (d, 3 * d)]
    mine = [m for m in all_four if STORED(*m, tokens)]
    rest = [m for m in all_four if m not in mine]
    return None if len(mine) < 3 and GROUP_SLICES(*sizes(rest), len(rest), tokens) > 0 else mine


def shares(d, ff, tokens):
    mine = stored_matrices(d, ff, tokens)
    return len(mine) > 1 and WINS(*sizes(mine), len(mine), tokens)


@pytest.mark.parametrize("d,tokens", [
    (1664, 512), (1664, 896), (2304, 896), (2880, 512), (3072, 768),         # ranges of fewer than 1024 tokens are not cut, and share a launch whole
    (1152, 8192), (1280, 8704), (768, 8192), (768, 16384), (768, 32768)])    # in slices: four matrices and, at 768 x 8192, three
def test_layers_that_share_a_launch(d, tokens):
    assert shares(d, 4 * d, tokens)


@pytest.mark.parametrize("ratio", [1, 4])
def test_no_layer_that_would_gain_runs_its_matrices_apart(ratio):
    seen = 0
    for d in range(256, 4097, 64):
        for tokens in [128, 256, 512, 640, 768, 896] + [int(1024 * 1.12**i) // 8 * 8 for i in range(33)]:
            mine = stored_matrices(d, ratio * d, tokens)
            if not mine or len(mine) < 2:
                continue
            # as the launch cuts them
            slices = GROUP_SLICES(*sizes(mine), len(mine), tokens)
            together = us(mine, max(1, slices), tokens)
            apart = sum(us([m], SLICES(*m, tokens), tokens) for m in mine)
            if slices > 0 or sum(-(-m // 256) * -(-n // 256) for m, n in mine) >= 224:
                seen += 1
                assert shares(d, ratio * d, tokens) or together >= 0.97 * apart, (d, tokens, slices, together, apart)
    assert seen > 400
