"""GPU parity of the weight gradients that share a launch because a layer's matrices are not enough work one by one: the large-tile kernel
on operands as stored, the small tiles on transposed ones; whole and ragged tiles and k ranges, with and
without slices, accumulated over groups and micro-batches.  16-bit results against the fp32 ones of the same weights and inputs (2e-2, the
gate of 16-bit stacks), groupings against each other 1e-5 (fp32 sums in another order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as S
from gpu_helpers import run_gpu_step, rel_err, profiled


def launches(kernels, start):
    return sum(k["launches"] for name, k in kernels.items() if name.startswith(start) and name.endswith("(grouped)"))


@pytest.mark.parametrize("d,heads,ff,s,kernel,slices", [
    (768, 12, 3072, 1024, "gemm_bf16_dma_tn_kernel", True),        # 108 tiles, 2 x 2048 tokens
    (520, 13, 2088, 1032, "gemm_bf16_dma_tn_kernel", True),        # ragged tiles and k steps: 90 tiles, 3 slices, the last of 1344
    (1304, 163, 1304, 300, "gemm_bf16_dma_tn_kernel", False),      # ragged tiles, 1200 tokens in one piece
    (128, 2, 512, 64, "gemm_bf16_small_kernel", False),            # tiles of 32 x 64, four groups
    (136, 17, 264, 1250, "gemm_bf16_small_kernel", True),          # 34 tiles of 64 x 64, 5000 tokens in slices, ragged everywhere
    (256, 4, 1024, 40, "gemm_bf16_small_kernel", False),           # 192 tiles of 64 x 64, two groups
    (320, 5, 1288, 40, "gemm_bf16_small_kernel", False),           # 312
    (512, 8, 2048, 40, "gemm_bf16_small_kernel", False)])          # 768, one group
def test_sixteen_bit_weight_gradients_in_one_launch(d, heads, ff, s, kernel, slices):
    w = S.Workload("together_bf16", 1, d, heads, ff, s, 4, 2, "bf16")
    x, G, params = S.make_inputs(w, seed=4)
    runs = []

    def step(**kw):
        kernels = profiled(lambda: runs.append(run_gpu_step(w, x, G, params, retain=1, **kw)))
        return launches(kernels, kernel), "splitk_reduce_kernel" in kernels

    assert step(wgrad_groups=1) == (2, slices)
    assert step(order="mbmajor") == (2, slices)
    step(wgrad_groups=2)
    exact = run_gpu_step(S.Workload("together_fp32", 1, d, heads, ff, s, 4, 2, "fp32"), x, G, params, retain=1)
    for got in runs[1:]:
        assert np.array_equal(got["dx"], runs[0]["dx"]) and np.array_equal(got["boundaries"], runs[0]["boundaries"])
        assert rel_err(got["grads"][0], runs[0]["grads"][0]) < 1e-5
    for name, sl in S.tensor_slices(d, ff).items():
        assert rel_err(runs[0]["grads"][0][sl], exact["grads"][0][sl]) < 2e-2, name
