"""GPU parity of the 16-bit GEMM for small problems: every tile size and number of k groups its rule chooses, ragged in m, n and
k (a k group with a partial step, and one with nothing at all to do), all epilogues, and the weight gradient with its k range in
slices.  Tolerances as for the other 16-bit GEMMs: one rounding of the result (test_gpu_ops.TOL_OUT), fp32 results 1e-5."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import to_dev, rel_err, profiled
from test_gpu_ops import check_gemm, fvec, rnd, BF16, F16

EPILOGUES = (B.LGA_EPI_STORE, B.LGA_EPI_BIAS, B.LGA_EPI_BIAS_RESID, B.LGA_EPI_BIAS_GELU, B.LGA_EPI_MUL_DGELU, B.LGA_EPI_ACCUM_F32)
SHAPES = [  # 32 x 64 tiles (weight gradients: four k groups)
          (1, 8, 8), (33, 72, 64), (33, 136, 72), (31, 64, 136), (256, 512, 328), (160, 1920, 1000),
          # 64 x 64 tiles, the two ranges below 512 and that below 768 of them (weight gradients: two groups, one)
          (700, 776, 72), (700, 776, 456), (1064, 1064, 136), (1064, 1064, 520), (1400, 1800, 264),
          # 128 x 128 tiles, up to 256 and more; rows shorter than 128 bytes
          (1700, 2056, 328), (1300, 3848, 72), (1300, 3848, 328), (2000, 2000, 40)]


@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_small_gemm_at_the_edges_of_its_tiles(shape, dt):
    for epi in EPILOGUES:
        check_gemm((dt, 1, 1, epi) + shape)


@pytest.mark.parametrize("K,N", [(200, 264), (1000, 1536)])
def test_a_row_of_the_result_does_not_depend_on_the_number_of_rows(K, N):
    """Every tile size of the small kernel and the large-tile kernel add an element's products in the same order: a bias + GELU
    GEMM over more and more rows, each prefix bit for bit the same."""
    rng = np.random.default_rng(K)
    rows = [8, 40, 520, 1600, 2600, 4200, 45000 if N < 1000 else 9000]
    A, Bm = rnd(rng, (rows[-1], K), BF16), rnd(rng, (N, K), BF16, 0.1)
    Ad, Bd, bias = to_dev(A, BF16), to_dev(Bm, BF16), fvec(rng.standard_normal(N).astype(np.float32))
    full = None
    for M in reversed(rows):
        out, out2 = torch.zeros(M, N, device="cuda", dtype=torch.bfloat16), torch.zeros(M, N, device="cuda", dtype=torch.bfloat16)
        B.check(B.lib.lga_op_gemm(BF16, 1, 1, B.LGA_EPI_BIAS_GELU, M, N, K, Ad.data_ptr(), K, Bd.data_ptr(), K, out.data_ptr(),
                                  out2.data_ptr(), None, N, bias.data_ptr(), None, 0.0, None))
        torch.cuda.synchronize()
        full = full or (out, out2)
        assert torch.equal(out, full[0][:M]) and torch.equal(out2, full[1][:M]), M


@pytest.mark.parametrize("M,N,K,beta", [(64, 192, 5000, 1.0), (128, 512, 8192, 0.0), (40, 72, 40000, 0.5), (768, 520, 4104, 1.0)])
def test_weight_gradient_of_a_narrow_layer_with_and_without_slices(M, N, K, beta):
    rng = np.random.default_rng(M + N + K)
    A, Bm = rnd(rng, (M, K + 8), BF16), rnd(rng, (N, K + 16), BF16)
    acc = A[:, :K].astype(np.float64) @ Bm[:, :K].astype(np.float64).T
    old = rng.standard_normal((M, N + 8)).astype(np.float32)
    Ad, Bd = to_dev(A, BF16), to_dev(Bm, BF16)
    ref = beta * old[:, :N].astype(np.float64) + acc
    for floats in (0, 3 * M * N, B.lib.lga_op_gemm_splitk_slices(M, N, K) * M * N):
        scratch = torch.full((floats + 16,), float("nan"), device="cuda")
        results = []
        for _ in range(2):
            outf = fvec(old)
            B.check(B.lib.lga_op_gemm_splitk(BF16, M, N, K, Ad.data_ptr(), K + 8, Bd.data_ptr(), K + 16, outf.data_ptr(), N + 8, beta,
                                             scratch.data_ptr() if floats else None, floats, None))
            torch.cuda.synchronize()
            results.append(outf.cpu().numpy())
        assert rel_err(results[0][:, :N], ref) < 1e-5, floats
        assert np.array_equal(results[0][:, N:], old[:, N:]) and np.array_equal(results[0], results[1])
        assert torch.isnan(scratch[floats:]).all()                   # nothing behind the scratch is written


@pytest.mark.parametrize("M,N,K,large", [(768, 768, 8192, False), (768, 768, 16384, True), (640, 640, 8192, False), (640, 640, 16392, True),
                                         (256, 1024, 16384, False), (256, 1024, 40008, True), (128, 512, 40008, False)])
def test_a_weight_gradient_over_a_long_k_range_leaves_the_small_tiles_in_time(M, N, K, large):
    """Few tiles: the small kernel up to 8192 k for one of its workgroups, slices of large tiles beyond."""
    rng = np.random.default_rng(M + K)
    A, Bm = rnd(rng, (M, K), BF16), rnd(rng, (N, K), BF16)
    Ad, Bd, out = to_dev(A, BF16), to_dev(Bm, BF16), torch.empty(M, N, device="cuda")
    floats = B.lib.lga_op_gemm_splitk_slices(M, N, K) * M * N
    scratch = torch.empty(floats, device="cuda")
    kernels = profiled(lambda: B.check(B.lib.lga_op_gemm_splitk(BF16, M, N, K, Ad.data_ptr(), K, Bd.data_ptr(), K, out.data_ptr(), N, 0.0,
                                                                scratch.data_ptr(), floats, None)))
    assert any(k.startswith("gemm_bf16_dma_kernel") for k in kernels) == large, kernels.keys()
    assert any(k.startswith("gemm_bf16_small_kernel") for k in kernels) != large
    assert rel_err(out.cpu().numpy(), (Ad.float() @ Bd.float().T).cpu().numpy()) < 1e-5


@pytest.mark.parametrize("M,N", [(64, 64), (768, 768), (2048, 2048), (4096, 4096)])
def test_a_weight_gradient_over_no_tokens_scales_what_is_there(M, N):
    A, out = torch.empty(max(M, N), 8, device="cuda", dtype=torch.bfloat16), torch.randn(M, N, device="cuda")
    want, scratch = 0.5 * out, torch.full((1 << 20,), float("nan"), device="cuda")
    B.check(B.lib.lga_op_gemm_splitk(BF16, M, N, 0, A.data_ptr(), 8, A.data_ptr(), 8, out.data_ptr(), N, 0.5, scratch.data_ptr(), 1 << 20, None))
    torch.cuda.synchronize()
    assert torch.equal(out, want)
