"""GPU parity of the fp32 GEMM at the edges of its 64 x 64 tiles and 32-k steps, in all four operand layouts, with leading
dimensions and bases that take 16-byte accesses and such that do not, through one, two and four k groups per workgroup
and through slices of the k range.  Gate 1e-5: sums of at most 4096 fp32 products of N(0, 1) values (unit roundoff 6e-8, error
growing as the root of the chain length: below 1e-6 measured on such sums)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import lga_oracle as O
import synth_inputs as S
from paper_2106_02679_amd import binding as B
from gpu_helpers import rel_err, run_gpu_step, oracle_shape, oracle_adam, adam_struct, compare_with_oracle

#        M,    N,    K: k groups 1 (K <= 32 or >= 512 tiles), 2 (K <= 64), 4
SHAPES = [(1, 1, 1), (63, 65, 31), (64, 64, 32), (65, 63, 33), (33, 130, 64), (64, 64, 65), (130, 31, 129), (7, 200, 500),
          (64, 192, 256), (1600, 1500, 70), (128, 64, 0)]


def dev(a, shift):
    """A device copy of `a` whose first element lies `shift` floats behind a 256-byte boundary."""
    t = torch.empty(a.size + 8, device="cuda")
    v = t[shift:shift + a.size]
    v.copy_(torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().reshape(-1))
    return t, v


@pytest.mark.parametrize("akm,bkm", [(1, 0), (1, 1), (0, 0), (0, 1)])
@pytest.mark.parametrize("pad,shift", [(0, 0), (4, 0), (1, 0), (4, 1)])
def test_fp32_gemm_at_tile_edges(akm, bkm, pad, shift):
    for M, N, K in SHAPES:
        rng = np.random.default_rng(M * 7 + N * 3 + K)
        lda, ldb, ldc = (K if akm else M) + pad, (K if bkm else N) + pad, N + pad
        A = rng.standard_normal((M if akm else K, lda)).astype(np.float32)
        Bm = rng.standard_normal((N if bkm else K, ldb)).astype(np.float32)
        a = A[:, :K] if akm else A[:, :M].T
        b = Bm[:, :K].T if bkm else Bm[:, :N]
        acc = a.astype(np.float64) @ b.astype(np.float64)
        bias, aux = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, ldc)).astype(np.float32)
        old = rng.standard_normal((M, ldc)).astype(np.float32)
        (_, Ad), (_, Bd), (_, biasd), (_, auxd) = dev(A, shift), dev(Bm, shift), dev(bias, shift), dev(aux, shift)
        a64 = aux[:, :N].astype(np.float64)
        for epi in (B.LGA_EPI_STORE, B.LGA_EPI_BIAS, B.LGA_EPI_BIAS_RESID, B.LGA_EPI_BIAS_GELU, B.LGA_EPI_MUL_DGELU, B.LGA_EPI_ACCUM_F32):
            (_, out), (_, out2) = dev(old, shift), dev(old, shift)
            beta = 0.5 if epi == B.LGA_EPI_ACCUM_F32 else 0.0
            B.check(B.lib.lga_op_gemm(B.LGA_FP32, akm, bkm, epi, M, N, K, Ad.data_ptr(), lda, Bd.data_ptr(), ldb, out.data_ptr(),
                                      out2.data_ptr(), out.data_ptr(), ldc, biasd.data_ptr(), auxd.data_ptr(), beta, None))
            torch.cuda.synchronize()
            want = {B.LGA_EPI_STORE: acc, B.LGA_EPI_BIAS: acc + bias, B.LGA_EPI_BIAS_RESID: acc + bias + a64,
                    B.LGA_EPI_BIAS_GELU: O.gelu(acc + bias), B.LGA_EPI_MUL_DGELU: acc * O.gelu_grad(a64),
                    B.LGA_EPI_ACCUM_F32: 0.5 * old[:, :N].astype(np.float64) + acc}[epi]
            got = out.cpu().numpy().reshape(M, ldc)
            assert rel_err(got[:, :N], want) < 1e-5, (M, N, K, epi)
            assert np.array_equal(got[:, N:], old[:, N:]), (M, N, K, epi)              # padding untouched
            if epi == B.LGA_EPI_BIAS_GELU:
                assert rel_err(out2.cpu().numpy().reshape(M, ldc)[:, :N], acc + bias) < 1e-5, (M, N, K)


@pytest.mark.parametrize("d,heads,ff,group", [(60, 3, 140, 4), (64, 2, 256, 2), (30, 3, 70, 1)])
def test_fp32_stack_with_weight_gradients_over_slices_of_the_tokens(d, heads, ff, group):
    """Enough tokens per group that the weight gradients' k range is cut into slices (5, 2 and 1 of them), accumulated over
    groups, against the oracle; twice, bit for bit."""
    w = S.Workload("fp32_slices", 1, d, heads, ff, 90, 4, 4, "fp32")
    x, G, params = S.make_inputs(w, seed=3, weight_std=0.1, bias_std=0.1)
    adam = adam_struct(lr=1e-2, step=2)
    ref = O.step_microbatch_major(x, G, params, oracle_shape(w), oracle_adam(adam))
    got = [run_gpu_step(w, x, G, params, group=group, retain=1, adam=adam) for _ in range(2)]
    compare_with_oracle(w, got[0], ref, 1e-5, adam, zero_init=False)
    assert np.array_equal(got[0]["grads"][0], got[1]["grads"][0])


@pytest.mark.parametrize("K", [1, 32, 33, 64, 65, 96, 100, 129, 160, 1000, 1024])
def test_a_row_of_the_result_does_not_depend_on_the_number_of_rows(K):
    """More and more rows, on both sides of the 512 tiles from which on one group of wavefronts has the whole k range: each prefix bit for
    bit the same."""
    N, rows = 1030, (1, 64, 500, 1900, 2000)                      # 17 tiles across, 31 and 32 down
    rng = np.random.default_rng(K)
    A, Bm = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda() for s in ((rows[-1], K), (K, N)))
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).cuda()
    full = None
    for M in reversed(rows):
        out, out2 = torch.zeros(M, N, device="cuda"), torch.zeros(M, N, device="cuda")
        B.check(B.lib.lga_op_gemm(B.LGA_FP32, 1, 0, B.LGA_EPI_BIAS_GELU, M, N, K, A.data_ptr(), K, Bm.data_ptr(), N, out.data_ptr(),
                                  out2.data_ptr(), None, N, bias.data_ptr(), None, 0.0, None))
        torch.cuda.synchronize()
        full = full or (out, out2)
        assert torch.equal(out, full[0][:M]) and torch.equal(out2, full[1][:M]), M


def test_fp32_orders_and_group_sizes_agree_bit_for_bit():
    """The size of the paper's X_16 as its encoder: the first feed-forward GEMM has 512, 256 and 128 tiles at groups of 4, 2 and 1
    micro-batches."""
    w = S.Workload("fp32_groups", 1, 256, 8, 1024, 256, 2, 4, "fp32")
    x, G, params = S.make_inputs(w, seed=5)
    runs = [run_gpu_step(w, x, G, params, group=g, retain=1, attention=B.LGA_ATTN_FULL) for g in (1, 2, 4)]
    runs.append(run_gpu_step(w, x, G, params, retain=1, order="mbmajor", attention=B.LGA_ATTN_FULL))
    for got in runs[1:]:
        assert np.array_equal(got["boundaries"], runs[0]["boundaries"]) and np.array_equal(got["dx"], runs[0]["dx"])
        assert rel_err(got["grads"][0], runs[0]["grads"][0]) < 1e-5
