"""GPU parity of the weight gradients that share a launch because a layer's matrices are not enough work one by one, or fill its rounds better: the large-tile kernel
on operands as stored, the small tiles on transposed ones, the fp32 kernel; whole and ragged tiles and k ranges, with and
without slices, accumulated over groups and micro-batches.  16-bit results against the fp32 ones of the same weights and inputs (2e-2, the
gate of 16-bit stacks), groupings against each other 1e-5 (fp32 sums in another order)."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import lga_oracle as O
import synth_inputs as S
from paper_2106_02679_amd import binding as B
from gpu_helpers import run_gpu_step, oracle_shape, rel_err, compare_with_oracle, profiled


def launches(kernels, start):
    return sum(k["launches"] for name, k in kernels.items() if name.startswith(start) and name.endswith("(grouped)"))


@pytest.mark.parametrize("d,heads,ff,s,kernel,slices", [
    (768, 12, 3072, 1024, "gemm_bf16_dma_tn_kernel", True),        # 108 tiles, 2 x 2048 tokens
    (520, 13, 2088, 1032, "gemm_bf16_dma_tn_kernel", True),        # ragged tiles and k steps: 90 tiles, 3 slices, the last of 1344
    (1304, 163, 1304, 300, "gemm_bf16_dma_tn_kernel", False),      # ragged tiles, 1200 tokens in one piece
    (2048, 16, 4104, 258, "gemm_bf16_dma_tn_kernel", False),       # 136, 136 and 192 tiles, two rounds instead of three; W_o apart
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


@pytest.mark.parametrize("d,heads,ff,s,b", [(64, 4, 256, 33, 2), (60, 3, 140, 90, 8), (30, 3, 71, 90, 8), (132, 3, 68, 300, 8)],
                         ids=["one_piece", "slices", "widths_of_no_whole_pieces", "slices_of_two_groups"])
def test_fp32_weight_gradients_in_one_launch(d, heads, ff, s, b):
    w = S.Workload("together_fp32", 1, d, heads, ff, s, b, 2, "fp32")
    x, G, params = S.make_inputs(w, seed=3, weight_std=0.1, bias_std=0.1)
    ref = O.step_microbatch_major(x, G, params, oracle_shape(w), None)
    for kw in (dict(group=1), dict(group=2), dict(order="mbmajor")):
        got = []
        kernels = profiled(lambda: got.append(run_gpu_step(w, x, G, params, retain=1, **kw)))
        assert launches(kernels, "gemm_f32_kernel") == 2 // kw.get("group", 1)
        assert launches(kernels, "gemm_f32_kernel<dma>") == (2 // kw.get("group", 1) if d % 4 == 0 and ff % 4 == 0 else 0)
        compare_with_oracle(w, got[0], ref, 1e-5, None, zero_init=False)


#        M,   N,   K: whole 16-byte pieces; steps of 32 k and tiles of 64 whole and ragged; one, two and four groups; more than 256 tiles
DIRECT = [(4, 4, 4), (64, 64, 32), (68, 60, 36), (132, 200, 64), (64, 128, 96), (60, 64, 132), (100, 1024, 260), (1090, 1088, 100),
          (1156, 1024, 288), (64, 64, 1028)]


@pytest.mark.parametrize("shape", DIRECT, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("akm,bkm,epi", [(1, 0, B.LGA_EPI_BIAS), (1, 1, B.LGA_EPI_STORE), (0, 0, B.LGA_EPI_ACCUM_F32)])
def test_fp32_operands_straight_to_lds_agree_with_the_general_kernel(akm, bkm, epi, shape):
    """The same product from operands whose rows are whole 16-byte pieces and from copies that start 4 bytes further, which the general
    kernel takes (as it does rows of 1090 weight-gradient columns either way): both within 1e-5 of exact sums (see the tolerance of the other fp32 GEMM tests); nothing outside the operands is
    used (NaN lies around them)."""
    M, N, K = shape
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    results = []
    for shift in (0, 1):
        gen.manual_seed(M + N + K)

        def operand(rows, width):
            pitch = (width + 3) // 4 * 4
            buf = torch.full((rows * pitch + 256,), float("nan"), device="cuda")
            m = buf[64 + shift:64 + shift + rows * pitch].view(rows, pitch)
            m[:, :width] = torch.randn(rows, width, device="cuda", generator=gen)
            return m, pitch, m[:, :width].double()

        a, lda, a64 = operand(*((M, K) if akm else (K, M)))
        b, ldb, b64 = operand(*((N, K) if bkm else (K, N)))
        bias = torch.randn(N, device="cuda", generator=gen)
        out = torch.zeros(M, N, device="cuda")
        want = (a64 if akm else a64.t()) @ (b64.t() if bkm else b64) + (bias.double() if epi == B.LGA_EPI_BIAS else 0.0)
        kernels = profiled(lambda: B.check(B.lib.lga_op_gemm(B.LGA_FP32, akm, bkm, epi, M, N, K, a.data_ptr(), lda, b.data_ptr(), ldb, out.data_ptr(),
                                                             None, out.data_ptr(), N, bias.data_ptr(), None, 0.0, None)))
        whole = shift == 0 and (K if akm else M) % 4 == 0 and (K if bkm else N) % 4 == 0
        assert list(kernels) == ["gemm_f32_kernel<dma>" if whole else "gemm_f32_kernel"]
        results.append(out)
        assert float((out.double() - want).norm() / want.norm()) < 1e-5
    assert float((results[0] - results[1]).norm() / results[1].norm()) < 1e-5


@pytest.mark.parametrize("dtype,d,s,widths", [
    ("bf16", 2048, 763, (5, 3)), ("fp32", 1024, 1000, (9, 7)),               # LayerNorm with a row per workgroup
    ("bf16", 768, 2047, (5, 3)), ("bf16", 512, 2049, (8, 3)),                # ... per wavefront, two packs a lane and one (and b_o once with a transpose)
    ("fp32", 512, 1025, (9, 7)), ("fp32", 256, 2049, (9, 7))], ids=["bf16", "fp32", "bf16_768", "bf16_512", "fp32_512", "fp32_256"])
def test_bias_gradients_summed_where_their_matrices_are_made(dtype, d, s, widths):
    """From 64 MB on (here two micro-batches per launch; one has it for du at most, in bf16) the second LayerNorm's backward and the GELU' product
    leave the bias gradients' first passes: the same values in other chunks, so 1e-5 between the two, over a ragged last chunk; b_2
    against the column sum of the output gradient itself."""
    w = S.Workload("sums", 1, d, 16, 4 * d, s, 8, 4, dtype)
    gen = torch.Generator(device="cuda").manual_seed(2)
    params = np.random.default_rng(2).standard_normal(w.params_per_layer).astype(np.float32) * 0.02
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, g = (torch.randn(4, 8, s, d, device="cuda", generator=gen).to(tdt) for _ in range(2))
    dx, sl, got = torch.empty_like(x), S.tensor_slices(d, 4 * d), []
    for group in (1, 2):
        st = B.Stack(B.make_config(1, d, 16, 4 * d, s, 8, 4, B.LGA_BF16 if dtype == "bf16" else B.LGA_FP32, group=group, retain_grads=1), params)
        st.forward_layered(x.data_ptr(), None)
        kernels = profiled(lambda: st.backward_layered(g.data_ptr(), dx.data_ptr(), None))
        grads = B.read_device(*st.grads(0), "float32").astype(np.float64)
        st.close()
        got.append({n: grads[sl[n]] for n in ("b_qkv", "b_o", "b_1", "b_2", "ln2_g", "ln2_b")})
        sums = [k for n, k in kernels.items() if n.startswith("colsum_partial")]
        assert sum(k["bytes"] for k in sums) == tdt.itemsize * 4 * 8 * s * d * widths[group - 1]        # what is left of 9 widths
    for name, ref in got[0].items():
        assert rel_err(got[1][name], ref) < 1e-5, name
    for run in got:
        assert rel_err(run["b_2"], g.double().sum((0, 1, 2)).cpu().numpy()) < 1e-6


class GemmParams(C.Structure):
    """The launcher's own argument (csrc/common.h), which no entry point passes through."""
    _fields_ = ([(n, C.c_void_p) for n in ("A", "B")] + [(n, C.c_int) for n in ("M", "N", "K", "lda", "ldb", "ldc")] +
                [(n, C.c_void_p) for n in ("out", "out2", "outf", "bias", "aux", "colsum")] +
                [("beta", C.c_float), ("partial", C.c_void_p), ("partial_floats", C.c_size_t), ("ksplit", C.c_int), ("kchunk", C.c_int),
                 ("batch", C.c_int), ("strideA", C.c_longlong), ("strideB", C.c_longlong), ("strideC", C.c_longlong), ("tri", C.c_int),
                 ("sblock", C.c_int)])


def test_fp32_group_keeps_to_its_scratch():
    """Outputs of odd sizes, whose partial results begin on 16-byte boundaries: with as many floats as the results alone the k range stays whole, with
    what the library asks for it is cut, and either way nothing behind the scratch is written.  Only the first product names the scratch."""
    sizes, K = [(61, 63), (63, 61), (5, 7), (65, 67)], 4000
    ints = lambda v: (C.c_int * len(v))(*v)
    M, N = ints([m for m, _ in sizes]), ints([n for _, n in sizes])
    slices = B.lib._ZN3lga21gemm_f32_group_slicesEPKiS1_ii(M, N, 4, K)
    floats_of = B.lib._ZN3lga21gemm_f32_group_floatsEPKiS1_ii
    floats_of.restype = C.c_size_t
    asked, bare = floats_of(M, N, 4, slices), slices * sum(m * n for m, n in sizes)
    assert slices > 1 and bare < asked < bare + 16
    launch = B.lib._ZN3lga21launch_gemm_f32_groupEPKNS_10GemmParamsIfEEiP12ihipStream_t
    launch.restype, launch.argtypes = None, [C.c_void_p, C.c_int, C.c_void_p]
    gen = torch.Generator(device="cuda").manual_seed(6)
    a, b = ([torch.randn(K, mn[i], device="cuda", generator=gen) for mn in sizes] for i in (0, 1))
    for floats, cut in ((asked, True), (bare, False), (asked - 1, False), (0, False)):
        scratch = torch.full((asked + 64,), float("nan"), device="cuda")
        out = [torch.zeros(m, n, device="cuda") for m, n in sizes]
        p = (GemmParams * 4)()
        for i, (m, n) in enumerate(sizes):
            p[i].A, p[i].B, p[i].outf = a[i].data_ptr(), b[i].data_ptr(), out[i].data_ptr()
            p[i].M, p[i].N, p[i].K, p[i].lda, p[i].ldb, p[i].ldc = m, n, K, m, n, n
        p[0].partial, p[0].partial_floats = scratch.data_ptr(), floats
        launch(C.addressof(p), 4, None)
        torch.cuda.synchronize()
        written = ~torch.isnan(scratch)
        assert bool(written.any()) == cut and not bool(written[floats:].any())
        for i in range(4):
            want = a[i].double().t() @ b[i].double()
            assert float((out[i].double() - want).norm() / want.norm()) < 1e-5
