"""GPU parity of the weight gradient that takes its operands as stored (both contiguous along the output's dimensions): the large-tile
kernel at its edges, and a stack whose merged weight gradients keep several groups' activations and gradients for it.  Tolerances as
for the other 16-bit GEMMs (fp32 results 1e-5) and stacks (2e-2 against exact arithmetic, 1e-5 between ways of merging)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import lga_oracle as O
import synth_inputs as S
from paper_2106_02679_amd import binding as B
from gpu_helpers import run_gpu_step, oracle_shape, rel_err, compare_with_oracle, profiled
from test_gpu_ops import check_gemm, BF16, F16

SHAPES = [  # at least 128 tiles of 256 x 256, whole and ragged; k of one, two and three steps of 64, and of the unrolled loop's lengths
          (2056, 4104, 8), (2056, 4104, 64), (2056, 4104, 72), (2840, 2840, 136), (2840, 2840, 200), (264, 33000, 456), (4096, 4096, 520),
          (2304, 4096, 1031), (2840, 2856, 704),
          # leading dimensions below 256, and fewer tiles: the kernels for other layouts
          (96, 66000, 72), (1000, 1000, 333)]


@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_weight_gradient_of_operands_as_stored(shape, dt):
    check_gemm((dt, 0, 0, B.LGA_EPI_ACCUM_F32) + shape)


@pytest.mark.parametrize("overlap", [0, B.LGA_OVERLAP_ADAM])
def test_stack_whose_weight_gradients_take_stored_operands(overlap):
    """W_1 and W_2 on the large-tile kernel, W_o and W_qkv on transposed copies; five groups in merged GEMMs of 1, 2 (a ragged last
    one), 3 and 5, over two layers, so that the ring of activation gradients wraps."""
    w = S.Workload("stored_bf16", 2, 1536, 12, 6144, 40, 1, 5, "bf16")
    x, G, params = S.make_inputs(w, seed=3)
    ref = O.step_microbatch_major(x, G, params, oracle_shape(w), None)
    runs = [run_gpu_step(w, x, G, params, retain=1, wgrad_groups=wb, overlap=overlap) for wb in (1, 2, 3, 5)]
    compare_with_oracle(w, runs[0], ref, 2e-2, None)
    runs.append(run_gpu_step(w, x, G, params, retain=1, order="mbmajor", overlap=overlap))
    for got in runs[1:]:
        assert np.array_equal(got["dx"], runs[0]["dx"]) and np.array_equal(got["boundaries"], runs[0]["boundaries"])
        for l in range(w.n_layers):
            assert rel_err(got["grads"][l], runs[0]["grads"][l]) < 1e-5


@pytest.mark.parametrize("d,heads,ff,expected", [
    # launches of one matrix's slices, of several matrices' slices, and sums of slices: two groups in turn, merged, one group of both, micro-batches in turn.
    # Three matrices of either 8200 tokens in two slices of 4160 (the last 4040) in one launch, W_o on small tiles from transposed copies (over 16400 in
    # slices of large tiles); all four over 16400 in two of 8256 (8144)
    (768, 12, 3072, [(0, 2, 2), (0, 1, 2), (0, 1, 1), (0, 2, 2)]),
    # ragged tiles: three in slices of 2752 (2696) and, over 16400, four of 5504 (5392)
    (776, 97, 3080, [(0, 2, 2), (0, 1, 2), (0, 1, 1), (0, 2, 2)]),
    # W_qkv alone in 8 of 1088 (584), the other three in one launch
    (768, 12, 768, [(2, 2, 4), (1, 1, 2), (0, 1, 1), (2, 2, 4)]),
    # W_qkv alone in 6 of 1408 (1160) on ragged tiles, the others on transposed copies (merged, W_o in slices of large tiles and W_1, W_2 of small ones);
    # over 16400 W_o and W_qkv in four of 4160 (3920)
    (776, 97, 128, [(2, 0, 2), (1, 0, 3), (0, 1, 2), (2, 0, 2)])])
def test_narrow_stack_whose_weight_gradients_take_stored_operands_in_slices(d, heads, ff, expected):
    """The few output tiles of a narrow layer, their k range in slices, the last of them no whole number of steps.
    The slices cut the tokens elsewhere in every grouping, so that a token left out or taken twice would show."""
    w = S.Workload("stored_slices_bf16", 1, d, heads, ff, 1025, 8, 2, "bf16")
    x, G, params = S.make_inputs(w, seed=4)
    runs = []

    def step(**kw):
        kernels = profiled(lambda: runs.append(run_gpu_step(w, x, G, params, retain=1, **kw)))
        sliced = {n: k["launches"] for n, k in kernels.items() if n.startswith("gemm_bf16_dma_tn_kernel")}
        together = sum(k for n, k in sliced.items() if n.endswith("(grouped)"))
        return sum(sliced.values()) - together, together, kernels["splitk_reduce_kernel"]["launches"] if "splitk_reduce_kernel" in kernels else 0

    assert [step(wgrad_groups=1), step(wgrad_groups=2), step(group=2), step(order="mbmajor")] == expected
    exact = run_gpu_step(S.Workload("stored_slices_fp32", 1, d, heads, ff, 1025, 8, 2, "fp32"), x, G, params, retain=1)
    for got in runs[1:]:
        assert np.array_equal(got["dx"], runs[0]["dx"]) and np.array_equal(got["boundaries"], runs[0]["boundaries"])
        assert rel_err(got["grads"][0], runs[0]["grads"][0]) < 1e-5
    for name, sl in S.tensor_slices(w.d_model, w.d_ff).items():
        assert rel_err(runs[0]["grads"][0][sl], exact["grads"][0][sl]) < 2e-2, name


@pytest.mark.parametrize("d,heads,ff", [(1536, 12, 6144), (128, 2, 512)], ids=["ring", "in_place"])
@pytest.mark.parametrize("layers", [1, 2])
def test_gradient_buffers_that_overlap_or_are_misaligned(d, heads, ff, layers):
    """The sweep reads dy and writes dx without copies where it can: dx in dy's place, shifted against it, and both at 8 bytes past
    an aligned address give the same bits as buffers of their own; so does one layer's call."""
    n_micro, s, shift = 5, 40, 4
    params = [np.random.default_rng(l).standard_normal(B.params_per_layer(B.make_config(1, d, heads, ff, s, 1, n_micro, BF16))).astype(np.float32)
              * 0.02 for l in range(layers)]
    st = B.Stack(B.make_config(layers, d, heads, ff, s, 1, n_micro, BF16, group=1, retain_grads=1, wgrad_groups=2), np.concatenate(params))
    gen = torch.Generator(device="cuda").manual_seed(9)
    n, row = n_micro * s * d, s * d
    x, g = (torch.randn(n, device="cuda", generator=gen).bfloat16() for _ in range(2))

    def run(dy_at, dx_at, per_layer=False):
        buf = torch.full((3 * n + 64,), float("nan"), device="cuda", dtype=torch.bfloat16)
        dy, dx = buf[dy_at:dy_at + n], buf[dx_at:dx_at + n]
        dy.copy_(g)
        st.forward_layered(x.data_ptr(), None)
        if per_layer:
            for l in reversed(range(layers)):
                st.backward_layer(l, (dy if l == layers - 1 else dx).data_ptr(), dx.data_ptr(), None)
        else:
            st.backward_layered(dy.data_ptr(), dx.data_ptr(), None)
        torch.cuda.synchronize()
        return [dx.clone()] + [torch.from_numpy(B.read_device(*st.grads(l), "float32")) for l in range(layers)]

    try:
        ref = run(0, 2 * n)
        assert torch.isfinite(ref[0].float()).all()
        for args in ((0, 0), (0, row), (row, 0), (shift, 2 * n), (0, 2 * n + shift), (shift, shift), (0, 2 * n, True), (0, 0, True), (row, 0, True)):
            for got, want in zip(run(*args), ref):
                assert torch.equal(got, want), args
    finally:
        st.close()


@pytest.mark.parametrize("d,heads,ff", [(1536, 12, 6144), (128, 2, 512)], ids=["ring", "in_place"])
def test_gradient_buffers_in_pinned_host_memory_are_copied(d, heads, ff):
    """A caller may keep dy and dx in pinned host memory: the sweep and the per-layer call give the bits of device buffers (and copy, instead
    of reading dy over the bus in every kernel that wants it)."""
    n_micro, s = 4, 80
    cfg = B.make_config(1, d, heads, ff, s, 1, n_micro, BF16, group=1, retain_grads=1, wgrad_groups=2)
    st = B.Stack(cfg, np.random.default_rng(1).standard_normal(B.params_per_layer(cfg)).astype(np.float32) * 0.02)
    gen = torch.Generator(device="cuda").manual_seed(9)
    x, g = (torch.randn(n_micro * s * d, device="cuda", generator=gen).bfloat16() for _ in range(2))
    try:
        results = []
        for call in (st.backward_layered, lambda dy, dx, adam: st.backward_layer(0, dy, dx, adam)):
            for host in (False, True):
                dy, dx = (torch.zeros(g.numel(), dtype=torch.bfloat16, pin_memory=True) for _ in range(2)) if host else (g, torch.zeros_like(g))
                if host:
                    dy.copy_(g)
                st.forward_layered(x.data_ptr(), None)
                call(dy.data_ptr(), dx.data_ptr(), None)
                torch.cuda.synchronize()
                results.append([dx.cpu(), torch.from_numpy(B.read_device(*st.grads(0), "float32"))])
        for got in results[1:]:
            assert all(torch.equal(a, b) for a, b in zip(got, results[0]))
    finally:
        st.close()
