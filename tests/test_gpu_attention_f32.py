"""GPU parity of the fp32 attention at the edges of its 32-position blocks, of its four-way split of the streamed blocks and of
its head-size ranges (up to 32, 64, 128; above: the one-wavefront kernels), with 16-byte-aligned rows and without.  Gates as
for every fp32 kernel: 1e-5 forward, 2e-5 backward."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import rel_err, profiled
from test_gpu_ops import attention_reference


def run(qkv, dout, n_seq, s, heads, dh, causal, shift=0):
    d = heads * dh

    def place(a):
        t = torch.full((a.size + 8,), float("nan"), device="cuda")
        v = t[shift:shift + a.size]
        v.copy_(torch.from_numpy(np.ascontiguousarray(a)).cuda().reshape(-1))
        return v
    q, g = place(qkv), place(dout)
    out, dqkv = place(np.full((n_seq * s, d), np.nan, np.float32)), place(np.full((n_seq * s, 3 * d), np.nan, np.float32))
    lse, delta = torch.empty(n_seq * heads * s, device="cuda"), torch.empty(n_seq * heads * s, device="cuda")
    B.check(B.lib.lga_op_attention_fwd(B.LGA_FP32, 0, q.data_ptr(), out.data_ptr(), lse.data_ptr(), n_seq, s, heads, dh, int(causal), None))
    B.check(B.lib.lga_op_attention_bwd(B.LGA_FP32, 0, q.data_ptr(), out.data_ptr(), lse.data_ptr(), g.data_ptr(), dqkv.data_ptr(),
                                       delta.data_ptr(), n_seq, s, heads, dh, int(causal), None))
    torch.cuda.synchronize()
    return (out.cpu().numpy().reshape(n_seq * s, d), lse.cpu().numpy().reshape(n_seq, heads, s), dqkv.cpu().numpy().reshape(n_seq * s, 3 * d))


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,shift", [(1, 0), (10, 0), (16, 0), (32, 0), (32, 1), (36, 0), (64, 0), (65, 0), (100, 0), (128, 0), (132, 0)])
def test_fp32_attention_at_block_edges(dh, shift, causal):
    for n_seq, s, heads in ((1, 2, 1), (2, 31, 2), (1, 32, 3), (1, 33, 1), (1, 129, 2), (1, 300, 1)):
        rng = np.random.default_rng(dh * 1000 + s)
        qkv = rng.standard_normal((n_seq * s, 3 * heads * dh)).astype(np.float32)
        dout = rng.standard_normal((n_seq * s, heads * dh)).astype(np.float32)
        want = attention_reference(qkv, dout, n_seq, s, heads, dh, causal)
        got = run(qkv, dout, n_seq, s, heads, dh, causal, shift)
        assert rel_err(got[0], want[0]) < 1e-5, (s, heads)
        assert np.abs(got[1] - want[1]).max() < 1e-5 * max(1.0, np.abs(want[1]).max()), (s, heads)
        d = heads * dh
        for i in range(3):
            assert rel_err(got[2][:, i * d:(i + 1) * d], want[2][:, i * d:(i + 1) * d]) < 2e-5, (s, heads, "dq dk dv".split()[i])


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("s,dh", [(40, 32), (200, 64)])
def test_fp32_causal_attention_keeps_the_future_out_even_if_it_is_not_finite(s, dh, bad):
    rng = np.random.default_rng(s)
    qkv = rng.standard_normal((s, 3 * dh)).astype(np.float32)
    dout = rng.standard_normal((s, dh)).astype(np.float32)
    n = s - 3                                               # positions n .. s - 1 are not finite: nobody before them may notice
    want = attention_reference(qkv[:n], dout[:n], 1, n, 1, dh, True)
    q2 = qkv.copy()
    q2[n:] = bad
    out, lse, dqkv = run(q2, dout, 1, s, 1, dh, True)
    assert rel_err(out[:n], want[0]) < 1e-5 and np.abs(lse[0, 0, :n] - want[1][0, 0]).max() < 1e-4
    assert rel_err(dqkv[:n, :dh], want[2][:, :dh]) < 2e-5
    # a query and its output gradient that are not finite reach no key after them
    q2, d2 = qkv.copy(), dout.copy()
    q2[0, :dh] = bad
    d2[0] = bad
    want = attention_reference(qkv, np.concatenate([np.zeros_like(dout[:1]), dout[1:]]), 1, s, 1, dh, True)
    _, _, dqkv = run(q2, d2, 1, s, 1, dh, True)
    assert rel_err(dqkv[1:, dh:], want[2][1:, dh:]) < 2e-5


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [8, 10, 32, 64, 128])
def test_fp32_attention_on_either_side_of_the_length_from_which_on_the_matrix_instruction_serves_it(dh, causal):
    for n_seq, s, heads, matrix in ((1, 16, 2, False), (2, 48, 1, False), (1, 49, 2, True), (2, 63, 1, True), (1, 64, 3, True), (1, 65, 1, True),
                                    (1, 97, 2, True)):
        rng = np.random.default_rng(dh * 1000 + s)
        qkv = rng.standard_normal((n_seq * s, 3 * heads * dh)).astype(np.float32)
        dout = rng.standard_normal((n_seq * s, heads * dh)).astype(np.float32)
        want, got = attention_reference(qkv, dout, n_seq, s, heads, dh, causal), []
        kernels = profiled(lambda: got.append(run(qkv, dout, n_seq, s, heads, dh, causal)))
        assert any(k.startswith("attn_fwd_f32") for k in kernels) == any(k.startswith("attn_bwd_dq_f32") for k in kernels) == matrix
        assert any(k.startswith("attn_fwd_simple") for k in kernels) == any(k.startswith("attn_bwd_simple") for k in kernels) != matrix
        assert rel_err(got[0][0], want[0]) < 1e-5, (s, heads)
        assert np.abs(got[0][1] - want[1]).max() < 1e-5 * max(1.0, np.abs(want[1]).max()), (s, heads)
        d = heads * dh
        for i in range(3):
            assert rel_err(got[0][2][:, i * d:(i + 1) * d], want[2][:, i * d:(i + 1) * d]) < 2e-5, (s, heads, "dq dk dv".split()[i])
