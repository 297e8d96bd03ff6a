"""GPU parity of the fused attention for head sizes above 160: every padded size and its neighbours, sequence lengths at the edges of
the 32-position tiles and 128-position blocks, and scores that keep growing along the keys, so that the softmax reference moves
in tile after tile.  Gates as for the other 16-bit attention kernels (test_gpu_ops.TOL_ATTN)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
import synth_inputs as S
from gpu_helpers import to_dev, empty_dev, to_host, rel_err, profiled, run_gpu_step
from test_gpu_ops import attention_reference, rnd, ROUND, TOL_ATTN, BF16, F16


def run(dt, qkv, dout, n_seq, s, heads, dh, causal):
    d = heads * dh
    qd, dod = to_dev(qkv, dt), to_dev(dout, dt)
    out, dqkv = empty_dev((n_seq * s, d), dt), empty_dev((n_seq * s, 3 * d), dt)
    lse, delta = torch.empty(n_seq * heads * s, device="cuda"), torch.empty(n_seq * heads * s, device="cuda")
    ws = torch.empty(int(B.lib.lga_op_attention_gemm_workspace_bytes(s, heads)), device="cuda", dtype=torch.uint8)
    B.check(B.lib.lga_op_attention_gemm_fwd(dt, qd.data_ptr(), out.data_ptr(), lse.data_ptr(), n_seq, s, heads, dh, int(causal),
                                            ws.data_ptr(), ws.numel(), None))
    B.check(B.lib.lga_op_attention_gemm_bwd(dt, qd.data_ptr(), out.data_ptr(), lse.data_ptr(), dod.data_ptr(), dqkv.data_ptr(),
                                            delta.data_ptr(), n_seq, s, heads, dh, int(causal), ws.data_ptr(), ws.numel(), None))
    torch.cuda.synchronize()
    return to_host(out), lse.cpu().numpy().reshape(n_seq, heads, s), to_host(dqkv)


def check(dt, got, want, d, loose=1.0):
    out, lse, dqkv = got
    assert rel_err(out, want[0]) < TOL_ATTN[dt][0]
    assert np.abs(lse - want[1]).max() < 1e-3 * max(1.0, np.abs(want[1]).max())
    for i, name in enumerate(("dq", "dk", "dv")):
        sl = slice(i * d, (i + 1) * d)
        assert rel_err(dqkv[:, sl], want[2][:, sl]) < loose * TOL_ATTN[dt][1], name


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("dh", [168, 192, 200, 224, 232, 256, 264, 320])
def test_wide_heads_at_the_edges_of_tiles_and_blocks(dh, dt, causal):
    # (above 224 channels the backward pass of these runs on the GEMMs: the fused one has cases of its own below)
    for n_seq, s, heads in ((1, 8, 1), (2, 40, 2), (1, 128, 1), (1, 136, 2), (1, 264, 45), (2, 160, 40)):
        rng = np.random.default_rng(dh + s)
        qkv, dout = rnd(rng, (n_seq * s, 3 * heads * dh), dt), rnd(rng, (n_seq * s, heads * dh), dt)
        check(dt, run(dt, qkv, dout, n_seq, s, heads, dh, causal),
              attention_reference(qkv, dout, n_seq, s, heads, dh, causal), heads * dh)


@pytest.mark.parametrize("dt,dh,causal", [(BF16, 216, True), (F16, 216, False), (BF16, 320, False), (F16, 256, True)])
def test_wide_heads_with_scores_that_keep_growing_along_the_keys(dt, dh, causal):
    n_seq, s, heads = 1, 320, 2
    d = heads * dh
    rng = np.random.default_rng(77 + dh)
    qkv = rng.standard_normal((s, 3 * d)).astype(np.float32)
    for h in range(heads):
        qkv[:, h * dh] = math.sqrt(dh)                            # q[:, 0] = sqrt(dh)
        qkv[:, d + h * dh] = 0.25 * np.arange(s)                  # k[j, 0] = j / 4: key j scores about j / 4 nats with every query
    qkv, dout = ROUND[dt](qkv), rnd(rng, (s, d), dt)
    # near one-hot probabilities times keys of size ~80: the rounding of dS weighs more than on ordinary inputs
    check(dt, run(dt, qkv, dout, n_seq, s, heads, dh, causal), attention_reference(qkv, dout, n_seq, s, heads, dh, causal), d, loose=2.0)


@pytest.mark.parametrize("dh,products", [(168, 4), (192, 4), (200, 4), (224, 4), (232, 5), (320, 5)])
def test_the_profile_counts_the_products_that_the_key_gradients_take(dh, products):
    """One run up to 224 channels (S, dP, dV, dK), beyond it two that both compute S; 2 s^2 dh operations each."""
    n_seq, s, heads = 1, 512, 56
    qkv = torch.zeros(n_seq * s, 3 * heads * dh, device="cuda", dtype=torch.bfloat16)
    dout = torch.zeros(n_seq * s, heads * dh, device="cuda", dtype=torch.bfloat16)
    kernels = profiled(lambda: run(BF16, qkv.float().cpu().numpy(), dout.float().cpu().numpy(), n_seq, s, heads, dh, False))
    flops = sum(k["flops"] for name, k in kernels.items() if name.startswith("attn_wide_dkv"))
    assert flops == products * 2.0 * heads * s * s * dh


@pytest.mark.parametrize("dh", [168, 216, 256, 320])
def test_large_gradients_in_half_precision_stay_finite(dh):
    """dS = P (dP - delta) / sqrt(d_h) is rounded to half precision with the factor in it: gradients whose unscaled dS lies beyond the
    format's 65504 while everything that is returned lies within it."""
    n_seq, s, heads = 1, 264, 104
    d = heads * dh
    rng = np.random.default_rng(dh)
    qkv, dout = rnd(rng, (n_seq * s, 3 * d), F16), ROUND[F16](rng.standard_normal((n_seq * s, d)).astype(np.float32) * 6000)
    want = attention_reference(qkv, dout, n_seq, s, heads, dh, True)
    assert np.abs(want[2]).max() < 60000
    got = []
    kernels = profiled(lambda: got.append(run(F16, qkv, dout, n_seq, s, heads, dh, True)))
    assert any(k.startswith("attn_wide_dq") for k in kernels)
    assert np.isfinite(got[0][2]).all()
    check(F16, got[0], want, d)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,fused,n_seq,s,heads", [
    (232, True, 1, 264, 80), (256, True, 1, 136, 110), (256, True, 2, 48, 70), (264, True, 1, 264, 104), (320, True, 2, 160, 170),
    (320, True, 1, 136, 210), (168, False, 1, 1000, 1), (224, False, 2, 520, 3), (256, False, 1, 520, 4), (320, False, 2, 520, 4)])
def test_wide_heads_on_either_side_of_the_rule_between_fused_kernels_and_gemms(dh, fused, n_seq, s, heads, causal):
    rng = np.random.default_rng(dh + s)
    d, got = heads * dh, []
    qkv, dout = rnd(rng, (n_seq * s, 3 * d), BF16), rnd(rng, (n_seq * s, d), BF16)
    kernels = profiled(lambda: got.append(run(BF16, qkv, dout, n_seq, s, heads, dh, causal)))
    assert any(k.startswith("attn_wide_dq") for k in kernels) == fused
    assert any(k.startswith("attn_ds_rows") for k in kernels) != fused
    check(BF16, got[0], attention_reference(qkv, dout, n_seq, s, heads, dh, causal), d)


@pytest.mark.parametrize("dh,heads,groups", [(256, 8, (1, 2)), (320, 4, (1, 2, 4))])
def test_wide_heads_do_not_depend_on_how_many_sequences_share_a_launch(dh, heads, groups):
    """128 and 256 workgroups of the fused kernels: the orders and group sizes agree bit for bit."""
    w = S.Workload("wide_groups", 1, heads * dh, heads, 512, 256, 8, groups[-1], "bf16")
    x, G, params = S.make_inputs(w, seed=5)
    runs = [run_gpu_step(w, x, G, params, group=g, retain=1) for g in groups] + [run_gpu_step(w, x, G, params, retain=1, order="mbmajor")]
    for got in runs[1:]:
        assert np.array_equal(got["boundaries"], runs[0]["boundaries"])
        assert np.array_equal(got["dx"], runs[0]["dx"])
