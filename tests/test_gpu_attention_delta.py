"""The row sums delta = sum_c dO O that the dQ kernels leave for the dK/dV kernels: every head of every position, at head sizes inside and
at the edges of the padded ones and lengths inside and past a block of 128 queries.  Products of 16-bit values are exact in 32 bits,
so n of them add up with at most n 2^-24 of the sum of their magnitudes lost, in any order."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import to_dev, empty_dev, to_host
from test_gpu_ops import rnd, BF16, F16


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("dh", [8, 32, 40, 64, 96, 104, 128, 152, 160, 168, 192, 216])
def test_dq_leaves_the_row_sums_for_dk_and_dv(dh, dt, causal):
    wide = dh > 160
    for n_seq, s, heads in ((1, 8, 1), (2, 136, 2), (1, 264, 45)):
        d = heads * dh
        rng = np.random.default_rng(dh + s)
        qd, dod = to_dev(rnd(rng, (n_seq * s, 3 * d), dt), dt), to_dev(rnd(rng, (n_seq * s, d), dt), dt)
        out, dqkv = empty_dev((n_seq * s, d), dt), empty_dev((n_seq * s, 3 * d), dt)
        lse, delta = torch.empty(n_seq * heads * s, device="cuda"), torch.full((n_seq * heads * s,), float("nan"), device="cuda")
        ws = torch.empty(int(B.lib.lga_op_attention_gemm_workspace_bytes(s, heads)), device="cuda", dtype=torch.uint8)
        tail = (n_seq, s, heads, dh, int(causal)) + ((ws.data_ptr(), ws.numel(), None) if wide else (None,))
        head = (dt,) if wide else (dt, 1)
        fwd, bwd = ((B.lib.lga_op_attention_gemm_fwd, B.lib.lga_op_attention_gemm_bwd) if wide else
                    (B.lib.lga_op_attention_fwd, B.lib.lga_op_attention_bwd))
        B.check(fwd(*head, qd.data_ptr(), out.data_ptr(), lse.data_ptr(), *tail))
        B.check(bwd(*head, qd.data_ptr(), out.data_ptr(), lse.data_ptr(), dod.data_ptr(), dqkv.data_ptr(), delta.data_ptr(), *tail))
        torch.cuda.synchronize()
        prod = (to_host(out).astype(np.float64) * to_host(dod).astype(np.float64)).reshape(n_seq, s, heads, dh)
        err = np.abs(delta.cpu().numpy().reshape(n_seq, heads, s).transpose(0, 2, 1) - prod.sum(-1))
        assert (err <= dh * 2.0**-24 * np.abs(prod).sum(-1) + 1e-30).all()
