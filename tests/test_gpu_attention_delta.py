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


@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("dh", [24, 64, 128, 160, 216, 320])
def test_the_result_may_take_the_memory_of_the_attention_output(dh, dt):
    """The gradient written where O is read from: at the start of it, at its end, and across its start.  delta is then the same sum in another
    order (bound as above, twice), which moves 16-bit results by their last bit at most here and there."""
    wide = dh > 160
    n_seq, s, heads = 2, 520, 48                                  # heads enough for the fused kernels at every head size
    d, n = heads * dh, n_seq * s * heads * dh
    rng = np.random.default_rng(dh)
    qd, dod = to_dev(rnd(rng, (n_seq * s, 3 * d), dt), dt), to_dev(rnd(rng, (n_seq * s, d), dt), dt)
    o = empty_dev((n_seq * s, d), dt)
    lse, delta = torch.empty(n_seq * heads * s, device="cuda"), torch.empty(n_seq * heads * s, device="cuda")
    ws = torch.empty(int(B.lib.lga_op_attention_gemm_workspace_bytes(s, 1)), device="cuda", dtype=torch.uint8)
    tail = (n_seq, s, heads, dh, 1) + ((ws.data_ptr(), ws.numel(), None) if wide else (None,))
    head = (dt,) if wide else (dt, 1)
    fwd, bwd = ((B.lib.lga_op_attention_gemm_fwd, B.lib.lga_op_attention_gemm_bwd) if wide else
                (B.lib.lga_op_attention_fwd, B.lib.lga_op_attention_bwd))
    B.check(fwd(*head, qd.data_ptr(), o.data_ptr(), lse.data_ptr(), *tail))

    def backward(out, dqkv):
        delta.fill_(float("nan"))
        B.check(bwd(*head, qd.data_ptr(), out.data_ptr(), lse.data_ptr(), dod.data_ptr(), dqkv.data_ptr(), delta.data_ptr(), *tail))
        torch.cuda.synchronize()
        return to_host(dqkv), delta.cpu().numpy().astype(np.float64)

    apart, delta_apart = backward(o, empty_dev((3 * n,), dt))
    prod = (to_host(o) * to_host(dod)).reshape(n_seq, s, heads, dh)
    bound = 2 * dh * 2.0**-24 * np.abs(prod).sum(-1).transpose(0, 2, 1).ravel() + 1e-30
    memory = empty_dev((4 * n,), dt)
    for first in (n, 3 * n, n // 2):                              # where O lies; dQKV: n ... 4 n
        memory.fill_(float("nan"))
        memory[first:first + n] = o.view(-1)
        dqkv, dl = backward(memory[first:first + n], memory[n:])
        assert (np.abs(dl - delta_apart) <= bound).all(), first
        assert np.linalg.norm(dqkv - apart) <= (2.0**-8 if dt == BF16 else 2.0**-10) * np.linalg.norm(apart), first
