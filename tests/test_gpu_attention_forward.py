"""The forward kernels' two widths of a wavefront, 32 and 64 queries: chosen by the number of workgroups, with the same results bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import rel_err
from test_gpu_ops import BF16, F16

TYPE = {BF16: torch.bfloat16, F16: torch.float16}


def forward(qkv, n_seq, s, heads, dh, dt, causal):
    out = torch.full((n_seq * s, heads * dh), float("nan"), device="cuda", dtype=TYPE[dt])
    lse = torch.full((n_seq, heads, s), float("nan"), device="cuda")
    B.check(B.lib.lga_op_attention_fwd(dt, 1, qkv.data_ptr(), out.data_ptr(), lse.data_ptr(), n_seq, s, heads, dh, int(causal), None))
    torch.cuda.synchronize()
    return out, lse


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("dh", [8, 32, 64, 96, 128, 152, 160])
def test_a_sequence_does_not_depend_on_how_many_share_the_launch(dh, dt, causal):
    """One sequence alone (a wavefront per 32 queries), then as the last of as many as fill the chip (64): lengths around the ends of key tiles, of a
    wavefront's queries and of a workgroup's.  Against 64 bits: P and the result are rounded to 16 bits once each, and the scores are sums in 32."""
    for s in (1, 31, 33, 64, 65, 127, 129, 192, 257, 321):
        heads, many = 4, 300
        g = torch.Generator(device="cuda").manual_seed(s + dh)
        qkv = torch.randn(many * s, 3 * heads * dh, device="cuda", generator=g).to(TYPE[dt])
        all_out, all_lse = forward(qkv, many, s, heads, dh, dt, causal)
        again_out, again_lse = forward(qkv, many, s, heads, dh, dt, causal)
        assert torch.equal(all_out, again_out) and torch.equal(all_lse, again_lse), s
        one_out, one_lse = forward(qkv[-s:].clone(), 1, s, heads, dh, dt, causal)
        assert torch.equal(all_out[-s:], one_out) and torch.equal(all_lse[-1], one_lse[0]), s
        q, k, v = (qkv[-s:].double().view(s, 3, heads, dh)[:, i].permute(1, 0, 2).contiguous() for i in range(3))
        scores = q @ k.transpose(1, 2).contiguous() / dh**0.5
        if causal:
            scores = scores.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
        ref = (torch.softmax(scores, -1) @ v).permute(1, 0, 2).reshape(s, heads * dh)
        ulp = 2.0**-9 if dt == BF16 else 2.0**-12
        assert rel_err(one_out.double().cpu().numpy(), ref.cpu().numpy()) <= 3 * ulp, s
        assert np.abs((one_lse[0].double() - torch.logsumexp(scores, -1)).cpu().numpy()).max() <= 1e-5, s
