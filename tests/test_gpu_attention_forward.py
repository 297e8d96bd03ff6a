"""The forward kernels' two widths of a wavefront, 32 and 64 queries: chosen by the number of workgroups, with the same results bit for bit, also where a
workgroup starts over."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import profiled, rel_err
from test_gpu_ops import BF16, F16

TYPE = {BF16: torch.bfloat16, F16: torch.float16}


def forward(qkv, n_seq, s, heads, dh, dt, causal):
    out = torch.full((n_seq * s, heads * dh), float("nan"), device="cuda", dtype=TYPE[dt])
    lse = torch.full((n_seq, heads, s), float("nan"), device="cuda")
    B.check(B.lib.lga_op_attention_fwd(dt, 1, qkv.data_ptr(), out.data_ptr(), lse.data_ptr(), n_seq, s, heads, dh, int(causal), None))
    torch.cuda.synchronize()
    return out, lse


def width(call):
    """Query sub-blocks of the forward kernel that `call` launches."""
    (name,) = profiled(call)
    return int(name[name.index(", ") + 2:-1])


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("dh", [8, 32, 64, 96, 128, 152, 160])
def test_a_sequence_does_not_depend_on_how_many_share_the_launch(dh, dt, causal):
    """One sequence alone (a wavefront per 32 queries), then as the last of as many as fill the chip (64, but for lengths that leave workgroups of 256 queries half
    empty): lengths around the ends of key tiles, of a wavefront's queries and of a workgroup's.  Against 64 bits: P and the result are rounded to 16 bits once each, and
    the scores are sums in 32."""
    for s, wide in ((1, 1), (31, 1), (33, 1), (64, 1), (65, 1), (127, 1), (129, 2), (192, 2), (255, 2), (256, 2), (257, 1), (321, 1), (385, 2), (448, 2), (511, 2), (641, 2)):
        heads, many = 4, 256
        g = torch.Generator(device="cuda").manual_seed(s + dh)
        qkv = torch.randn(many * s, 3 * heads * dh, device="cuda", generator=g).to(TYPE[dt])
        results = []
        assert width(lambda: results.append(forward(qkv, many, s, heads, dh, dt, causal))) == wide, s
        all_out, all_lse = results[0]
        again_out, again_lse = forward(qkv, many, s, heads, dh, dt, causal)
        assert torch.equal(all_out, again_out) and torch.equal(all_lse, again_lse), s
        assert width(lambda: results.append(forward(qkv[-s:].clone(), 1, s, heads, dh, dt, causal))) == 1, s
        one_out, one_lse = results[1]
        assert torch.equal(all_out[-s:], one_out) and torch.equal(all_lse[-1], one_lse[0]), s
        q, k, v = (qkv[-s:].double().view(s, 3, heads, dh)[:, i].permute(1, 0, 2).contiguous() for i in range(3))
        scores = q @ k.transpose(1, 2).contiguous() / dh**0.5
        if causal:
            scores = scores.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
        ref = (torch.softmax(scores, -1) @ v).permute(1, 0, 2).reshape(s, heads * dh)
        ulp = 2.0**-9 if dt == BF16 else 2.0**-12
        assert rel_err(one_out.double().cpu().numpy(), ref.cpu().numpy()) <= 3 * ulp, s
        assert np.abs((one_lse[0].double() - torch.logsumexp(scores, -1)).cpu().numpy()).max() <= 1e-5, s


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("dh", [24, 32, 64, 96, 128, 152])
def test_a_query_that_starts_over_does_not_move_its_neighbours(dh, dt, causal):
    """Keys behind the first 32 score up to 34 (bf16: 150) log2 units with one query each, so that some queries in every other 128 start over, by their sums in 64 bits,
    and none in those between: one sequence alone, in workgroups of 128 queries, and as the last of many, in those of 256, over one to six
    of the larger.  Against 64 bits: the products of 16-bit values are exact, and a score's sum in fp32 is off by dh 2^-24 of its terms."""
    heads, many = 4, 128
    for s in (200, 256, 449, 512, 700, 1500):
        g = torch.Generator(device="cuda").manual_seed(s + dh)
        rand = lambda *shape: torch.randn(*shape, device="cuda", generator=g)
        q, k, v = (rand(many, s, heads, dh) for _ in range(3))
        q *= math.sqrt(dh) / q.norm(dim=-1, keepdim=True)            # no key scores more with another query
        at = torch.arange(60, s, 3, device="cuda")                   # query i's own key is i - 20
        starts = (at // 128 % 2 == 1)[:, None, None]
        share = torch.rand(many, at.numel(), heads, 1, device="cuda", generator=g)
        units = torch.where(starts, 20 + 14 * share, 14 + 6 * share) if dt == F16 else torch.where(starts, 90 + 60 * share, 20 + 70 * share)
        k[:, at - 20] = q[:, at] * units * math.log(2.0) / math.sqrt(dh)
        qkv = torch.stack([q, k, v], 2).reshape(many * s, 3 * heads * dh).to(TYPE[dt])
        results = []
        widths = [width(lambda: results.append(forward(qkv, many, s, heads, dh, dt, causal))),
                  width(lambda: results.append(forward(qkv[-s:].clone(), 1, s, heads, dh, dt, causal)))]
        assert widths == [2, 1], s
        (all_out, all_lse), (one_out, one_lse) = results
        q, k, v = (qkv[-s:].double().view(s, 3, heads, dh)[:, i].permute(1, 0, 2).contiguous() for i in range(3))
        scores = q @ k.transpose(1, 2).contiguous() / dh**0.5
        if causal:
            scores = scores.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
        lse = torch.logsumexp(scores, -1)
        # log2 of the sum above the kernel's reference.  From the limit (2^16, bf16 2^100) on, of which half a row holds half at least, a query starts over
        above = (lse - scores[..., :32].amax(-1)) / math.log(2.0) - (6.0 if dt == F16 else 0.0)
        over, high = above > (17 if dt == F16 else 101), (above > 8) & (above < (15 if dt == F16 else 98))
        alone = [b for b in range(0, s, 256) if (over[:, b + 128:b + 256].any(-1) & high[:, b:b + 128].any(-1) & (above[:, b:b + 128] < (15 if dt == F16 else 98)).all(-1)).any()]
        assert alone, s
        assert torch.equal(all_out[-s:], one_out) and torch.equal(all_lse[-1], one_lse[0]), s
        ref = (torch.softmax(scores, -1) @ v).permute(1, 0, 2).reshape(s, heads * dh)
        ulp = 2.0**-9 if dt == BF16 else 2.0**-12
        bound = dh * 2.0**-24 * float(scores[scores > float("-inf")].abs().max())
        assert rel_err(one_out.double().cpu().numpy(), ref.cpu().numpy()) <= 3 * ulp + bound, s
        assert (one_lse[0].double() - lse).abs().max().item() <= 1e-5 + bound, s
