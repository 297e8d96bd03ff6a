"""GPU parity of the LayerNorm kernels that give a wavefront a whole row, at the widths where a lane's number of packs changes and where the
kernels for wider rows take over, with few, odd and many rows; the sums for gain and bias over all of them.  fp32 1e-5 (sums of at most
2064 values), 16 bits one rounding of the result (4e-3, IEEE half 5e-4)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import TORCH_DTYPE, to_host, rel_err

WIDTHS = {B.LGA_FP32: (4, 60, 256, 260, 512, 516, 1024, 1028), B.LGA_BF16: (8, 120, 512, 520, 1024, 1032, 2048, 2056)}
GATE = {B.LGA_FP32: 1e-5, B.LGA_BF16: 4e-3, B.LGA_FP16: 5e-4}


@pytest.mark.parametrize("rows", [1, 4, 5, 1030, 8201])
@pytest.mark.parametrize("dt", [B.LGA_FP32, B.LGA_BF16, B.LGA_FP16])
def test_layernorm_at_pack_and_row_edges(dt, rows):
    for d in WIDTHS.get(dt, WIDTHS[B.LGA_BF16]):
        gen = torch.Generator(device="cuda").manual_seed(d + rows)
        x, dy, resid = (torch.randn(rows, d, device="cuda", generator=gen).to(TORCH_DTYPE[dt]) for _ in range(3))
        g, b = (1.0 + 0.1 * torch.randn(d, device="cuda", generator=gen) for _ in range(2))
        x += 3.0
        y, dx = torch.empty_like(x), torch.empty_like(x)
        mean, rstd = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
        old = torch.randn(2, d, device="cuda", generator=gen)
        sums = old.clone()
        scratch = torch.full((B.lib.lga_op_layernorm_bwd_scratch_floats(rows, d),), float("nan"), device="cuda")
        B.check(B.lib.lga_op_layernorm_fwd(dt, x.data_ptr(), g.data_ptr(), b.data_ptr(), y.data_ptr(), mean.data_ptr(), rstd.data_ptr(), rows, d, 1e-5, None))
        B.check(B.lib.lga_op_layernorm_bwd(dt, dy.data_ptr(), x.data_ptr(), mean.data_ptr(), rstd.data_ptr(), g.data_ptr(), resid.data_ptr(), dx.data_ptr(),
                                           sums[0].data_ptr(), sums[1].data_ptr(), 0.5, scratch.data_ptr(), rows, d, None))
        torch.cuda.synchronize()
        x64, dy64, g64 = to_host(x), to_host(dy), to_host(g)
        mu, var = x64.mean(1, keepdims=True), x64.var(1, keepdims=True)
        xhat = (x64 - mu) / np.sqrt(var + 1e-5)
        gd = dy64 * g64
        want_dx = to_host(resid) + (gd - gd.mean(1, keepdims=True) - xhat * (gd * xhat).mean(1, keepdims=True)) / np.sqrt(var + 1e-5)
        # (rows of 4 or 8 values: 1 / sqrt(var) passes the errors of the mean on several times over)
        gate = GATE[dt] * (8 if d <= 8 else 1)
        assert rel_err(to_host(y), xhat * g64 + to_host(b)) < gate, d
        assert rel_err(to_host(dx), want_dx) < gate, d
        assert rel_err(to_host(mean), mu[:, 0]) < 1e-6 and rel_err(to_host(rstd), 1 / np.sqrt(var[:, 0] + 1e-5)) < 1e-5 * (8 if d <= 8 else 1), d
        assert rel_err(to_host(sums[0]), 0.5 * to_host(old[0]) + (dy64 * xhat).sum(0)) < 1e-5 * (8 if d <= 8 else 1), d
        assert rel_err(to_host(sums[1]), 0.5 * to_host(old[1]) + dy64.sum(0)) < 1e-5, d


def test_a_row_that_is_not_finite_stays_alone():
    x = torch.randn(9, 768, device="cuda").bfloat16()
    g, b = torch.ones(768, device="cuda"), torch.zeros(768, device="cuda")
    clean, got = torch.empty_like(x), torch.empty_like(x)
    mean, rstd = torch.empty(9, device="cuda"), torch.empty(9, device="cuda")
    call = lambda y: B.check(B.lib.lga_op_layernorm_fwd(B.LGA_BF16, x.data_ptr(), g.data_ptr(), b.data_ptr(), y.data_ptr(), mean.data_ptr(), rstd.data_ptr(), 9, 768, 1e-5, None))
    call(clean)
    x[2, 700], x[5, 0] = float("inf"), float("nan")
    call(got)
    torch.cuda.synchronize()
    bad = torch.zeros(9, dtype=torch.bool, device="cuda")
    bad[2] = bad[5] = True
    assert torch.isnan(got[bad]).any(1).all() and torch.equal(got[~bad], clean[~bad])
