"""fp32 products on tiles of 32 rows: the edges of those tiles and of the stages, up to the most tiles that take them and one more, each a row's
bits the same as in a product of many rows (64-row tiles), and within 1e-5 of 64 bits (see test_gpu_gemm_f32)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B


def product(kc, epi, a, w, out, out2, bias, aux, M, N, K):
    B.check(B.lib.lga_op_gemm(B.LGA_FP32, 1, kc, epi, M, N, K, a.data_ptr(), K, w.data_ptr(), K if kc else N, out.data_ptr(),
                              out2.data_ptr() if epi == 3 else None, None, N, bias.data_ptr(), aux.data_ptr(), 0.0, None))


@pytest.mark.parametrize("N,K", [(4, 4), (60, 32), (64, 36), (192, 64), (68, 96), (128, 100), (256, 256), (512, 1028)])
@pytest.mark.parametrize("epi,kc", [(0, 1), (4, 1), (1, 0), (2, 0), (3, 0)])
def test_a_row_does_not_depend_on_the_height_of_the_tiles(N, K, epi, kc):
    tall = 32 * (256 // ((N + 63) // 64)) + 1                       # one tile of 32 rows more than take them
    g = torch.Generator(device="cuda").manual_seed(N + K)
    a, aux = torch.randn(tall, K, device="cuda", generator=g), torch.randn(tall, N, device="cuda", generator=g)
    w, bias = torch.randn(K, N, device="cuda", generator=g), torch.randn(N, device="cuda", generator=g)
    stored = w.t().contiguous() if kc else w
    all_out, all_out2 = torch.empty(tall, N, device="cuda"), torch.empty(tall, N, device="cuda")
    product(kc, epi, a, stored, all_out, all_out2, bias, aux, tall, N, K)
    u = a.double() @ w.double()
    if epi in (1, 2, 3): u += bias.double()
    if epi == 2: u += aux.double()
    if epi == 3: u = torch.nn.functional.gelu(u, approximate="tanh")
    if epi == 4:
        x = aux.double().requires_grad_()
        torch.nn.functional.gelu(x, approximate="tanh").sum().backward()
        u *= x.grad
    assert torch.linalg.norm(all_out.double() - u) <= 1e-5 * torch.linalg.norm(u)
    for rows in (1, 31, 32, 33, 65, tall - 1):
        out, out2 = (torch.full((rows + 1, N), float("nan"), device="cuda") for _ in range(2))
        product(kc, epi, a[:rows], stored, out, out2, bias, aux[:rows], rows, N, K)
        assert torch.equal(out[:rows], all_out[:rows]) and out[rows:].isnan().all(), rows
        assert epi != 3 or (torch.equal(out2[:rows], all_out2[:rows]) and out2[rows:].isnan().all()), rows


@pytest.mark.parametrize("M,N", [(1, 4), (28, 64), (32, 68), (36, 192), (100, 256), (512, 512)])
@pytest.mark.parametrize("K", [4, 32, 100, 512, 1000])
def test_weight_gradients_on_few_tiles(M, N, K):
    M = (M + 3) // 4 * 4
    rng = np.random.default_rng(M + N + K)
    x, dy = rng.standard_normal((K, M)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    old = rng.standard_normal((M, N)).astype(np.float32)
    xd, dyd, out = (torch.from_numpy(t).cuda() for t in (x, dy, old))
    B.check(B.lib.lga_op_gemm(B.LGA_FP32, 0, 0, B.LGA_EPI_ACCUM_F32, M, N, K, xd.data_ptr(), M, dyd.data_ptr(), N, None, None, out.data_ptr(), N, None, None,
                              0.5, None))
    want = 0.5 * old.astype(np.float64) + x.astype(np.float64).T @ dy.astype(np.float64)
    assert np.linalg.norm(out.cpu().numpy() - want) <= 1e-5 * np.linalg.norm(want)
