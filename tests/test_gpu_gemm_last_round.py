"""GPU check of the columns that the large-tile GEMM leaves to the small one behind its whole rounds of 256 tiles: the same bits as the two
parts called one by one, every epilogue, ragged rows, columns and k; nothing but the result is written."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import TORCH_DTYPE, profiled

#         M,    N,     K,   columns of the whole rounds
SHAPES = [(2000, 17024, 456, 16384), (4100, 4360, 200, 3840), (2056, 15368, 1096, 14336)]


@pytest.mark.parametrize("dt", [B.LGA_BF16, B.LGA_FP16])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_columns_behind_the_last_whole_round(shape, dt):
    M, N, K, keep = shape
    gen = torch.Generator(device="cuda").manual_seed(K)
    tdt, pad = TORCH_DTYPE[dt], 8
    A = torch.randn(M, K, device="cuda", generator=gen).to(tdt)
    W = (torch.randn(N, K, device="cuda", generator=gen) * 0.05).to(tdt)
    aux = torch.randn(M, N + pad, device="cuda", generator=gen).to(tdt)
    bias = torch.randn(N, device="cuda", generator=gen)

    def call(epi, out, out2, n0, n):
        B.check(B.lib.lga_op_gemm(dt, 1, 1, epi, M, n, K, A.data_ptr(), K, W[n0:].data_ptr(), K, out[:, n0:].data_ptr(), out2[:, n0:].data_ptr(), None,
                                  N + pad, bias[n0:].data_ptr(), aux[:, n0:].data_ptr(), 0.0, None))

    for epi in (B.LGA_EPI_STORE, B.LGA_EPI_BIAS, B.LGA_EPI_BIAS_RESID, B.LGA_EPI_BIAS_GELU, B.LGA_EPI_MUL_DGELU):
        whole, whole2, parts, parts2 = (torch.full((M, N + pad), 7.0, device="cuda", dtype=tdt) for _ in range(4))
        kernels = profiled(lambda: call(epi, whole, whole2, 0, N))
        assert sorted(k["launches"] for n, k in kernels.items() if "gemm" in n) == [1, 1] and any("small" in n for n in kernels), kernels.keys()
        assert not any("small" in n for n in profiled(lambda: call(epi, parts, parts2, 0, keep)))
        call(epi, parts, parts2, keep, N - keep)
        torch.cuda.synchronize()
        assert torch.equal(whole, parts) and torch.equal(whole2, parts2), epi
        assert bool((whole[:, N:] == 7.0).all()) and bool((whole2[:, N:] == 7.0).all()), epi
    want = A[::97].double() @ W.double().t() * 1.0
    got = torch.empty(M, N + pad, device="cuda", dtype=tdt)
    call(B.LGA_EPI_STORE, got, got, 0, N)
    torch.cuda.synchronize()
    assert float((got[::97, :N].double() - want).norm() / want.norm()) < (4e-3 if dt == B.LGA_BF16 else 5e-4)      # one rounding of the result


#        M,     N,    K,  epilogue, whether the columns behind the whole rounds go to the small tiles
ROUTES = [(4096, 4224, 1024, B.LGA_EPI_MUL_DGELU, True), (11320, 1312, 2048, B.LGA_EPI_BIAS_GELU, True),
          (65280, 264, 1024, B.LGA_EPI_STORE, False),        # the rows' way through memory: 134 MB for 8 columns
          (57336, 1032, 640, B.LGA_EPI_STORE, False), (25600, 2536, 64, B.LGA_EPI_MUL_DGELU, False),      # ... the results'
          (45880, 1688, 64, B.LGA_EPI_BIAS_GELU, False)]


@pytest.mark.parametrize("M,N,K,epi,apart", ROUTES)
def test_columns_apart_only_where_they_cost_less_than_a_round(M, N, K, epi, apart):
    gen = torch.Generator(device="cuda").manual_seed(N)
    A, W, aux = (torch.randn(r, c, device="cuda", generator=gen).bfloat16() for r, c in ((M, K), (N, K), (M, N)))
    out, out2, bias = torch.empty_like(aux), torch.empty_like(aux), torch.randn(N, device="cuda", generator=gen)
    kernels = profiled(lambda: B.check(B.lib.lga_op_gemm(B.LGA_BF16, 1, 1, epi, M, N, K, A.data_ptr(), K, W.data_ptr(), K, out.data_ptr(), out2.data_ptr(),
                                                         None, N, bias.data_ptr(), aux.data_ptr(), 0.0, None)))
    assert any("small" in n for n in kernels) == apart, kernels.keys()
