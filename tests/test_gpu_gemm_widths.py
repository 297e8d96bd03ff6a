"""Products on tiles of 256 x 192 and 256 x 128: sizes at the edges of tiles (one row and one column of 8 more and less), k ranges that end inside
a k tile and around the unrolled part of the loop, every epilogue, against the same rows multiplied a few at a time - which the small kernel does, in
the same order of every sum - bit for bit, and against 64 bits within the rounding of the result."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import profiled
from test_gpu_ops import BF16, F16

TYPE = {BF16: torch.bfloat16, F16: torch.float16}
# (M, N, K) and the columns of a tile: whole tiles, and 8 rows and columns more and less; a round and several, full and part; k ranges of less than the unrolled part of the
# loop, of it with a k tile of 8 behind it, and of more
SIZES = [(32768, 384, 72, 192), (32760, 376, 520, 192), (2000, 4256, 704, 192), (2008, 4232, 840, 192), (1992, 4216, 1032, 192), (8200, 1160, 584, 192),
         (8184, 1144, 584, 192), (6400, 1152, 1024, 128), (6392, 1160, 1000, 128), (9216, 512, 704, 128), (9208, 504, 776, 128), (9208, 520, 776, 128),
         (4616, 1032, 712, 128)]


def product(dt, epi, a, w, out, out2, bias, aux, M, N, K):
    B.check(B.lib.lga_op_gemm(dt, 1, 1, epi, M, N, K, a.data_ptr(), K, w.data_ptr(), K, out.data_ptr(), out2.data_ptr() if epi == 3 else None, None, N,
                              bias.data_ptr(), aux.data_ptr(), 0.0, None))


@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_a_row_does_not_depend_on_the_width_of_the_tiles(size, dt):
    M, N, K, columns = size
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a, aux = (torch.randn(M, k, device="cuda", generator=g).to(TYPE[dt]) for k in (K, N))
    w = (torch.randn(N, K, device="cuda", generator=g) / K**0.5).to(TYPE[dt])
    bias = torch.randn(N, device="cuda", generator=g)
    rows = sorted({0, 8, 120, 248, 256, M // 2 // 8 * 8, M - 264, M - 8})
    for epi in range(5):
        out, out2 = (torch.full((M + 8, N), float("nan"), device="cuda", dtype=TYPE[dt]) for _ in range(2))
        kernels = profiled(lambda: product(dt, epi, a, w, out, out2, bias, aux, M, N, K))
        assert list(kernels) == [f"gemm_{'bf16' if dt == BF16 else 'f16'}_dma_kernel<256, {columns}, {epi}>"]
        part, part2 = (torch.full((8, N), float("nan"), device="cuda", dtype=TYPE[dt]) for _ in range(2))
        for r in rows:
            (small,) = profiled(lambda: product(dt, epi, a[r:r + 8], w, part, part2, bias, aux[r:r + 8], 8, N, K))
            assert "small" in small
            assert torch.equal(out[r:r + 8], part), (epi, r)
            assert epi != 3 or torch.equal(out2[r:r + 8], part2), (epi, r)
        assert out[M:].isnan().all() and out2[M:].isnan().all(), epi        # nothing behind the last row
        assert not out[:M].isnan().any(), epi
        u = a.double() @ w.double().t()
        if epi in (1, 2, 3): u += bias.double()
        if epi == 2: u += aux.double()
        if epi == 3: u = torch.nn.functional.gelu(u, approximate="tanh")
        if epi == 4:
            x = aux.double().requires_grad_()
            torch.nn.functional.gelu(x, approximate="tanh").sum().backward()
            u *= x.grad
        err = (torch.linalg.norm(out[:M].double() - u) / torch.linalg.norm(u)).item()
        assert err <= (2.0**-9 if dt == BF16 else 2.0**-12) + 1e-5, (epi, err)
