"""Column sums and transposes of one matrix on either side of the lines of their launch rules: 128 chunks of 128 rows (one or four columns
per thread in the second pass) and 65535 (a two- or a one-dimensional grid).  Small whole numbers, so that every sum is exact
in fp32 whatever its order."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B

ROWS = [1, 128 * 128, 128 * 128 + 1, 128 * 65535, 128 * 65535 + 8]


def matrix(rows, cols, dtype):
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    return torch.randint(-1, 2, (rows, cols), device="cuda", generator=gen, dtype=torch.int8).to(dtype)


@pytest.mark.parametrize("cols", [8, 12])
@pytest.mark.parametrize("rows", ROWS)
def test_column_sums_of_one_matrix(rows, cols):
    for code, dtype in ((B.LGA_BF16, torch.bfloat16), (B.LGA_FP32, torch.float32)):
        a = matrix(rows, cols, dtype)
        want = a.sum(0, dtype=torch.float64)
        scratch = torch.empty(int(B.lib.lga_op_colsum_scratch_floats(rows, cols)) + 1, device="cuda")
        for shift in (0, 1):                                  # the scratch need not be aligned
            out = torch.ones(cols, device="cuda")
            B.check(B.lib.lga_op_colsum(code, a.data_ptr(), rows, cols, cols, 2.0, out.data_ptr(), scratch.data_ptr() + 4 * shift, None))
            torch.cuda.synchronize()
            assert torch.equal(out.double(), want + 2), (dtype, shift)


@pytest.mark.parametrize("rows", [8, 128 * 128, 128 * 128 + 8, 128 * 65535, 128 * 65535 + 8])
def test_transpose_of_one_matrix(rows):
    cols = 16
    a, out, sums = matrix(rows, cols, torch.bfloat16), torch.empty(cols, rows, device="cuda", dtype=torch.bfloat16), torch.ones(cols, device="cuda")
    B.check(B.lib.lga_op_transpose(a.data_ptr(), out.data_ptr(), rows, cols, cols, rows, None))
    torch.cuda.synchronize()
    assert torch.equal(out, a.T)
    out.zero_()
    scratch = torch.empty(int(B.lib.lga_op_colsum_scratch_floats(rows, cols)), device="cuda")
    B.check(B.lib.lga_op_transpose_colsum(B.LGA_BF16, a.data_ptr(), out.data_ptr(), rows, cols, cols, rows, 1.0, sums.data_ptr(),
                                          scratch.data_ptr(), None))
    torch.cuda.synchronize()
    assert torch.equal(out, a.T) and torch.equal(sums.double(), a.sum(0, dtype=torch.float64) + 1)


@pytest.mark.parametrize("dtype,cols", [(torch.bfloat16, 1016), (torch.bfloat16, 1024), (torch.bfloat16, 2288), (torch.bfloat16, 2296), (torch.float16, 1024),
                                        (torch.float32, 508), (torch.float32, 512), (torch.float32, 513)])
@pytest.mark.parametrize("rows", [16456, 16384])
def test_a_column_does_not_depend_on_how_many_share_the_launch(rows, cols, dtype):
    """On either side of the 32 MB and 72 MB up to and from which rows are requested ahead: the order of a column's sums is the same as in a few columns of it."""
    code = {torch.bfloat16: B.LGA_BF16, torch.float16: B.LGA_FP16, torch.float32: B.LGA_FP32}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    a = torch.randn(rows, cols, device="cuda", generator=gen).to(dtype)

    def sums(at, n):
        out, scratch = torch.ones(n, device="cuda"), torch.empty(int(B.lib.lga_op_colsum_scratch_floats(rows, n)), device="cuda")
        B.check(B.lib.lga_op_colsum(code, a[:, at:].data_ptr(), rows, n, cols, 0.5, out.data_ptr(), scratch.data_ptr(), None))
        torch.cuda.synchronize()
        return out

    whole = sums(0, cols)
    few = 9 if cols % 8 == 1 else 16                         # (the second pass takes four columns a thread where their number allows)
    for at in (0, cols // 2 // 8 * 8, (cols - few) // 8 * 8):
        assert torch.equal(whole[at:at + few], sums(at, few)), at
    want = a.double().sum(0) + 0.5
    assert (whole.double() - want).abs().max() <= 2.0**-24 * 200 * a.abs().double().sum(0).max()         # 16 + 8 and some 100 additions one behind another
