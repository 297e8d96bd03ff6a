"""Device assembly of the products on tiles of fewer columns: their accumulators, too, belong to the matrix instructions alone until well after the last."""
import re

from test_generated_code import assembly, basic_blocks, kernels, registers


def test_no_instruction_reads_an_accumulator_that_a_matrix_instruction_is_updating():
    checked = 0
    for name, code in kernels(assembly("gemm_bf16.hip")).items():
        if "gemm_bf16_narrow_kernel" not in name:
            continue
        checked += 1
        for block, _ in basic_blocks(code):
            since, last = 99, None                           # wait states since the last matrix instruction of this block, and its result
            for t in block:
                nop = re.match(r"s_nop (\d+)", t)
                if t.startswith("v_mfma"):
                    result = t.split()[1]
                    # two products in a row on one accumulator: something stands between them
                    assert result != last or since >= 1, (name, t)
                    since, last = 0, result
                    continue
                assert since >= 32 or not any(kind == "a" for kind, _ in registers(t)), (name, t)
                since += int(nop.group(1)) + 1 if nop else 1
    assert checked == 20


def test_the_narrow_products_spill_nothing():
    spills = re.findall(r"\.symbol:\s+(\S+)\.kd.*?\.vgpr_spill_count:\s+(\d+)", assembly("gemm_bf16.hip"), re.S)
    narrow = [s for s in spills if "gemm_bf16_narrow_kernel" in s[0]]
    assert len(narrow) == 20 and [s for s in narrow if int(s[1])] == []
