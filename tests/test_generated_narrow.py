"""Device assembly of the direct-to-LDS products: their accumulators belong to the matrix instructions alone until well after the last, on every path
through the code, and those on tiles of fewer columns spill nothing."""
import re

from test_generated_code import assembly, basic_blocks, kernels, registers

SETTLED = 32                                                 # wait states behind which an accumulator may be read by anything


def accumulator_faults(code):
    """Instructions that touch an accumulation register fewer than SETTLED wait states behind a matrix instruction, or, matrix instructions, that
    update the accumulator of the one right before them.  State: result of a matrix instruction -> wait states since the last of them, the fewest over all paths."""
    blocks = basic_blocks(code)
    entry, work, faults = {0: {}}, [0], set()
    while work:
        b = work.pop()
        since = dict(entry[b])
        for t in blocks[b][0]:
            nop = re.match(r"s_nop (\d+)", t)
            if t.startswith("v_mfma"):
                result = t.split()[1]
                if since.get(result) == 0:
                    faults.add(t)
                since = {r: n + 1 for r, n in since.items() if n + 1 < SETTLED}
                since[result] = 0
                continue
            if since and any(kind == "a" for kind, _ in registers(t)):
                faults.add(t)
            states = int(nop.group(1)) + 1 if nop else 1
            since = {r: n + states for r, n in since.items() if n + states < SETTLED}
        for nxt in blocks[b][1]:
            old = entry.get(nxt)
            new = dict(old or {})
            for r, n in since.items():
                new[r] = min(n, new.get(r, n))
            if new != old:
                entry[nxt] = new
                work.append(nxt)
    return faults


def test_the_check_finds_planted_mistakes():
    one, two = ("v_mfma_f32_16x16x32_bf16 a[%s], v[16:19], v[20:23], a[%s]," % (r, r) for r in ("0:3", "4:7"))
    read, wait = "v_accvgpr_read_b32 v1, a2", ["s_nop 15", "s_nop 15"]
    assert not accumulator_faults([one, two, one, "s_nop 0", one, *wait, read, "s_endpgm"])
    assert accumulator_faults([one, one, "s_endpgm"]) == {one}
    assert accumulator_faults([one, "s_nop 15", read, "s_endpgm"]) == {read}
    # behind the edge of a loop, at its start for the next pass, and on one of two paths
    assert not accumulator_faults([".LBB0_1:", one, two, "s_cbranch_scc1 .LBB0_1", *wait, read, "s_endpgm"])
    assert accumulator_faults([".LBB0_1:", one, two, "s_cbranch_scc1 .LBB0_1", "s_nop 15", read, "s_endpgm"]) == {read}
    assert accumulator_faults([".LBB0_1:", read, "s_nop 15", one, "s_cbranch_scc1 .LBB0_1", "s_endpgm"]) == {read}
    assert accumulator_faults([one, "s_cbranch_scc1 .LBB0_1", *wait, ".LBB0_1:", read, "s_endpgm"]) == {read}
    assert accumulator_faults([one, "s_branch .LBB0_1", ".LBB0_1:", one, "s_endpgm"]) == set()          # (the branch stands between)
    assert accumulator_faults([one, ".LBB0_1:", one, "s_endpgm"]) == {one}


def test_no_instruction_reads_an_accumulator_that_a_matrix_instruction_is_updating():
    checked = []
    for name, code in kernels(assembly("gemm_bf16.hip")).items():
        if "gemm_bf16_narrow_kernel" in name or "gemm_bf16_dma_kernel" in name:
            checked.append("narrow" in name)
            faults = accumulator_faults(code)
            assert not faults, (name, sorted(faults)[:4])
    assert checked.count(True) == 20 and checked.count(False) == 14


def test_the_narrow_products_spill_nothing():
    spills = re.findall(r"\.symbol:\s+(\S+)\.kd.*?\.vgpr_spill_count:\s+(\d+)", assembly("gemm_bf16.hip"), re.S)
    narrow = [s for s in spills if "gemm_bf16_narrow_kernel" in s[0]]
    assert len(narrow) == 20 and [s for s in narrow if int(s[1])] == []
