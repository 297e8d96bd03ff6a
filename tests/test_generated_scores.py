"""Device assembly of the forward attention kernels, whose score products are assembly statements with results in ordinary registers.

The compiler does not know that such a result is still in the matrix pipe when its statement ends: a copy that it put right behind one would read
an old value now and then.  A 32x32x16 product is in the pipe for 8 issue slots, and another of them waits for the pipe; the instruction set asks
for a dozen wait states before anything else reads the result."""
import re

import pytest

from test_generated_code import assembly, basic_blocks, kernels, registers

NEEDED = 14
SCORES = re.compile(r"v_mfma_f32_32x32x16_\w+ (v\[\d+:\d+\]), ")


def early_reads(code):
    """Instructions other than matrix instructions on the same registers that touch a score product's result within NEEDED wait states, on any path."""
    blocks = basic_blocks(code)
    entry, work, faults = {0: {}}, [0], set()
    while work:
        b = work.pop()
        fresh = dict(entry[b])                               # register -> wait states since its product, the fewest over all paths
        for t in blocks[b][0]:
            m, nop = SCORES.match(t), re.match(r"s_nop (\d+)", t)
            touched = registers(t)
            if not m and touched & fresh.keys():
                faults.add(t)
            states = 8 if t.startswith("v_mfma_f32_32x32x16") else int(nop.group(1)) + 1 if nop else 1
            fresh = {r: n + states for r, n in fresh.items() if n + states < NEEDED}
            if m:
                fresh.update((r, 0) for r in registers(m.group(1)))
        for nxt in blocks[b][1]:
            old = entry.get(nxt)
            new = dict(old or {})
            for r, n in fresh.items():
                new[r] = min(n, new.get(r, n))
            if new != old:
                entry[nxt] = new
                work.append(nxt)
    return faults


def test_the_check_finds_planted_mistakes():
    product = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], 0"
    other = "v_mfma_f32_32x32x16_bf16 a[0:15], v[24:27], v[28:31], a[0:15]"
    use = "v_fma_f32 v40, v3, v41, v42"
    assert not early_reads([product, other, other, use, "s_endpgm"])
    assert not early_reads([product, "s_nop 15", use, "s_endpgm"])
    assert early_reads([product, use, "s_endpgm"]) == {use}
    assert early_reads([product, other, use, "s_endpgm"]) == {use}
    assert early_reads([product, "s_cbranch_scc1 .LBB0_1", other, other, ".LBB0_1:", use, "s_endpgm"]) == {use}
    assert early_reads([".LBB0_1:", use, "s_nop 15", product, "s_cbranch_scc1 .LBB0_1", "s_endpgm"]) == {use}


@pytest.mark.parametrize("dh", [32, 64, 96, 128, 160])
def test_no_instruction_reads_a_score_that_is_still_in_the_matrix_pipe(dh):
    checked = 0
    for name, code in kernels(assembly("attention_bf16.hip")).items():
        if f"attn_fwd_kernelILi{dh}E" not in name:
            continue
        checked += 1
        assert any(SCORES.match(t) for t in code), name
        assert not early_reads(code), (name, sorted(early_reads(code))[:4])
    assert checked == 4
