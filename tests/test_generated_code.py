"""Device assembly of the kernels whose transposing LDS reads are assembly statements.

The compiler does not know that such a read is still in flight when its statement ends, so nothing but the waits in the source keeps an
instruction from using the result too early - a copy or a spill that a compiler puts in between would carry a wrong value and
nothing would fail loudly.  These tests read the assembly generated from the sources and follow the LDS counter through
every path."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2106_02679_amd import build as bld

TR_READ = re.compile(r"ds_read_b64_tr_b16 (v\[\d+:\d+\]|v\d+), ")
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


@functools.lru_cache(maxsize=None)
def assembly(source):
    hipcc = bld._hipcc()
    if shutil.which(hipcc) is None and not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in bld.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "device.s")
        res = subprocess.run([hipcc, *flags, "-S", "--cuda-device-only", os.path.join(bld.CSRC, source), "-o", out],
                             capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-2000:]
        with open(out) as f:
            return f.read()


def kernels(text):
    """name -> its lines of code: labels ("x:") and instructions."""
    out, name = {}, None
    for line in text.splitlines():
        t = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):$", t)
        if m:
            name = m.group(1)
            out[name] = []
        elif t.startswith(".Lfunc_end"):
            name = None
        elif name and t and (t.endswith(":") or not t.startswith(".")):
            out[name].append(t)
    return out


@functools.lru_cache(maxsize=None)
def registers(text):
    regs = set()
    for kind, lo, hi, one in REG.findall(text):
        regs.update((kind, r) for r in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return frozenset(regs)


def basic_blocks(code):
    """[(instructions, successors)], blocks[0] the entry."""
    blocks, labels = [[]], {}
    for t in code:
        if t.endswith(":"):
            if blocks[-1]:
                blocks.append([])
            labels[t[:-1]] = len(blocks) - 1
        else:
            blocks[-1].append(t)
            if t.startswith(("s_cbranch", "s_branch", "s_endpgm")):
                blocks.append([])
    out = []
    for i, block in enumerate(blocks):
        last = block[-1] if block else ""
        after = [labels[last.split()[1]]] if last.startswith(("s_cbranch", "s_branch")) else []
        if not last.startswith(("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            after.append(i + 1)
        out.append((block, after))
    return out


def back_edges(blocks):
    """Edges to a block that is still open in a depth-first walk: where loops close."""
    edges, state, stack = set(), {0: "open"}, [(0, iter(blocks[0][1]))]
    while stack:
        b, it = stack[-1]
        nxt = next(it, None)
        if nxt is None:
            state[b] = "done"
            stack.pop()
        elif nxt not in state:
            state[nxt] = "open"
            stack.append((nxt, iter(blocks[nxt][1])))
        elif state[nxt] == "open":
            edges.add((b, nxt))
    return edges


def in_flight_faults(code):
    """(uses, loops): instructions that touch a register whose transposing read may not have returned, and the ends of loop bodies with
    such reads outstanding.  State: register -> LDS operations issued after its read, the fewest over all paths; LDS operations return in
    order, so a wait for n outstanding ones completes the reads with n or more behind them.  (A scalar load counts in the same
    counter and may return out of order: with one outstanding only a wait for zero completes anything.)"""
    blocks = basic_blocks(code)
    closing = back_edges(blocks)
    entry = [None] * len(blocks)
    entry[0] = ({}, 0)
    work, uses, loops = [0], set(), set()
    while work:
        b = work.pop()
        flight, scalar = dict(entry[b][0]), entry[b][1]
        for t in blocks[b][0]:
            op = t.split()[0]
            touched = registers(t) & flight.keys()
            if touched:
                uses.add(t)
                for r in touched:
                    del flight[r]
            if op.startswith("ds_"):
                flight = {r: min(n + 1, 64) for r, n in flight.items()}
                m = TR_READ.match(t)
                if m:
                    flight.update((r, 0) for r in registers(m.group(1)))
            elif op.startswith(("s_load", "s_buffer_load")):
                scalar = 1
            elif op == "s_waitcnt":
                w = re.search(r"lgkmcnt\((\d+)\)", t)
                n = int(w.group(1)) if w else 64
                if n == 0:
                    flight, scalar = {}, 0
                elif not scalar:
                    flight = {r: k for r, k in flight.items() if k < n}
        for nxt in blocks[b][1]:
            if flight and (b, nxt) in closing:
                loops.add((blocks[b][0][-1], len(flight)))
            old = entry[nxt]
            new = (dict(flight), scalar) if old is None else (dict(old[0]), old[1] | scalar)
            if old is not None:
                for r, n in flight.items():
                    new[0][r] = min(n, new[0].get(r, n))
            if new != old:
                entry[nxt] = new
                work.append(nxt)
    return uses, loops


def test_the_check_finds_planted_mistakes():
    read = "ds_read_b64_tr_b16 v[2:3], v9 offset:64"
    ok = [read, "ds_read_b128 v[4:7], v8", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v1, v2", "s_endpgm"]
    assert in_flight_faults(ok) == (set(), set())
    assert in_flight_faults([read, "v_mov_b32_e32 v1, v3", "s_endpgm"])[0] == {"v_mov_b32_e32 v1, v3"}
    assert in_flight_faults([read, "s_waitcnt lgkmcnt(1)", "v_accvgpr_write_b32 a0, v2", "s_endpgm"])[0]
    assert in_flight_faults([read, "s_waitcnt vmcnt(0)", "scratch_store_dword off, v2, off", "s_endpgm"])[0]
    assert in_flight_faults(["s_load_dword s4, s[0:1], 0x0"] + ok)[0]                      # out of order with a scalar load
    loop = [".LBB0_1:", read, "s_cbranch_scc1 .LBB0_1", "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v1, v2", "s_endpgm"]
    uses, loops = in_flight_faults(loop)
    assert loops == {("s_cbranch_scc1 .LBB0_1", 2)} and uses == {read}                     # the next pass overwrites v[2:3] in flight
    around = [read, "s_cbranch_scc1 .LBB0_2", "s_waitcnt lgkmcnt(0)", ".LBB0_2:", "v_mov_b32_e32 v1, v2", "s_endpgm"]
    assert in_flight_faults(around)[0] == {"v_mov_b32_e32 v1, v2"}                         # one of two paths lacks the wait


@pytest.mark.parametrize("source,min_reads", [("gemm_bf16.hip", 600), ("attention_bf16.hip", 1000), ("attention_wide.hip", 1000)])
def test_no_instruction_touches_a_transposing_read_in_flight(source, min_reads):
    reads = 0
    for name, code in kernels(assembly(source)).items():
        n = sum(1 for t in code if TR_READ.match(t))
        reads += n
        if n == 0:
            continue
        uses, loops = in_flight_faults(code)
        assert not uses, (name, sorted(uses)[:4])
        # a value that is carried around a loop is where a compiler puts copies: no read may be in flight there
        assert not loops, (name, sorted(loops)[:4])
    assert reads >= min_reads, reads


def test_no_instruction_reads_an_accumulator_that_a_matrix_instruction_is_updating():
    """The direct-to-LDS GEMM's matrix instructions are assembly too: a move that the compiler puts between two of them on an accumulation
    register would read it before the update has left the matrix pipe."""
    checked = 0
    for name, code in kernels(assembly("gemm_bf16.hip")).items():
        if "gemm_bf16_dma_kernel" not in name:
            continue
        checked += 1
        for block, _ in basic_blocks(code):
            since = 99                                       # wait states since the last matrix instruction of this block
            for t in block:
                nop = re.match(r"s_nop (\d+)", t)
                if t.startswith("v_mfma"):
                    since = 0
                    continue
                assert since >= 32 or not any(kind == "a" for kind, _ in registers(t)), (name, t)
                since += int(nop.group(1)) + 1 if nop else 1
    assert checked == 14


def test_the_attention_kernels_up_to_160_channels_spill_nothing():
    """A spilled register is reloaded with the counter that the tiles in flight use: a reload inside the loop over the tiles waits for the
    next tile before the present one is multiplied."""
    spills = re.findall(r"\.symbol:\s+(\S+)\.kd.*?\.vgpr_spill_count:\s+(\d+)", assembly("attention_bf16.hip"), re.S)
    assert len(spills) >= 30
    assert [s for s in spills if int(s[1])] == []
