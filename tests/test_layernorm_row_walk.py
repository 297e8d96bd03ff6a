"""Row counts at the end of what an int32 holds: which rows the wavefronts of the narrow LayerNorm kernels take, and how much scratch the backward
pass asks for.  On the host - tensors of so many rows take 34 GB each."""
import os
import shutil
import subprocess

import pytest

from paper_2106_02679_amd import binding as B
from paper_2106_02679_amd import build as bld

TOP = 2 ** 31 - 1

WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "row_walk.h"
int main(int argc, char **argv) {
    const int rows = atoi(argv[1]), most = atoi(argv[2]);
    if (!lga::row_walk_takes(rows)) return 2;
    if (most > lga::kMostWalkBlocks) return 3;
    const int blocks = lga::row_walk_blocks(rows, most);
    size_t walked = 0; int last = 0;
    for (int b : {0, blocks / 2, blocks - 1})
        for (unsigned wave = 0; wave < 4; ++wave) {
            if (b < 0) continue;
            lga::RowWalk w((unsigned)b, (unsigned)blocks, wave, rows);
            for (; w.valid(); w.advance()) {
                if (w.row < 0 || w.row >= rows || (w.has_next() && (w.next() < 0 || w.next() >= rows))) return 1;
                ++walked;
                if (w.row > last) last = w.row;
            }
        }
    printf("%d %zu %d\n", blocks, walked, last);
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("walk")
    (d / "walk.cpp").write_text(WALK)
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-ftrapv", "-I", bld.CSRC, str(d / "walk.cpp"), "-o", str(d / "walk")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return str(d / "walk")


@pytest.mark.parametrize("most", [2048, 1024])
@pytest.mark.parametrize("rows", [0, 1, 3, 4, 5, 8191, 8192, 8193, 10 ** 9, TOP - 8192 - 4096, TOP - 8192 - 1, TOP - 8192])
def test_every_row_of_a_wavefront_lies_inside_and_the_walk_ends(walk, rows, most):
    res = subprocess.run([walk, str(rows), str(most)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, "a row outside, or an index beyond an int"
    blocks, walked, last = map(int, res.stdout.split())
    assert blocks == min((rows + 3) // 4, most)
    seen = sum(len(range(4 * b + w, rows, 4 * blocks)) for b in (0, blocks // 2, blocks - 1) if b >= 0 and blocks for w in range(4))
    assert walked == seen and last == max([r for b in {0, blocks // 2, blocks - 1} if blocks and b >= 0 for w in range(4)
                                           for r in range(4 * b + w, rows, 4 * blocks)[-1:]], default=0)


@pytest.mark.parametrize("rows", [TOP - 8191, TOP - 3, TOP])
def test_more_rows_are_left_to_the_kernels_that_count_them_in_64_bits(walk, rows):
    assert subprocess.run([walk, str(rows), "2048"], timeout=60).returncode == 2


@pytest.mark.parametrize("d", [8, 64, 512])
@pytest.mark.parametrize("rows", [TOP - 4, TOP - 3, TOP - 2, TOP - 1, TOP])
def test_scratch_of_the_backward_pass_at_the_largest_row_counts(rows, d):
    chunks = -(-rows // 128)                                 # the column sums' own first pass, the larger need at so many rows
    assert B.lib.lga_op_layernorm_bwd_scratch_floats(rows, d) == chunks * 2 * d
