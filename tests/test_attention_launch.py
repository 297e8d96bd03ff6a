"""The rule for the forward kernels' workgroups, called on the host: 128 queries where workgroups of 256 are few or half empty, and never more than a launch holds."""
import ctypes as C

import pytest

from paper_2106_02679_amd import binding as B

SUBBLOCKS = B.lib["_ZN3lga18attn_fwd_subblocksERKNS_9AttnShapeE"]


def subblocks(n_seq, s, heads, dh, causal):
    return SUBBLOCKS((C.c_int * 5)(n_seq, s, heads, dh, causal))


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("dh", [8, 64, 72, 160])
@pytest.mark.parametrize("s", [1, 128, 129, 257, 300, 384, 600, 640])
def test_a_launch_has_fewer_than_two_to_the_32_work_items(s, dh, causal):
    """Wherever workgroups of 256 queries fit a launch, those that are chosen do."""
    seen = set()
    for n_seq in (1, 4096, 5591, 5592, 5593, 5700, 8191, 8388, 16383, 16384, 16777, 20000):
        for heads in (1, 100, 1000, 1024):
            u = subblocks(n_seq, s, heads, dh, causal)
            blocks = {w: n_seq * heads * -(-s // (128 * w)) for w in (1, 2)}
            assert u in (1, 2) and (256 * blocks[u] < 2**32 or 256 * blocks[2] >= 2**32), (n_seq, heads, u)
            seen.add(u)
    assert 1 in seen


@pytest.mark.parametrize("n_seq,s,heads,dh,causal,u", [
    (4, 1024, 12, 64, 1, 1), (32, 1024, 12, 64, 1, 2), (1, 1000, 28, 152, 1, 1), (2, 1000, 28, 152, 1, 1), (4, 1000, 28, 152, 1, 2),
    (1, 8100, 16, 128, 1, 2), (8, 1024, 32, 128, 0, 2), (1, 128, 2, 64, 1, 1),
    # one workgroup of 256 queries a sequence: two short ones only in one round, or where several share a compute unit
    (12, 137, 12, 112, 1, 2), (6, 132, 24, 128, 1, 2), (4, 153, 88, 48, 0, 2), (3, 236, 57, 96, 1, 2), (1, 129, 129, 72, 0, 2), (1, 256, 129, 72, 0, 2),
    (1, 137, 128, 112, 1, 1), (1, 137, 128, 48, 0, 1), (6, 210, 27, 48, 1, 1), (11, 216, 29, 32, 1, 1), (1, 128, 129, 112, 1, 1), (1, 257, 70, 112, 1, 1)])
def test_few_workgroups_are_short_ones(n_seq, s, heads, dh, causal, u):
    assert subblocks(n_seq, s, heads, dh, causal) == u
