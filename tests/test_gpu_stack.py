"""Decode stacks by data flow: the sizes where the split can go wrong.  Every layer of every sequence
against the oracle, and kept score rows against rows that stay inside the workspace, bit for bit."""
import pytest

from paper_2408_01890_amd import patterns as pt
from paper_2408_01890_amd import synth
from tests.test_gpu_parity import log, run_pattern_stack

pytestmark = pytest.mark.gpu

MIXED = (pt.STD, pt.LISA, pt.SHARE, pt.LISA, pt.STD, pt.SHARE, pt.SHARE, pt.LISA, pt.LISA, pt.LISA, pt.LISA, pt.STD)
# more layers than one group takes (48): the row passes from group to group, to a LiSA layer and, through
# layers that share directly, from one group to the one after the next
LONG = (pt.STD,) + (pt.LISA,) * 49 + (pt.STD,)
LONG_SHARE = (pt.STD, pt.LISA) + (pt.SHARE,) * 96 + (pt.LISA, pt.SHARE, pt.STD)

CASES = [  # H, Hkv, ctx, d_k, r, F, B, Lmax, dim_major, kinds
    (8, 8, 15, 128, 22, 16, 1, 16, True, MIXED),       # one split, one block of positions
    (8, 4, 127, 128, 7, 32, 2, 128, True, MIXED),      # exactly one split; odd rank; two heads per kv head
    (40, 40, 128, 128, 22, 80, 1, 131, True, MIXED),   # one key in the second split; rows that are not 16-byte aligned
    (16, 4, 300, 64, 20, 33, 2, 320, False, MIXED),    # row-major K_LR, d_k = 64, four heads per kv head
    (40, 8, 257, 128, 22, 80, 1, 264, True, MIXED),    # five heads per kv head
    (64, 2, 64, 64, 16, 128, 1, 72, True, MIXED),      # widest chain; 32 heads per kv head
    (33, 33, 40, 64, 3, 100, 1, 48, True, MIXED),      # heads in a block of their own
    (8, 8, 20, 64, 12, 16, 1, 24, True, LONG),
    (8, 8, 140, 64, 12, 16, 1, 144, True, LONG_SHARE),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"h{c[0]}_{c[1]}_ctx{c[2]}_dk{c[3]}_f{c[5]}_n{len(c[9])}")
def test_decode_stack_sizes(case):
    H, Hkv, ctx, dk, r, F, B, Lmax, dim_major, kinds = case
    log(f"[case] stack {case[:9]} {len(kinds)} layers")
    # (the identity-like FFN of the shared inputs needs F >= 2H)
    stk = synth.DecodeStack(f"stack_h{H}_ctx{ctx}", "bf16", B, H, Hkv, ctx, 256, dk, r, max(F, 2 * H), len(kinds), 1)
    run_pattern_stack(stk, kinds, list(range(B)), dim_major=dim_major, Lmax=Lmax)
