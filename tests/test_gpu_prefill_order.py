"""Prefill with more than a round of blocks, two per compute unit: every block of every prompt is computed once, whatever the order in
which they are dealt out. The cases are on either side of each line of the rule (on 256 compute units): eight units in groups of four
XCDs from 1.5 rounds on, 16 and 24 in pairs with a chunk of four and three from two rounds on, 32 and, with up to 32 blocks each, more
of them in chunks where few heads share a KV head, with four of them up to some numbers of rounds, of 64 and of 128 rows to a
workgroup, also a last chunk and a last round that are not full; against the fp64 oracle at the bar of the other prefill tests.
Capacities are far longer than the prompts: what is checked is the order, and the oracle's time goes with the lengths."""
import math

import pytest

from tests.test_gpu_prefill import B, case, check  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,L,Hq,Hkv", [
    (8, 600, 16, 1), (4, 1200, 16, 2), (8, 390, 16, 1), (8, 380, 16, 1), (4, 1700, 16, 2),   # 8 units: more than 1.5 rounds, the last one fewer
    (16, 450, 16, 1), (8, 1300, 16, 2), (8, 1000, 14, 2), (4, 300, 64, 4), (4, 200, 64, 4),         # 16: more than two rounds, the last one fewer
    (24, 256, 8, 1), (6, 400, 32, 4), (6, 150, 64, 4),                # 24, the same
    (16, 300, 16, 2), (8, 600, 8, 4), (16, 400, 8, 2), (16, 600, 16, 2),      # 32: 64 rows, the second and third in chunks; 128 rows
    (8, 1024, 8, 8), (20, 300, 6, 2), (10, 260, 64, 8), (10, 256, 64, 8),         # more, 40 and 80: 64 rows, the first in chunks
    (20, 220, 10, 5), (16, 700, 20, 5), (8, 1280, 8, 8), (5, 300, 32, 8), (11, 600, 32, 8),      # 64 and 128 rows, all in chunks
    (20, 140, 20, 5), (22, 600, 32, 8), (12, 300, 32, 8),                # four heads: not in chunks, beyond six rounds and three
    (67, 300, 2, 1), (67, 128, 7, 1), (13, 260, 20, 5), (11, 512, 12, 6)], ids=str)    # not a multiple of eight: 67, 65, 66
def test_order(B, P, L, Hq, Hkv):  # noqa: F811
    lens = [(37 * p * p + 11 * p) % min(L, 150) for p in range(P)]    # ragged, one of them empty
    lens[-1] = min(L, 210)
    check(B, case(L + Hq, P, L, Hq, Hkv, lens=lens), 1.0 / math.sqrt(128), (P, L, Hq, Hkv))


def test_blocks_that_all_have_work(B):  # noqa: F811
    check(B, case(7, 8, 320, 16, 2, lens=[320] * 8), 1.0 / math.sqrt(128), "16 units")
    check(B, case(8, 8, 130, 64, 8, lens=[130] * 8), 1.0 / math.sqrt(128), "64 units")
