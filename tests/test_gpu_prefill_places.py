"""Prefill with few (prompt, KV head) units: their blocks are dealt out over all XCDs one by one.

The line lies at multiples of eight units and at 64 of them, so both sides of each, ragged lengths
(whole blocks of padding, an empty prompt) and the three kernels (64 and 128 rows per workgroup, a
scale that is not positive) are compared with the fp64 oracle at the bar of the other prefill tests.
"""
import math

import pytest

from tests.test_gpu_prefill import B, case, check  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # P, L_cap, Hq, Hkv
    (1, 70, 6, 1),          # one unit
    (1, 190, 14, 7),        # 7 units; r = 2
    (2, 130, 16, 4),        # 8: whole units
    (3, 100, 9, 3),         # 9
    (9, 67, 21, 7),         # 63: the last spread one
    (8, 67, 16, 8),         # 64
    (13, 66, 20, 5),        # 65: whole units, the last round not full
]


@pytest.mark.parametrize("ragged", [False, True], ids=["full", "ragged"])
@pytest.mark.parametrize("case_", CASES, ids=lambda c: "P{}L{}H{}-{}".format(*c))
def test_places(B, case_, ragged):  # noqa: F811
    P, L, Hq, Hkv = case_
    x = case(900 + CASES.index(case_), P, L, Hq, Hkv, lens=None if ragged else [L] * P)
    if ragged:
        x["lens"][0] = 0
        x["lens"][-1] = L
    check(B, x, 1.0 / math.sqrt(128), (case_, ragged))


def test_places_of_the_two_block_kernel(B):  # noqa: F811
    # 5 units, 8 * ceil(3000 / 8) workgroups: 128 rows each
    check(B, case(940, 5, 3000, 16, 1, lens=[0, 1, 97, 212, 300]), 1.0 / math.sqrt(128), "two blocks")


@pytest.mark.parametrize("scale", [-0.05, 0.0])
def test_places_of_the_register_staged_kernel(B, scale):  # noqa: F811
    check(B, case(950, 3, 150, 12, 3), scale, scale)
