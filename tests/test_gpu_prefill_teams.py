"""The prefill of few, long blocks: two teams of wavefronts share a block's tiles.  Numbers of tiles around multiples of the
four that the teams take in turn (blocks whose second team has two tiles, one, none more, or only tiles in the future of some
rows), blocks of few tiles, which the first team takes alone (up to eight), both sides of the rule's lines (640, 896, 1024 and 1280
rows of capacity with 8, 9, 10 and 12 blocks to six compute units), scores that move the reference and scores that
make a workgroup start over; against the fp64 oracle at the bar of the other prefill tests."""
import math

import numpy as np
import pytest

from tests.test_gpu_prefill import B, case, check, run  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (7, 1), (8, 1), (6, 2)])
@pytest.mark.parametrize("cap", [639, 640, 700])
def test_numbers_of_tiles(B, Hq, Hkv, cap):  # noqa: F811
    lens = [1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 160, 193, 225, 0, cap,
            255, 256, 257, 288, 289, 320, 321, 352, 353, 384, 385, 416, 417, 448, 545, 608]
    for i in range(0, len(lens), 4):                               # few prompts, so that all blocks find a place at once
        x = case(cap + i + Hq, 4, cap, Hq, Hkv, lens=lens[i:i + 4])
        check(B, x, 1.0 / math.sqrt(128), (Hq, Hkv, cap, lens[i:i + 4]))


# (prompts, capacity): blocks of eight positions on either side of 8, 9, 10 and 12 to six compute units
@pytest.mark.parametrize("P,cap", [(2, 2048), (2, 2056), (4, 680), (4, 688), (3, 888), (3, 896), (3, 1016), (3, 1024), (3, 1032), (3, 1136),
                                   (3, 1144), (3, 1272), (3, 1280), (3, 1360), (3, 1368)])
def test_both_sides_of_the_blocks_a_compute_unit(B, P, cap):  # noqa: F811
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    teams = (P, cap) not in ((2, 2056), (4, 688), (3, 1144), (3, 1272), (3, 1368))
    assert cus != 256 or (B.rl_prefill_attn_debug_form(B.make_prefill_desc(1, P, 8, 1, 128, cap, 0.1), cus) == 3) == teams
    check(B, case(cap, P, cap, 8, 1, lens=[300, 555, 0, 640][:P]), 1.0 / math.sqrt(128), (P, cap))


@pytest.mark.parametrize("gain", [6.0, 60.0])
@pytest.mark.parametrize("first", [32, 64, 100])
@pytest.mark.parametrize("L", [530, 210])                          # 17 tiles, of both teams; 7, of the first and half a round over
def test_growing_scores(B, gain, first, L):  # noqa: F811
    """Keys past the first ones `gain` times as large: the reference follows the sums, or the workgroup starts over."""
    x = case(int(gain) + first, 1, 700, 8, 1, lens=[L])
    k = (x["k"].astype(np.uint32) << 16).view(np.float32).copy()
    k[:, :, first:] *= gain
    x["k"] = (k.view(np.uint32) >> 16).astype(np.uint16)
    check(B, x, 1.0 / math.sqrt(128), (gain, first, L))


def test_run_to_run(B):  # noqa: F811
    x = case(5, 1, 900, 8, 2, lens=[871])
    a, b = run(B, x, 0.1), run(B, x, 0.1)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
