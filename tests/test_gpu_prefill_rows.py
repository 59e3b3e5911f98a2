"""The prefill writes its rows through the LDS, two to an instruction, and masks its scores in place: last blocks of one row,
of an odd number, of all but one and of all rows of a wavefront and of a workgroup, on both kernels, with rows beyond the
lengths untouched; against the fp64 oracle at the bar of the other prefill tests."""
import math

import pytest

from tests.test_gpu_prefill import B, case, check  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 3, 5, 7, 8, 16])
@pytest.mark.parametrize("rows", [64, 128])
def test_last_blocks(B, r, rows):  # noqa: F811
    block = rows // r                                      # positions of a workgroup
    part = max(1, rows // 4 // r)                          # and of one of its wavefronts
    lens = sorted({2 * block + n for n in (1, 2, part - 1, part, part + 1, block - 1, block, 2 * part + 1)} | {1, 31, 32, 33})
    # a capacity of many blocks takes the kernel of 128 rows (512 workgroups and 600 * 1024 row-tiles), a short one that of 64
    cap = 4000 if rows == 128 else max(lens) + 3
    P = len(lens)
    Hkv = 2 if rows == 64 or P * -(-cap // block) >= 700 else 4
    check(B, case(rows + r, P, cap, r * Hkv, Hkv, lens=lens), 1.0 / math.sqrt(128), (r, rows))
