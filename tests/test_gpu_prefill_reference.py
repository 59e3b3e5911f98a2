"""Prefill where the maximum of a row's first 32 keys is a poor reference for its softmax.

The kernels take the exponents against that maximum, move it to the sums after every four tiles, and start
a workgroup over, with the reference following the running maximum, where a sum or an accumulator left its
range.  Both ways, and rows of both kinds in one workgroup, against the fp64 oracle at the bar of the other
prefill tests (1e-2 abs on out for values of unit size, 1e-3 abs on lse), for 64 and 128 rows per workgroup.
"""
import math

import numpy as np
import pytest

from oracle.prefill_ref import prefill_attn_ref
from paper_2512_21450_amd import workloads as wl
from tests.test_gpu_prefill import B, case, run  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu

SCALE = 1.0 / math.sqrt(128)
SHAPES = [(3, 150, 16, 2), (64, 260, 16, 2)]                 # 64 and 128 rows per workgroup


def scaled(bits, f):
    return wl.f32_to_bf16_bits((wl.bf16_bits_to_f32(bits) * f).astype(np.float32))


def set_up(kind, shape):
    P, L, Hq, Hkv = shape
    x = case(970, P, L, Hq, Hkv, lens=np.maximum(1, L - 7 * np.arange(P) % L))
    v_size = 1.0
    if kind == "later keys somewhat larger":                 # sums beyond 2^8, far inside the range
        x["k"][:, :, 32:] = scaled(x["k"][:, :, 32:], 6.0)
    elif kind == "later keys far larger":                    # scores tens of nats above the first tile's
        x["k"][:, :, 40:] = scaled(x["k"][:, :, 40:], 60.0)
    elif kind == "first keys far larger":
        x["k"][:, :, :32] = scaled(x["k"][:, :, :32], 60.0)
    elif kind == "one query row":                            # the others of its workgroup stay ordinary
        x["q"][0, 100, 3] = scaled(x["q"][0, 100, 3], 60.0)
        x["k"][0, :, :32] = scaled(x["k"][0, :, :32], 0.02)
    else:                                                    # weights of some 2^20 times 2^112; 2^8 times 2^112 is in range
        x["k"][:, :, 32:] = scaled(x["k"][:, :, 32:], 6.0)
        v_size = 2.0 ** 112
        x["v"] = scaled(x["v"], v_size)
    return x, v_size


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("kind", ["later keys somewhat larger", "later keys far larger", "first keys far larger",
                                  "one query row", "large values"])
def test_reference(B, kind, shape):  # noqa: F811
    x, v_size = set_up(kind, shape)
    out, lse = run(B, x, SCALE)
    ro, rl = prefill_attn_ref(x["q"], x["k"], x["v"], x["lens"], SCALE)
    valid = ~np.isnan(rl)
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    assert (out[~valid] == -7.0).all() and (lse[~valid] == -7.0).all()
    # lse: products of bf16 are exact, sums of 128 of them in fp32 err by less than 2^-20 of the score's size
    err_l = np.abs(lse[valid] - rl[valid]) / np.maximum(1.0, np.abs(rl[valid]) * 2.0 ** -10)
    assert np.abs(out[valid] - ro[valid]).max() / v_size <= 1e-2 and err_l.max() <= 1e-3
