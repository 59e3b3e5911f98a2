"""Prefill where scores go on growing behind a row's first 32 keys.

The kernels take the exponents against a reference that moves to the sum's logarithm after every four tiles (128 keys),
and start a workgroup over only where a weight left the range of fp32.  Growth over many such windows, jumps in the
first, a middle and the last one, rows that are not numbers, large values, for 64 and 128 rows per workgroup, against
the fp64 oracle at the bar of the other prefill tests; and the time of growing scores against that of plain ones."""
import numpy as np
import pytest

from oracle.prefill_ref import prefill_attn_ref
from paper_2512_21450_amd import workloads as wl
from tests.test_gpu_prefill import B, case, run  # noqa: F401  (B is the fixture)
from tests.test_gpu_prefill_reference import SCALE, scaled
from tests.test_gpu_unit_batches import us_per_call

pytestmark = pytest.mark.gpu
SHAPES = [(3, 601, 16, 2), (24, 530, 16, 2)]                 # 64 and 128 rows per workgroup


def grown(bits, factors):
    """keys [.., L, d] times one factor per key"""
    f = wl.bf16_bits_to_f32(bits) * np.asarray(factors, np.float32)[:, None]
    return wl.f32_to_bf16_bits(f.astype(np.float32))


def check(B, x, v_size=1.0):  # noqa: F811
    out, lse = run(B, x, SCALE)
    ro, rl = prefill_attn_ref(x["q"], x["k"], x["v"], x["lens"], SCALE)
    valid = ~np.isnan(rl)
    assert np.isfinite(out).all() and (out[~valid] == -7.0).all()
    # lse: products of bf16 are exact, sums of 128 of them in fp32 err by less than 2^-20 of the score's size
    err_l = np.abs(lse[valid] - rl[valid]) / np.maximum(1.0, np.abs(rl[valid]) * 2.0 ** -10)
    assert np.abs(out[valid] - ro[valid]).max() / v_size <= 1e-2 and err_l.max() <= 1e-3


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("kind", ["steady", "in steps", "first window", "middle window", "last keys", "back and forth"])
def test_growth(B, kind, shape):  # noqa: F811
    P, L, Hq, Hkv = shape
    n = np.arange(L)
    f = {"steady": 1 + n * 0.03, "in steps": 2.0 ** (n // 128), "first window": np.where(n < 60, 1, 60.0),
         "middle window": np.where(n < 300, 1, 60.0), "last keys": np.where(n < L - 9, 1, 12.0),
         "back and forth": np.where((n // 64) % 2, 15.0, 0.1)}[kind]
    x = case(980, P, L, Hq, Hkv, lens=np.maximum(1, L - 11 * np.arange(P)))
    x["k"] = grown(x["k"], f)
    check(B, x)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_values_that_overflow_against_an_old_reference(B, shape):  # noqa: F811
    """Weights of some 2^30 before the reference moves, times 2^110; 2^8 times 2^110 is in range."""
    P, L, Hq, Hkv = shape
    x = case(981, P, L, Hq, Hkv)
    x["k"] = grown(x["k"], np.where(np.arange(L) < 160, 1, 7.0))
    x["v"] = scaled(x["v"], 2.0 ** 110)
    check(B, x, 2.0 ** 110)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_a_row_that_is_not_a_number_leaves_the_others_alone(B, shape):  # noqa: F811
    P, L, Hq, Hkv = shape
    x = case(982, P, L, Hq, Hkv, lens=[L] * P)
    x["k"] = grown(x["k"], 1 + np.arange(L) * 0.03)
    q = x["q"].copy()
    x["q"][1, 200, 3, 5] = np.uint16(0x7FC0)
    out, lse = run(B, x, SCALE)
    ro, rl = prefill_attn_ref(q, x["k"], x["v"], x["lens"], SCALE)
    assert np.isnan(out[1, 200, 3]).all()
    out[1, 200, 3] = ro[1, 200, 3]
    assert np.abs(out - ro).max() <= 1e-2


def test_growing_scores_take_no_longer_than_plain_ones(B):  # noqa: F811
    """1.8 times as long when every workgroup walked its tiles twice."""
    import torch
    P, L, Hq, Hkv = 32, 1280, 28, 4
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).bfloat16()
    q, k, v = rnd(P, L, Hq, 128), rnd(P, Hkv, L, 128), rnd(P, Hkv, L, 128)
    lens = torch.full((P,), L, dtype=torch.int32, device="cuda")
    out, lse = torch.empty((P, L, Hq, 128), device="cuda"), torch.empty((P, L, Hq), device="cuda")
    t = {}
    for gain in (1, 6, 12):
        kk = k.clone()
        kk[:, :, 32:] *= gain
        t[gain] = us_per_call(lambda: B.rl_prefill_attn(q, kk, v, lens, SCALE, out=out, lse=lse), n=4)
    print("\n", {a: round(b, 1) for a, b in t.items()})
    assert max(t[6], t[12]) <= 1.3 * t[1], t
