"""The one-launch decode kernel where the score factor is far from 1 / sqrt(d): any finite scale, and factors of an e4m3
store from very small to large, against the fp64 oracle.

The softmax of scores that are far apart is the value row of the largest one, so out is compared with the same bar as
everywhere; inputs are chosen so that no two scores of a row are closer than the rounding of a 32-bit product q . k
times the factor (checked).  lse is a large number then: relative."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2512_21450_amd import binding
    return binding


def separated(seed, P, G, Hq, Hkv, d, Lp, Ls, dtype):
    """Products q . k that are whole numbers, hence exact in 32 bits, and ties only where the values tie as well:
    key rows are distinct multiples of one row."""
    rng = np.random.default_rng(seed)
    x = util.random_case(seed, P, G, Hq, Hkv, d, Lp, Ls, dtype, plens=np.full(P, Lp), slens=rng.integers(1, Ls + 1, P * G))
    narrow = (lambda a: a) if dtype == "f32" else wl.f32_to_bf16_bits
    t = lambda a: narrow(np.ascontiguousarray(a, dtype=np.float32))
    sign = rng.choice([-1.0, 1.0], d)
    x["q"] = t(np.broadcast_to(sign, (P * G, Hq, d)))
    ids = rng.permutation(Lp + Ls)                                        # < 256: exact in bf16
    k = (ids - 100.0)[:, None] * sign
    x["k_prefix"] = t(np.broadcast_to(k[:Lp], (P, Hkv, Lp, d)))
    x["k_suffix"] = t(np.broadcast_to(k[Lp:], (P * G, Hkv, Ls, d)))
    return x


@pytest.mark.parametrize("scale", [1e9, -1e9, 1e20, -3e33, 1e-30, -1e-38, 1e-45])
@pytest.mark.parametrize("dtype,d,r", [("f32", 64, 4), ("f32", 128, 2), ("bf16", 64, 7), ("bf16", 128, 17)])
def test_any_finite_scale(B, dtype, d, r, scale):
    x = separated(7, 3, 4, 2 * r, 2, d, 100, 120, dtype)
    out, lse = util.gpu_run(util.to_device(x), scale, 4)
    ro, rl = util.oracle(x, scale, 4)
    o, l = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    assert np.isfinite(o).all() and np.isfinite(l).all()
    assert np.abs(o - ro).max() <= 2e-5, np.abs(o - ro).max()
    assert (np.abs(l - rl) <= 2.0 ** -22 * np.maximum(1.0, np.abs(rl))).all()


@pytest.mark.parametrize("scale", [1e9, 1e30])
def test_small_batches_with_a_large_scale(B, scale):
    x = separated(8, 4, 4, 14, 2, 128, 100, 120, "bf16")
    out, lse = util.gpu_run(util.to_device(x), scale, 4)
    ro, rl = util.oracle(x, scale, 4)
    assert np.abs(out.cpu().numpy() - ro).max() <= 6e-5
    assert (np.abs(lse.cpu().numpy() - rl) <= 2.0 ** -22 * np.maximum(1.0, np.abs(rl))).all()


@pytest.mark.parametrize("fac", [1e-30, 1e-12, 1e6])
@pytest.mark.parametrize("scale", [0.125, -1e-20])
def test_factors_of_an_e4m3_store(B, scale, fac):
    x = wl.kv_to_e4m3(separated(9, 2, 4, 8, 2, 64, 90, 100, "bf16"))
    x["k_scale"] = np.array([fac, 2 * fac], np.float32)
    out, lse = util.gpu_run(util.to_device(x), scale, 4)
    ro, rl = util.oracle(x, scale, 4)
    o, l = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    assert np.isfinite(o).all()
    assert np.abs(o - ro).max() <= 5e-6 * max(1.0, np.abs(ro).max())
    assert (np.abs(l - rl) <= 2.0 ** -22 * np.maximum(1.0, np.abs(rl))).all()
