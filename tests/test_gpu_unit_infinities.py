"""The one-launch decode kernel on keys whose product with the query is -inf, against the fp64 oracle: such keys have
weight 0, also where they are all that a wavefront meets first."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util

pytestmark = pytest.mark.gpu
TYPES = [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)]      # bf16 of 128 columns: 17 heads per KV head


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2512_21450_amd import binding
    return binding


def narrow(dtype, v):
    return np.float32(v) if dtype == "f32" else wl.f32_to_bf16_bits(np.array([v], np.float32))[0]


def case(dtype, d, seed, Lp=300, Ls=90, G=3):
    r = 17 if (dtype, d) == ("bf16", 128) else 3
    return util.random_case(seed, 2, G, 2 * r, 2, d, Lp, Ls, dtype, plens=[Lp, Lp - 5], slens=np.arange(2 * G) * Ls // (2 * G))


def check(x, what, tol=2e-5):
    out, lse = util.gpu_run(util.to_device(x), 0.1, x["q"].shape[0] // 2)
    ro, rl = util.oracle(x, 0.1, x["q"].shape[0] // 2)
    o, l = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    same = (o == ro) | (np.isnan(o) & np.isnan(ro))
    with np.errstate(invalid="ignore"):
        assert (same | (np.abs(o - ro) <= tol)).all(), (what, np.argwhere(~(same | (np.abs(o - ro) <= tol)))[:5])
        assert (np.abs(l - rl) <= 1e-5).all(), what


@pytest.mark.parametrize("dtype,d", TYPES)
@pytest.mark.parametrize("first", [1, 32, 64, 270])                      # of 300 keys: tiles of wavefronts 0, 1, ...
def test_infinite_keys_have_no_weight(B, dtype, d, first):
    x = case(dtype, d, 3)
    x["q"][:, :, 0] = narrow(dtype, 1.0)
    x["k_prefix"][:, :, :first, 0] = narrow(dtype, -np.inf)
    check(x, first)


@pytest.mark.parametrize("dtype,d", TYPES)
def test_products_that_overflow_for_some_rows_only(B, dtype, d):
    x = case(dtype, d, 4)
    for k in ("k_prefix", "k_suffix"):
        x[k][..., 0] = 0                                                 # the other scores stay ordinary
    x["q"][:, :, 0] = narrow(dtype, 2.0 ** -126)
    x["q"][:, ::2, 0] = narrow(dtype, 2.0 ** 10)                         # every other head: below -2^128 on the keys below
    x["k_prefix"][:, :, 32:288, 0] = narrow(dtype, -2.0 ** 120)
    check(x, "rows")
