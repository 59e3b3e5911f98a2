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


@pytest.mark.parametrize("dtype,d", TYPES)
def test_infinite_values_give_infinite_results(B, dtype, d):
    """In the last row of a segment (re-read for the rows past it), in the middle, of both signs in one column, and NaN;
    columns without one stay as they are, and an infinite value beyond the length is not seen."""
    x = case(dtype, d, 5)
    inf, nan = narrow(dtype, np.inf), narrow(dtype, np.nan)
    x["v_prefix"][0, :, 299, 3] = inf
    x["v_prefix"][1, :, 40, d - 1] = narrow(dtype, -np.inf)
    x["v_prefix"][1, :, 41, 17], x["v_prefix"][1, :, 200, 17] = inf, narrow(dtype, -np.inf)
    x["v_prefix"][1, 0, 100, 20] = nan
    x["v_prefix"][1, :, 295:] = inf
    for b in range(1, 6):
        x["v_suffix"][b, :, x["suffix_lens"][b] - 1, 5 + b] = inf
        x["v_suffix"][b, :, x["suffix_lens"][b]:] = nan
    check(x, "values")


@pytest.mark.parametrize("page", [8, 64])
def test_infinite_values_in_pages(B, page):
    x = case("bf16", 64, 6)
    x["v_suffix"][4, :, 33, 2] = narrow("bf16", np.inf)
    x["v_suffix"][5, :, 74, 60] = narrow("bf16", -np.inf)
    x["suffix_lens"][5] = 75
    y = wl.to_pages(x, page, seed=2)
    out, lse = util.gpu_run_paged(util.to_device(y), 0.1, 3)
    ro, rl = util.oracle_paged(y, 0.1, 3)
    o = out.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isinf(o), np.isinf(ro)) and np.isinf(ro).any()
    assert np.abs(np.where(np.isinf(ro), 0, o) - np.where(np.isinf(ro), 0, ro)).max() <= 2e-5


def test_small_batches_with_infinite_values(B):
    x = util.random_case(11, 2, 4, 14, 2, 128, 300, 90, "bf16", plens=[299, 35])
    x["v_prefix"][0, :, 298, 9] = narrow("bf16", np.inf)
    x["v_prefix"][1, :, 3, 127] = narrow("bf16", -np.inf)
    check(x, "small batch", 6e-5)
