"""The one-launch decode kernel (one workgroup per sequence and KV head) against the fp64 oracle, through the C ABI:
what the shared-prefix kernels do not take, and the small batches that run faster in one launch.

Tolerances.  Stores the shared-prefix kernels do not take: the softmax weights keep 24 bits, so what is left is fp32
rounding: scores |s| <= 40 are good to 2^-24 |s| c, hence weights to 5e-6 relative, outputs to 5e-6 max|v| <= 2e-5
on N(0, 1) values.  Small batches at 128 columns: weights of 16 bits, 2^-17 max|v| = 4e-5 on top of that."""
import math

import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util

pytestmark = pytest.mark.gpu
EXACT, LEAN = 2e-5, 6e-5


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2512_21450_amd import binding
    return binding


def compare(out, lse, ro, rl, tol, what):
    o, l = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    inf = np.isneginf(rl)
    assert np.array_equal(np.isneginf(l), inf), what
    eo = np.abs(o - ro).max()
    el = np.abs(np.where(inf, 0.0, l) - np.where(inf, 0.0, rl)).max()
    assert eo <= tol and el <= 1e-5, f"{what}: out {eo:.2e}, lse {el:.2e}"


def case(seed, P, G, Hq, Hkv, d, Lp, Ls, dtype, edges=True):
    """Lengths include every edge of the 32-key tiles and of the turn of the wavefronts."""
    rng = np.random.default_rng(seed)
    edge = [0, 1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 289]
    pick = lambda n, cap: np.array([min(cap, e) for e in rng.permutation(edge * (n // len(edge) + 1))[:n]], np.int32)
    x = util.random_case(seed, P, G, Hq, Hkv, d, Lp, Ls, "f32" if dtype == "f32" else "bf16", pick(P, Lp), pick(P * G, Ls))
    return wl.kv_to_e4m3(x) if dtype == "e4m3" else x


SHAPES = [(1, 4, 2, 1, 300, 300),       # two units a head
          (3, 5, 14, 2, 129, 290),      # 30 units in plain order
          (9, 3, 12, 4, 290, 64),       # 36 groups on eight dies: the last round of groups is not full
          (40, 8, 4, 2, 70, 40)]        # more units than compute units: the four-wavefront form


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("e4m3", 64)])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_what_the_shared_kernels_do_not_take(B, shape, dtype, d):
    P, G, Hq, Hkv, Lp, Ls = shape
    x = case(P + d, P, G, Hq, Hkv, d, Lp, Ls, dtype)
    out, lse = util.gpu_run(util.to_device(x), 1 / math.sqrt(d), G)
    ro, rl = util.oracle(x, 1 / math.sqrt(d), G)
    compare(out, lse, ro, rl, EXACT, f"{dtype} d={d} {shape}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "e4m3"])
@pytest.mark.parametrize("r", [17, 32, 40])
def test_more_than_sixteen_heads_per_kv_head(B, r, dtype, d):
    x = case(r, 3, 4, 2 * r, 2, d, 100, 290, dtype)
    out, lse = util.gpu_run(util.to_device(x), 0.1, 4)
    ro, rl = util.oracle(x, 0.1, 4)
    compare(out, lse, ro, rl, EXACT, f"r={r}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "e4m3"])
@pytest.mark.parametrize("scale", [-0.1, 0.0])
def test_scales_that_are_not_positive(B, scale, dtype, d):
    x = case(5, 3, 4, 8, 2, d, 129, 290, dtype)
    out, lse = util.gpu_run(util.to_device(x), scale, 4)
    ro, rl = util.oracle(x, scale, 4)
    compare(out, lse, ro, rl, EXACT, f"scale {scale}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "e4m3"])
@pytest.mark.parametrize("page", [1, 4, 16, 32, 128])
def test_pages_of_any_size_and_finished_sequences(B, page, dtype, d):
    import torch
    P, G = 4, 5
    x = wl.to_pages(case(page, P, G, 10, 2, d, 70, 290, dtype), page, seed=2)     # NaN in every row without a live key
    act = (np.arange(P * G) % 4 != 1).astype(np.uint8)
    act[:G] = 0                                                                   # a whole group finished
    t = util.to_device(x)
    lean = d == 128 and page >= 32 and dtype != "f32"
    for a in (None, act):
        out, lse = util.gpu_run_paged(t, 0.1, G, active=None if a is None else torch.from_numpy(a).cuda())
        ro, rl = util.oracle_paged(x, 0.1, G, active=a)
        compare(out, lse, ro, rl, LEAN if lean else EXACT, f"page {page}")


@pytest.mark.parametrize("dtype", ["bf16", "e4m3"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_small_batches_take_one_launch(B, shape, dtype):
    """Under AUTO; forced onto the shared-prefix kernels the same batches give the same result within their tolerance."""
    P, G, Hq, Hkv, Lp, Ls = shape
    x = case(P, P, G, Hq, Hkv, 128, Lp, Ls, dtype)
    t = util.to_device(x)
    ro, rl = util.oracle(x, 0.09, G)
    out, lse = util.gpu_run(t, 0.09, G)
    compare(out, lse, ro, rl, LEAN, f"one launch {shape}")
    out, lse = util.gpu_run(t, 0.09, G, algo=B.RLDA_ALGO_SHARED)
    util.compare(out, lse, ro, rl, "bf16", f"shared-prefix kernels {shape}")


def test_stores_off_sixteen_bytes_stay_on_the_simple_kernel(B):
    import torch
    x = case(8, 2, 3, 4, 2, 64, 70, 100, "bf16")
    t = util.to_device(x)
    for k in ("v_prefix", "v_suffix"):                       # a view that starts two bytes into its storage
        buf = torch.empty(t[k].numel() + 1, dtype=t[k].dtype, device="cuda")
        buf[1:] = t[k].reshape(-1)
        t[k] = buf[1:].view(t[k].shape)
    out, lse = util.gpu_run(t, 0.1, 3)
    ro, rl = util.oracle(x, 0.1, 3)
    compare(out, lse, ro, rl, EXACT, "misaligned values")


# shapes of the shared-prefix kernels that AUTO now runs in one launch: forced, they stay covered
@pytest.mark.parametrize("shape", [(3, 8, 28, 4, 200, 300), (2, 8, 16, 2, 131, 257), (2, 16, 16, 2, 97, 65), (3, 1, 8, 8, 50, 40),
                                   (1, 2, 32, 2, 40, 33), (5, 7, 6, 3, 31, 1), (2, 10, 16, 2, 140, 90), (3, 9, 14, 2, 75, 120),
                                   (2, 13, 10, 2, 100, 64), (2, 32, 14, 2, 150, 60), (1, 16, 32, 2, 100, 40), (2, 17, 16, 2, 70, 33)],
                         ids=str)
def test_shared_prefix_kernels_when_forced(B, shape):
    P, G, Hq, Hkv, Lp, Ls = shape
    x = util.random_case(300 + P * G, P, G, Hq, Hkv, 128, Lp, Ls, "bf16")
    out, lse = util.gpu_run(util.to_device(x), 0.09, G, algo=B.RLDA_ALGO_SHARED)
    ro, rl = util.oracle(x, 0.09, G)
    util.compare(out, lse, ro, rl, "bf16", str(shape))
