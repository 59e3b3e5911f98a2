"""The one-launch decode kernel asks for a wavefront's first K tile before it knows the lengths, where the first segment's
capacity has room for a whole tile, and for its second tile before the first has landed.

Capacities and lengths on both sides of every line of that: a capacity that ends inside a tile, a first segment that is
shorter than the tile asked for or empty, one, two and three tiles per wavefront.  Rows past the lengths hold NaN, as a store
may, so that a tile that was asked for too early shows.  Tolerances as in test_gpu_unit."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util
from tests.test_gpu_unit import EXACT, LEAN, B, compare  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu


def poison(x):
    """NaN behind the lengths."""
    for s in ("prefix", "suffix"):
        for i, n in enumerate(x[s + "_lens"]):
            for kv in ("k_", "v_"):
                t = x[kv + s]
                t[i, :, n:] = 0x7FC0 if t.dtype == np.uint16 else (0x7F if t.dtype == np.uint8 else np.nan)
    return x


# eight wavefronts (few units) and, with 300 units, the forms of four and fewer
@pytest.mark.parametrize("P,G", [(5, 2), (75, 4)])
@pytest.mark.parametrize("Lp,plens", [(31, 31), (33, 33), (255, 255), (256, 256), (288, 33), (288, 0), (800, 257), (800, 513), (800, 800)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("e4m3", 64), ("bf16", 128), ("e4m3", 128)])
def test_first_and_second_tiles(B, dtype, d, Lp, plens, P, G):  # noqa: F811
    Ls, rng = 70, np.random.default_rng(Lp + plens)
    pl = np.full(P, plens, np.int32)
    pl[1::3] = rng.integers(0, plens + 1, len(pl[1::3]))
    sl = rng.integers(0, Ls + 1, P * G).astype(np.int32)
    x = util.random_case(Lp * d + plens, P, G, 4, 1, d, Lp, Ls, "f32" if dtype == "f32" else "bf16", pl, sl)
    x = poison(wl.kv_to_e4m3(x) if dtype == "e4m3" else x)
    out, lse = util.gpu_run(util.to_device(x), 0.1, G)
    ro, rl = util.oracle(x, 0.1, G)
    compare(out, lse, ro, rl, LEAN if d == 128 and dtype != "f32" else EXACT, (dtype, d, Lp, plens, P))


@pytest.mark.parametrize("cap", [33, 256, 600])
def test_first_and_second_tiles_of_a_tree(B, cap):  # noqa: F811
    from oracle import ref
    levels = [(4, cap, ("uniform", cap)), (2, 70, ("uniform", 70))]
    x = wl.make_tree_inputs(cap, 16, 7, 1, 128, levels, 90, ("uniform", 90), empty=0.2)
    lv = [tuple(util.to_device({"k": k, "v": v, "n": n}).values()) + (g,) for k, v, n, g in x["levels"]]
    t = util.to_device({k: x[k] for k in ("q", "k_suffix", "v_suffix", "suffix_lens")})
    out, lse = B.rl_decode_attn_tree(t["q"], lv, t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1)
    ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.1)
    compare(out, lse, ro, rl, LEAN, cap)
