"""The 32-lane combine kernel where a row's partials take more than one batch of 32 lanes, on both kinds of batch
(prefix-heavy or not) and on every level of a tree, against the fp64 oracle and bit for bit between its forms."""
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


# few units, so that every unit is cut among most of the workgroups
CASES = {"one sequence": (1, 1, 8, 1, 3000, 2900, None, None), "long suffixes": (1, 8, 8, 1, 100, 4000, None, None),
         "prefix-heavy": (1, 8, 8, 1, 6000, 40, [6000], None), "32 and 33 parts": (1, 2, 4, 1, 33 * 32, 32 * 32, [33 * 32], [32 * 32, 31]),
         "one long, others empty": (3, 2, 16, 2, 900, 3000, [0, 900, 5], [0, 3000, 0, 0, 1, 64])}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("paged", [False, True])
def test_rows_of_many_partials(B, name, paged):
    import torch
    P, G, Hq, Hkv, Lp, Ls, pl, sl = CASES[name]
    x = util.random_case(len(name), P, G, Hq, Hkv, 128, Lp, Ls, "bf16", plens=pl, slens=sl)
    ro, rl = util.oracle(x, 0.1, G)
    if paged:
        y = wl.to_pages(x, 32, seed=1)
        act = torch.ones(P * G, dtype=torch.uint8, device="cuda")
        out, lse = util.gpu_run_paged(util.to_device(y), 0.1, G, active=act, algo=B.RLDA_ALGO_SHARED)
    else:
        out, lse = util.gpu_run(util.to_device(x), 0.1, G, algo=B.RLDA_ALGO_SHARED)
    util.compare(out, lse, ro, rl, "bf16", name)


def test_tree_rows_of_many_partials(B):
    """Four levels and a suffix, each cut among several workgroups; one level equals the shared-prefix call."""
    import torch
    from oracle import ref
    Bn, Hq, Hkv = 8, 8, 1
    levels = [(8, 1500, ("const", 1500)), (4, 900, ("uniform", 900)), (2, 700, ("const", 700)), (1, 650, ("uniform", 650))]
    x = wl.make_tree_inputs(7, Bn, Hq, Hkv, 128, levels, 2500, ("uniform", 2500))
    lv = [tuple(util.to_device({"k": k, "v": v, "n": n}).values()) + (g,) for k, v, n, g in x["levels"]]
    t = util.to_device({k: x[k] for k in ("q", "k_suffix", "v_suffix", "suffix_lens")})
    out, lse = B.rl_decode_attn_tree(t["q"], lv, t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1)
    ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.1)
    util.compare(out, lse, ro, rl, "bf16", "four levels")
    o1, l1 = B.rl_decode_attn_tree(t["q"], lv[:1], t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1)
    o2, l2 = B.rl_decode_attn(t["q"], lv[0][0], lv[0][1], lv[0][2], t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1, 8)
    assert torch.equal(o1, o2) and torch.equal(l1, l2)
