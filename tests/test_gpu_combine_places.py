"""The combine kernel with teams of 32 lanes where a row's partials stand in many places: few units, so that 8 to 32 teams share
a row, on both kinds of batch (prefix-heavy or not) and on every level of a tree; and one long prompt and sequence beside
short ones, so that each of 2, 4 or 8 teams has more than one batch of 32 partials; against the fp64 oracle and bit for bit
between its forms."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util
from tests.test_partition import partition

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


# P, G, Hkv, keys of the long sequence
SKEWED = {2: (8, 8, 4, 4096), 4: (8, 8, 1, 9000), 8: (8, 4, 1, 16000)}


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("others", ["empty", "few keys"])
@pytest.mark.parametrize("teams", SKEWED)
def test_more_than_one_batch_of_partials_a_team(B, teams, others, paged):
    """The long sequence's rows hold more than 32 partials per team, the others of its prompt those of the prompt."""
    import torch
    P, G, Hkv, Ls = SKEWED[teams]
    rng = np.random.default_rng(teams)
    few = others == "few keys"
    pl, sl = rng.integers(0, 70, P) * few, rng.integers(0, 40, P * G) * few
    pl[P // 2], sl[P // 2 * G + 1] = 6000, Ls
    assert util.merge(B.make_desc(B.RLDA_BF16, P, G, 7 * Hkv, Hkv, 128, 6000, Ls, 0.1, algo=B.RLDA_ALGO_SHARED)) == teams
    parts = partition(P, G, Hkv, 6000, Ls, pl, sl, R=7 * G)[1]
    of = lambda kind, unit: int(((parts[:, 0] == kind) & (parts[:, 1] == unit) & (parts[:, 2] == 0)).sum())
    assert of(0, P // 2) + of(1, P // 2 * G + 1) > 40 * teams
    x = util.random_case(teams, P, G, 7 * Hkv, Hkv, 128, 6000, Ls, "bf16", plens=pl, slens=sl)
    if paged:
        y = wl.to_pages(x, 64, seed=2)
        act = (np.arange(P * G) % 3 != 2).astype(np.uint8)
        act[P // 2 * G + 1] = 1
        out, lse = util.gpu_run_paged(util.to_device(y), 0.1, G, active=torch.from_numpy(act).cuda(), algo=B.RLDA_ALGO_SHARED)
        ro, rl = util.oracle_paged(y, 0.1, G, active=act)
    else:
        out, lse = util.gpu_run(util.to_device(x), 0.1, G, algo=B.RLDA_ALGO_SHARED)
        ro, rl = util.oracle(x, 0.1, G)
    util.compare(out, lse, ro, rl, "bf16", (teams, others))


@pytest.mark.parametrize("teams,Bn,Hkv,groups,Ls", [(2, 32, 4, (8, 2), 4096), (4, 64, 1, (8, 4), 9000), (8, 16, 1, (8, 2), 16000)])
def test_more_than_one_batch_of_partials_a_team_on_a_tree(B, teams, Bn, Hkv, groups, Ls):
    from oracle import ref
    caps = (5000, 700)
    levels = [(g, cap, ("uniform", 40)) for g, cap in zip(groups, caps)]
    x = wl.make_tree_inputs(teams, Bn, 7 * Hkv, Hkv, 128, levels, Ls, ("uniform", 30))
    for (_, _, n, _), cap in zip(x["levels"], caps):
        n[-1] = cap
    x["suffix_lens"][-1] = Ls
    lv = [tuple(util.to_device({"k": k, "v": v, "n": n}).values()) + (g,) for k, v, n, g in x["levels"]]
    t = util.to_device({k: x[k] for k in ("q", "k_suffix", "v_suffix", "suffix_lens")})
    ds = B.make_tree_desc(B.RLDA_BF16, Bn, 7 * Hkv, Hkv, 128, Ls, 0.1, [(None, None, None, g, cap) for g, cap in zip(groups, caps)])
    assert util.merge(ds) == teams
    out, lse = B.rl_decode_attn_tree(t["q"], lv, t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1)
    ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.1)
    util.compare(out, lse, ro, rl, "bf16", teams)


def test_tree_rows_of_many_partials(B):
    """Four levels and a suffix, each cut among several workgroups; one level equals the shared-prefix call, also with a store that
    takes it to the same kernels."""
    import torch
    from oracle import ref
    Bn, Hq, Hkv = 8, 8, 1
    levels = [(8, 1500, ("const", 1500)), (4, 900, ("uniform", 900)), (2, 700, ("const", 700)), (1, 650, ("uniform", 650))]
    x = wl.make_tree_inputs(7, Bn, Hq, Hkv, 128, levels, 2500, ("uniform", 2500))
    lv = [tuple(util.to_device({"k": k, "v": v, "n": n}).values()) + (g,) for k, v, n, g in x["levels"]]
    t = util.to_device({k: x[k] for k in ("q", "k_suffix", "v_suffix", "suffix_lens")})
    route = lambda caps, Ls: util.route(B.make_tree_desc(B.RLDA_BF16, Bn, Hq, Hkv, 128, Ls, 0.1, [(None, None, None, g, c) for g, c in caps]))
    assert route([lv[:2] for lv in levels], 2500) == B.RLDA_ALGO_SHARED
    out, lse = B.rl_decode_attn_tree(t["q"], lv, t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1)
    ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.1)
    util.compare(out, lse, ro, rl, "bf16", "four levels")
    for Ls, want in ((2500, B.RLDA_ROUTE_UNIT), (9000, B.RLDA_ALGO_SHARED)):
        wide = torch.full((2, Bn, Hkv, Ls, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        wide[0, :, :, :2500], wide[1, :, :, :2500] = t["k_suffix"], t["v_suffix"]
        ds = B.make_desc(B.RLDA_BF16, 1, 8, Hq, Hkv, 128, 1500, Ls, 0.1)
        assert route([(8, 1500)], Ls) == util.route(ds) == want
        o1, l1 = B.rl_decode_attn_tree(t["q"], lv[:1], wide[0], wide[1], t["suffix_lens"], 0.1)
        o2, l2 = B.rl_decode_attn(t["q"], lv[0][0], lv[0][1], lv[0][2], wide[0], wide[1], t["suffix_lens"], 0.1, 8)
        assert torch.equal(o1, o2) and torch.equal(l1, l2)
        ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"][:1], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.1)
        util.compare(o1, l1, ro, rl, "bf16", "one level")
