"""The merge of the partials with 1, 2, 4, 8, 16 and 32 teams of 32 lanes per row, which follows from how few (prompt, KV head)
and (sequence, KV head) units there are: lengths with no part at all, one part, fewer parts than teams and many, contiguous,
paged with finished sequences and on a tree, against the fp64 oracle at the bar of the shared-prefix kernels."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util

pytestmark = pytest.mark.gpu

# P, G, Hkv on 256 workgroup pairs: 256 / (P Hkv) + 2048 / (P G Hkv) parts
TEAMS = {32: (1, 1, 1), 16: (1, 8, 1), 8: (2, 4, 4), 4: (4, 8, 4), 2: (8, 8, 4), 1: (16, 8, 4)}


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2512_21450_amd import binding
    return binding


def case(seed, teams, Lp, Ls, lens):
    P, G, Hkv = TEAMS[teams]
    rng = np.random.default_rng(seed + teams)
    pl, sl = rng.integers(0, Lp + 1, P), rng.integers(0, Ls + 1, P * G)
    if lens == "full":
        pl[:], sl[:] = Lp, Ls
    elif lens == "one long":
        pl[:], sl[:] = 0, 0
        sl[-1] = Ls
    elif lens == "empty":
        pl[:], sl[:] = 0, 0
    return util.random_case(seed, P, G, 7 * Hkv, Hkv, 128, Lp, Ls, plens=pl, slens=sl), G


@pytest.mark.parametrize("lens", ["drawn", "full", "one long", "empty"])
@pytest.mark.parametrize("Lp,Ls", [(40, 33), (700, 900), (2100, 20)])
@pytest.mark.parametrize("teams", TEAMS)
def test_teams(B, teams, Lp, Ls, lens):
    x, G = case(1, teams, Lp, Ls, lens)
    P, Hkv = TEAMS[teams][0], TEAMS[teams][2]
    assert util.merge(B.make_desc(B.RLDA_BF16, P, G, 7 * Hkv, Hkv, 128, Lp, Ls, 0.09, algo=B.RLDA_ALGO_SHARED)) == teams
    out, lse = util.gpu_run(util.to_device(x), 0.09, G, algo=B.RLDA_ALGO_SHARED)
    ro, rl = util.oracle(x, 0.09, G)
    util.compare(out, lse, ro, rl, "bf16", (teams, Lp, Ls, lens))


@pytest.mark.parametrize("teams", TEAMS)
def test_teams_on_pages_with_finished_sequences(B, teams):
    import torch
    x, G = case(2, teams, 300, 800, "drawn")
    y = wl.to_pages(x, 32, seed=1)
    n = len(y["suffix_lens"])
    for act in (np.arange(n) % 3 != 1, np.arange(n) < 0):
        act = act.astype(np.uint8)
        out, lse = util.gpu_run_paged(util.to_device(y), 0.09, G, active=torch.from_numpy(act).cuda(), algo=B.RLDA_ALGO_SHARED)
        ro, rl = util.oracle_paged(y, 0.09, G, active=act)
        util.compare(out, lse, ro, rl, "bf16", teams)


@pytest.mark.parametrize("seqs,Hkv", [(2, 1), (8, 1), (16, 2), (32, 4), (64, 4), (128, 4)])
def test_teams_on_a_tree(B, seqs, Hkv):
    from oracle import ref
    levels = [(2, 300, ("uniform", 300)), (1, 90, ("uniform", 90))]
    x = wl.make_tree_inputs(seqs, seqs, 5 * Hkv, Hkv, 128, levels, 2100, ("uniform", 500), empty=0.2)   # > 2048 rows: two launches
    lv = [tuple(util.to_device({"k": k, "v": v, "n": n}).values()) + (g,) for k, v, n, g in x["levels"]]
    t = util.to_device({k: x[k] for k in ("q", "k_suffix", "v_suffix", "suffix_lens")})
    out, lse = B.rl_decode_attn_tree(t["q"], lv, t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.09)
    ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.09)
    util.compare(out, lse, ro, rl, "bf16", seqs)


@pytest.mark.parametrize("a_team", [1, 3, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("teams", [32, 16, 8])
def test_numbers_of_parts_a_team(B, teams, a_team):
    """A team asks for four, eight or sixteen parts at first: each line of them crossed, by one sequence whose tiles are a part
    each; the others have two tiles, so that the rows of a wavefront disagree."""
    P, G, Hkv = TEAMS[teams]
    Ls = 32 * min(a_team * teams, 2048 // Hkv)
    sl = np.full(P * G, min(Ls, 64))
    sl[0] = Ls
    x = util.random_case(a_team, P, G, 7 * Hkv, Hkv, 128, 8, Ls, plens=np.full(P, 5), slens=sl)
    assert util.merge(B.make_desc(B.RLDA_BF16, P, G, 7 * Hkv, Hkv, 128, 8, Ls, 0.09, algo=B.RLDA_ALGO_SHARED)) == teams
    out, lse = util.gpu_run(util.to_device(x), 0.09, G, algo=B.RLDA_ALGO_SHARED)
    ro, rl = util.oracle(x, 0.09, G)
    util.compare(out, lse, ro, rl, "bf16", (teams, a_team))
