"""Units of many keys that several workgroups share in the one-launch decode: lengths at the edges of how many take part (none, a tile
less and more than where the second, the third ... begins), every store type and form, contiguous, paged with finished sequences
and trees; workspaces that hold anything, are smaller than asked for or missing; replays of a captured call.  Against the fp64
oracle, tolerances as in test_gpu_unit."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util
from tests.test_gpu_unit import EXACT, LEAN, B, compare  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu
# tiles of a sequence: one workgroup, two, three ... of four or eight wavefronts, all of them in one round, two and three
TILES = [0, 1, 4, 5, 8, 9, 14, 16, 17, 24, 25, 32, 33, 40, 41, 57, 64, 65, 128, 129, 260]


def case(B, dtype, d, P, G, r, Lp, Ls, seed=1, Hkv=1):
    """Prefixes and suffixes that end on either side of a tile, together TILES in turn, as far as the buffers reach."""
    rng = np.random.default_rng(seed)
    pl, sl = np.zeros(P, int), np.zeros(P * G, int)
    for b in range(P * G):
        n = TILES[(b * 7 + seed) % len(TILES)]
        if b % G == 0:
            pl[b // G] = min(Lp, max(0, 32 * rng.integers(0, n + 1) - rng.integers(0, 32)))
        sl[b] = min(Ls, max(0, 32 * n - pl[b // G] - rng.integers(0, 32)))
    x = util.random_case(seed, P, G, Hkv * r, Hkv, d, Lp, Ls, "f32" if dtype == "f32" else "bf16", pl, sl)
    return wl.kv_to_e4m3(x) if dtype == "e4m3" else x


def desc(B, t, G, workspace=None, algo=None):
    import torch
    n, Hq, d = t["q"].shape
    out, lse = torch.full((n, Hq, d), 7.0, device="cuda"), torch.full((n, Hq), 7.0, device="cuda")
    ds = B.desc_from_tensors(t["q"], t["k_prefix"], t["v_prefix"], t["prefix_lens"], t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1, G,
                             out, lse, workspace, B.RLDA_ALGO_AUTO_SCRATCH if algo is None else algo,
                             k_scale=t.get("k_scale"), v_scale=t.get("v_scale"))
    return ds, out, lse


# P, G, rows per KV head, capacities: 16, 8, 4, 3 and 2 workgroups a unit, groups on one die each and in plain order
SHAPES = [(2, 1, 1, 4200, 4200), (5, 4, 7, 900, 3000), (8, 8, 4, 480, 500), (3, 9, 5, 200, 290), (10, 8, 16, 2000, 90), (16, 8, 2, 2100, 1000)]


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("e4m3", 64), ("bf16", 128), ("e4m3", 128)])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shared_units(B, dtype, d, shape):  # noqa: F811
    P, G, r, Lp, Ls = shape
    scale = 0.1
    if d == 128 and dtype != "f32":                                      # what the shared-prefix kernels do not take either: 24-bit weights
        scale = -0.1
    for seed in (1, 2):
        x = case(B, dtype, d, P, G, r, Lp, Ls, seed)
        out, lse = util.gpu_run(util.to_device(x), scale, G)
        ro, rl = util.oracle(x, scale, G)
        compare(out, lse, ro, rl, EXACT, (dtype, d, shape, seed))


# two, three and four blocks of 16 rows a KV head, each with a counter of its own: in groups on one die, and in plain order
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("e4m3", 64), ("bf16", 128), ("e4m3", 128)])
@pytest.mark.parametrize("P,G,Hkv,r", [(4, 4, 1, 17), (3, 5, 1, 40), (2, 2, 4, 32), (3, 1, 1, 17), (2, 1, 2, 40), (1, 1, 1, 64)])
def test_more_than_sixteen_rows_per_kv_head(B, dtype, d, P, G, Hkv, r):  # noqa: F811
    code = {"f32": B.RLDA_F32, "bf16": B.RLDA_BF16, "e4m3": B.RLDA_BF16_KV8}[dtype]
    ds = B.make_desc(code, P, G, Hkv * r, Hkv, d, 1000, 1800, 0.1, B.RLDA_ALGO_AUTO_SCRATCH)
    assert B.rl_decode_attn_workspace_bytes(ds) > 0 and util.route(ds) == B.RLDA_ROUTE_UNIT
    x = case(B, dtype, d, P, G, r, 1000, 1800, r, Hkv=Hkv)
    out, lse = util.gpu_run(util.to_device(x), 0.1, G)
    ro, rl = util.oracle(x, 0.1, G)
    compare(out, lse, ro, rl, EXACT, (dtype, d, P, G, Hkv, r))


@pytest.mark.parametrize("dtype", ["bf16", "e4m3"])
@pytest.mark.parametrize("shape", [(5, 4, 7, 700, 1500), (8, 8, 4, 480, 500), (10, 8, 16, 700, 90), (16, 8, 2, 500, 2000)], ids=str)
def test_small_batches_of_long_sequences(B, dtype, shape):  # noqa: F811
    P, G, r, Lp, Ls = shape
    x = case(B, dtype, 128, P, G, r, Lp, Ls, 3)
    assert util.route(B.make_desc(B.RLDA_BF16 if dtype == "bf16" else B.RLDA_BF16_KV8, P, G, r, 1, 128, Lp, Ls, 0.1)) == B.RLDA_ROUTE_UNIT
    out, lse = util.gpu_run(util.to_device(x), 0.1, G)
    ro, rl = util.oracle(x, 0.1, G)
    compare(out, lse, ro, rl, LEAN, (dtype, shape))


@pytest.mark.parametrize("dtype,page", [("f32", 32), ("bf16", 64), ("e4m3", 128)])
def test_pages_and_finished_sequences(B, dtype, page):  # noqa: F811
    import torch
    P, G = 6, 5
    x = case(B, dtype, 64, P, G, 3, 700, 2500, 4, Hkv=2)
    y = wl.to_pages(x, page, seed=1)
    act = (np.arange(P * G) % 4 != 2).astype(np.uint8)
    act[G:2 * G] = 0
    out, lse = util.gpu_run_paged(util.to_device(y), 0.1, G, active=torch.from_numpy(act).cuda())
    ro, rl = util.oracle_paged(y, 0.1, G, active=act)
    compare(out, lse, ro, rl, EXACT, (dtype, page))


@pytest.mark.parametrize("seqs,Hkv,caps", [(8, 1, (600, 450)), (16, 2, (480, 300)), (32, 4, (550, 500))])
def test_trees(B, seqs, Hkv, caps):  # noqa: F811
    from oracle import ref
    x = wl.make_tree_inputs(seqs, seqs, 5 * Hkv, Hkv, 128, [(8, caps[0], ("uniform", caps[0])), (2, caps[1], ("uniform", caps[1]))], 400,
                            ("uniform", 400), empty=0.2)
    lv = [tuple(util.to_device({"k": k, "v": v, "n": n}).values()) + (g,) for k, v, n, g in x["levels"]]
    t = util.to_device({k: x[k] for k in ("q", "k_suffix", "v_suffix", "suffix_lens")})
    out, lse = B.rl_decode_attn_tree(t["q"], lv, t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1)
    ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.1)
    compare(out, lse, ro, rl, LEAN, seqs)


def test_infinite_values_and_keys(B):  # noqa: F811
    """A row's sum is that of all its workgroups, also where columns are looked at again."""
    x = util.random_case(9, 2, 2, 6, 2, 64, 3000, 400, "f32", [3000, 2999], [400, 0, 33, 399])
    x["v_prefix"][0, :, 2999, 3], x["v_prefix"][1, :, 1040, 63], x["v_prefix"][1, 0, 1700, 9] = np.inf, -np.inf, np.nan
    x["q"][:, :, 0], x["k_prefix"][1, :, :600, 0] = 1.0, -np.inf
    out, lse = util.gpu_run(util.to_device(x), 0.1, 2)
    ro, rl = util.oracle(x, 0.1, 2)
    o = out.cpu().numpy().astype(np.float64)
    same = (o == ro) | (np.isnan(o) & np.isnan(ro))
    with np.errstate(invalid="ignore"):
        assert (same | (np.abs(o - ro) <= 2e-5)).all()
    assert np.isinf(ro).any() and np.isnan(ro).any() and np.abs(lse.cpu().numpy() - rl).max() <= 1e-5


def same_with_infinities(out, lse, ro, rl, tol):
    o = out.cpu().numpy().astype(np.float64)
    same = (o == ro) | (np.isnan(o) & np.isnan(ro))
    with np.errstate(invalid="ignore"):
        assert (same | (np.abs(o - ro) <= tol)).all()
    assert np.isinf(ro).any() and np.isnan(ro).any() and np.abs(lse.cpu().numpy() - rl).max() <= 1e-5


def bits(dtype, v):
    return np.float32(v) if dtype == "f32" else wl.f32_to_bf16_bits(np.array([v], np.float32))[0]


@pytest.mark.parametrize("page", [0, 64])
@pytest.mark.parametrize("dtype,d,r", [("f32", 128, 3), ("bf16", 64, 3), ("bf16", 64, 20), ("bf16", 128, 3), ("bf16", 128, 20)])
def test_infinite_values_in_shared_units(B, dtype, d, r, page):  # noqa: F811
    """In every segment, in one column and in both directions, which gives none; rows of 24-bit and of 16-bit weights."""
    x = util.random_case(10, 2, 2, 2 * r, 2, d, 1500, 1100, dtype, [1500, 1499], [1100, 0, 33, 1099])
    v = lambda y: bits(dtype, y)
    x["v_prefix"][0, :, 1499, 3], x["v_prefix"][1, :, 1040, d - 1], x["v_prefix"][1, 0, 700, 9] = v(np.inf), v(-np.inf), v(np.nan)
    x["v_suffix"][0, 1, 1099, 3], x["v_suffix"][3, 0, 5, 2] = v(-np.inf), v(np.inf)
    lean = d == 128 and dtype == "bf16" and r <= 16
    code = B.RLDA_F32 if dtype == "f32" else B.RLDA_BF16
    if page:
        y = wl.to_pages(x, page, seed=1)
        out, lse = util.gpu_run_paged(util.to_device(y), 0.1, 2)
        ro, rl = util.oracle_paged(y, 0.1, 2)
    else:
        assert util.route(B.make_desc(code, 2, 2, 2 * r, 2, d, 1500, 1100, 0.1)) == B.RLDA_ROUTE_UNIT
        out, lse = util.gpu_run(util.to_device(x), 0.1, 2)
        ro, rl = util.oracle(x, 0.1, 2)
    same_with_infinities(out, lse, ro, rl, LEAN if lean else EXACT)


def test_infinite_values_in_a_tree(B):  # noqa: F811
    from oracle import ref
    x = wl.make_tree_inputs(3, 8, 10, 2, 128, [(8, 600, ("const", 600)), (2, 450, ("const", 450))], 400, ("const", 400))
    for i, (at, y) in enumerate([((0, 0, 599, 3), np.inf), ((2, 1, 449, 77), -np.inf)]):
        x["levels"][i][1][at] = bits("bf16", y)
    x["v_suffix"][5, 0, 399, 3], x["v_suffix"][6, 1, 0, 9] = bits("bf16", -np.inf), bits("bf16", np.nan)
    lv = [tuple(util.to_device({"k": k, "v": v, "n": n}).values()) + (g,) for k, v, n, g in x["levels"]]
    t = util.to_device({k: x[k] for k in ("q", "k_suffix", "v_suffix", "suffix_lens")})
    assert util.route(B.make_tree_desc(B.RLDA_BF16, 8, 10, 2, 128, 400, 0.1, [(None, None, None, 8, 600), (None, None, None, 2, 450)])) == B.RLDA_ROUTE_UNIT
    out, lse = B.rl_decode_attn_tree(t["q"], lv, t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1)
    ro, rl = ref.decode_attn_tree_ref(x["q"], x["levels"], x["k_suffix"], x["v_suffix"], x["suffix_lens"], 0.1)
    same_with_infinities(out, lse, ro, rl, LEAN)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_any_workspace(B, dtype, d):  # noqa: F811
    """Whatever a workspace holds the bits are the same, also where an earlier call with other shapes left it; so are they in the
    library's own array.  With less of it fewer workgroups share a unit, with none one: the oracle's result all the same."""
    import torch
    x = case(B, dtype, d, 5, 4, 7, 400, 900, 5)
    t = util.to_device(x)
    ro, rl = util.oracle(x, 0.1, 4)
    stream = torch.cuda.current_stream().cuda_stream
    ds, out, lse = desc(B, t, 4)
    need = B.rl_decode_attn_workspace_bytes(ds)
    assert need > 0 and util.route(ds) == B.RLDA_ROUTE_UNIT
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    first = None
    for fill in (0, 0xFF, 0x5A, None, None, "other", 1):
        if fill == "other":
            z = case(B, dtype, d, 2, 3, 7, 300, 800, 6)
            do, oo, lo = desc(B, util.to_device(z), 3, ws)
            assert B.rl_decode_attn_raw(do, stream) == 0
            compare(oo, lo, *util.oracle(z, 0.1, 3), EXACT if d == 64 else LEAN, "other")
        elif fill is not None:
            ws.fill_(fill)
        ds.workspace, ds.workspace_bytes = ws.data_ptr(), need
        out.fill_(7.0), lse.fill_(7.0)
        assert B.rl_decode_attn_raw(ds, stream) == 0
        compare(out, lse, ro, rl, EXACT if d == 64 else LEAN, fill)
        first = first or (out.clone(), lse.clone())
        assert torch.equal(out, first[0]) and torch.equal(lse, first[1]), fill
    so, sl = torch.empty_like(out), torch.empty_like(lse)
    B.rl_decode_attn_static(t["q"], t["k_prefix"], t["v_prefix"], t["prefix_lens"], t["k_suffix"], t["v_suffix"], t["suffix_lens"], 0.1, 4, so, sl,
                            algo=B.RLDA_ALGO_AUTO_SCRATCH)
    assert torch.equal(so, first[0]) and torch.equal(sl, first[1])
    if d == 64:                                                          # the shared-prefix plan insists on its workspace
        for less, at in ((need - 1, 0), (need // 3, 0), (256, 0), (0, 0), (need, 16)):
            ds.workspace, ds.workspace_bytes = (ws.data_ptr() + at if less else None), less
            out.fill_(7.0), lse.fill_(7.0)
            before = ws.clone()
            assert B.rl_decode_attn_raw(ds, stream) == 0
            compare(out, lse, ro, rl, EXACT, less)
            mine = 0 if at else less                                     # off 256 bytes: not used
            assert torch.equal(ws[mine:], before[mine:]), less


def test_calls_that_asked_for_no_scratch_leave_the_workspace_alone(B):  # noqa: F811
    """One workspace carried through calls on two streams, and the library's own array: under AUTO a plan without scratch writes to neither,
    so nothing orders the calls and the bits are those of a call without a workspace."""
    import torch
    work = []
    ws = torch.full((1 << 20,), 0x5A, dtype=torch.uint8, device="cuda")
    for seed in (8, 9):
        x = case(B, "f32", 64, 5, 4, 7, 400, 900, seed)
        t = util.to_device(x)
        alone, ao, al = desc(B, t, 4, algo=B.RLDA_ALGO_AUTO)
        assert B.rl_decode_attn_raw(alone, torch.cuda.current_stream().cuda_stream) == 0
        compare(ao, al, *util.oracle(x, 0.1, 4), EXACT, seed)
        for raw in (B.rl_decode_attn_raw, B.rl_decode_attn_static_raw):
            work.append((raw, *desc(B, t, 4, ws, B.RLDA_ALGO_AUTO), ao, al, t, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(20):
        for raw, ds, _, _, _, _, _, st in work:
            assert raw(ds, st.cuda_stream) == 0
    torch.cuda.synchronize()
    assert (ws == 0x5A).all()
    for _, _, out, lse, ao, al, _, _ in work:
        assert torch.equal(out, ao) and torch.equal(lse, al)


def test_replays_of_a_captured_call(B):  # noqa: F811
    """Every replay carries the same number of the call and has to find its counters as the last one left them; lengths that change
    in between change how many workgroups take part."""
    import torch
    x = case(B, "f32", 64, 6, 2, 3, 600, 2000, 7)
    t = util.to_device(x)
    ds, out, lse = desc(B, t, 2)
    ws = torch.full((B.rl_decode_attn_workspace_bytes(ds),), 0xA5, dtype=torch.uint8, device="cuda")
    ds.workspace, ds.workspace_bytes = ws.data_ptr(), ws.numel()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        for _ in range(3):
            assert B.rl_decode_attn_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
    for k in range(6):
        sl = np.roll(x["suffix_lens"], k)
        t["suffix_lens"].copy_(torch.from_numpy(sl))
        out.fill_(7.0), lse.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        got = out.clone(), lse.clone()
        compare(*got, *util.oracle({**x, "suffix_lens": sl}, 0.1, 2), EXACT, k)
        assert B.rl_decode_attn_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
        assert torch.equal(out, got[0]) and torch.equal(lse, got[1])


def test_two_streams_with_a_workspace_each(B):  # noqa: F811
    import torch
    xs = [case(B, "bf16", 64, 8, 4, 5, 900, 1500, s) for s in (8, 9)]
    work = []
    for x in xs:
        t = util.to_device(x)
        ds, out, lse = desc(B, t, 4)
        ws = torch.empty(B.rl_decode_attn_workspace_bytes(ds), dtype=torch.uint8, device="cuda")
        ds.workspace, ds.workspace_bytes = ws.data_ptr(), ws.numel()
        work.append((ds, out, lse, ws, t, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(20):
        for ds, _, _, _, _, st in work:
            assert B.rl_decode_attn_raw(ds, st.cuda_stream) == 0
    torch.cuda.synchronize()
    for x, (_, out, lse, _, _, _) in zip(xs, work):
        compare(out, lse, *util.oracle(x, 0.1, 4), EXACT, "streams")
