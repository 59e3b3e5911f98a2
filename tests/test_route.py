"""Which kernels a call runs on, by the host-side rule alone (no GPU): rl_decode_attn_debug_route, how its partials are merged:
rl_decode_attn_debug_merge, and the kernel of a prefill: rl_prefill_attn_debug_form."""
import pytest

from paper_2512_21450_amd import binding as B

UNIT, SIMPLE, SHARED = B.RLDA_ROUTE_UNIT, B.RLDA_ALGO_SIMPLE, B.RLDA_ALGO_SHARED


def desc(dtype=B.RLDA_BF16, P=8, G=8, Hq=16, Hkv=2, d=128, Lp=452, Ls=512, scale=0.1, **kw):
    return B.make_desc(dtype, P, G, Hq, Hkv, d, Lp, Ls, scale, **kw)


def test_an_explicit_algo_keeps_its_kernels():
    assert B.rl_decode_attn_debug_route(desc()) == UNIT
    assert B.rl_decode_attn_debug_route(desc(algo=SHARED)) == SHARED
    assert B.rl_decode_attn_debug_route(desc(algo=SIMPLE)) == SIMPLE
    assert B.rl_decode_attn_debug_route(desc(d=64)) == UNIT
    assert B.rl_decode_attn_debug_route(desc(d=64, algo=SIMPLE)) == SIMPLE


def test_errors_are_those_of_the_plan():
    assert B.rl_decode_attn_debug_route(desc(d=96)) == B.RLDA_ERR_UNSUPPORTED
    assert B.rl_decode_attn_debug_route(desc(d=64, algo=SHARED)) == B.RLDA_ERR_UNSUPPORTED
    assert B.rl_decode_attn_debug_route(desc(), 0) == B.RLDA_ERR_INVALID
    ds = B.make_tree_desc(B.RLDA_F32, 8, 16, 2, 128, 64, 0.1, [(None, None, None, 4, 64)])
    assert B.rl_decode_attn_debug_route(ds) == B.RLDA_ERR_UNSUPPORTED


def test_pointers_off_sixteen_bytes_and_factors_that_are_not_finite_stay_on_the_simple_kernel():
    assert B.rl_decode_attn_debug_route(desc(d=64, k_suffix=1 << 20)) == UNIT
    assert B.rl_decode_attn_debug_route(desc(d=64, k_suffix=(1 << 20) + 2)) == SIMPLE
    assert B.rl_decode_attn_debug_route(desc(k_suffix=(1 << 20) + 2)) == SHARED
    for s in (float("inf"), float("-inf"), float("nan")):
        assert B.rl_decode_attn_debug_route(desc(d=64, scale=s)) == SIMPLE


@pytest.mark.parametrize("cus,units", [(256, 512), (128, 256), (64, 128), (32, 64)])
def test_how_many_units_fill_the_chip_follows_the_device(cus, units):
    """1024 keys a unit: 2048 keys per workgroup pair are two units per pair, on a partition as on the whole device."""
    tree = lambda n: B.make_tree_desc(B.RLDA_BF16, n, 8, 1, 128, 512, 0.1, [(None, None, None, 1, 512)])
    for n, want in ((units, UNIT), (units + 1, SHARED)):
        assert B.rl_decode_attn_debug_route(desc(P=n, G=1, Hq=8, Hkv=1, Lp=512, Ls=512), cus) == want
        assert B.rl_decode_attn_debug_route(tree(n), cus) == want


def test_a_launch_holds_less_than_two_to_the_32_threads():
    """What one launch cannot hold stays on the simple kernel, which spends 64 threads on a row.  One query head per KV head:
    256 threads a sequence with long stores, 64 with short ones or with pages of fewer rows than a tile."""
    one = lambda n, G=1, Ls=600, **kw: B.rl_decode_attn_debug_route(desc(P=n, G=G, Hq=1, Hkv=1, d=64, Lp=1, Ls=Ls, **kw))
    assert [one((1 << 24) + k) for k in (-1, 0, 1)] == [UNIT, SIMPLE, SIMPLE]
    assert [one((1 << 22) + k, 4) for k in (-8, -7, 0)] == [UNIT, SIMPLE, SIMPLE]     # groups rounded up to the eight dies
    assert [one((1 << 26) + k, Ls=100) for k in (-1, 0)] == [UNIT, SIMPLE]
    assert one((1 << 23) + 1, algo=SIMPLE) == SIMPLE and one(1 << 30) == SIMPLE
    paged = lambda n: B.rl_decode_attn_debug_route(
        B.make_paged_desc(B.RLDA_BF16, n, 1, 1, 1, 64, 1, 8, 10, 1, 0.1, block_table=1 << 20))
    assert [paged((1 << 26) + k) for k in (-1, 0)] == [UNIT, SIMPLE]


# (dtype, d, units, heads per KV head, keys): on either side of the lines of the rule, on 256 compute units
KEPT = [(0, 64, 64, 1, 24), (0, 64, 64, 2, 96), (0, 64, 1024, 1, 64), (0, 64, 4096, 1, 128), (0, 64, 4096, 4, 16),
        (0, 128, 512, 1, 64), (0, 128, 4096, 1, 256), (0, 128, 4096, 2, 48), (1, 64, 1024, 1, 1), (1, 64, 4096, 1, 48),
        (1, 64, 4096, 4, 1), (1, 128, 4096, 1, 64), (2, 64, 65536, 1, 1), (2, 128, 65536, 1, 16)]
BACK = [(0, 64, 64, 1, 16), (0, 64, 4096, 1, 100), (0, 64, 4096, 2, 24), (0, 64, 16384, 4, 1), (0, 128, 4096, 1, 128),
        (0, 128, 4096, 4, 1), (1, 64, 4096, 1, 16), (1, 64, 65536, 1, 32), (1, 128, 4096, 1, 48)]


@pytest.mark.parametrize("want,cases", [(UNIT, KEPT), (SIMPLE, BACK)], ids=["kept", "back"])
def test_few_rows_over_few_keys_go_to_the_simple_kernel(want, cases):
    for dtype, d, units, r, keys in cases:
        scale = -0.1 if d == 128 and dtype else 0.1                       # not the shared-prefix path's
        ds = desc(dtype, units // 8, 1, 8 * r, 8, d, keys // 2, keys - keys // 2, scale)
        assert B.rl_decode_attn_debug_route(ds) == want, (dtype, d, units, r, keys)


@pytest.mark.parametrize("dtype,d,r,keys,units,want", [
    (1, 128, 1, 1024, 4096, SIMPLE), (1, 128, 1, 1024, 1024, UNIT), (1, 128, 4, 32, 4096, UNIT), (1, 64, 1, 64, 4096, UNIT),
    (0, 64, 1, 1024, 4096, SIMPLE), (0, 64, 1, 256, 1024, SIMPLE), (0, 64, 4, 64, 4096, UNIT), (0, 64, 4, 32, 256, SIMPLE),
    (0, 128, 1, 1024, 1024, SIMPLE), (0, 128, 2, 256, 4096, SIMPLE), (0, 128, 4, 64, 4096, UNIT), (0, 128, 1, 1024, 256, UNIT),
    (2, 128, 1, 32, 4096, UNIT)])
def test_pages_of_fewer_rows_than_a_tile(dtype, d, r, keys, units, want):
    ds = B.make_paged_desc(dtype, units // 8, 1, 8 * r, 8, d, keys // 2, 16, keys // 32, units * keys // 32, 0.1,
                           block_table=1 << 20)
    assert B.rl_decode_attn_debug_route(ds) == want


def test_units_of_hardly_any_key_in_large_numbers_stay_on_the_shared_path():
    tree = lambda n: B.make_tree_desc(B.RLDA_BF16, n // 8, 8, 8, 128, 1, 0.1, [(None, None, None, 1, 1)])
    for units, want in ((16384, UNIT), (16384 + 8, SHARED)):
        assert B.rl_decode_attn_debug_route(desc(P=units // 8, G=1, Hq=8, Hkv=8, Lp=1, Ls=1)) == want
    for units, want in ((8192, UNIT), (16384 + 8, SHARED)):
        assert B.rl_decode_attn_debug_route(tree(units)) == want


# (prefix, suffix) capacities on both sides of every line of the rule for one launch, and whether that takes an empty batch
EMPTY = [(0, 0, UNIT), (452, 512, UNIT), (517, 2048, UNIT), (518, 2048, SHARED), (1200, 0, UNIT), (1201, 0, SHARED), (500, 2049, SHARED),
         (4096, 4096, SHARED), (8000, 960, SHARED), (8000, 961, SHARED), (30000, 30000, SHARED)]


@pytest.mark.parametrize("Lp,Ls,want", EMPTY)
@pytest.mark.parametrize("dtype", [B.RLDA_BF16, B.RLDA_BF16_KV8])
def test_queries_about_empty_batches_answer(dtype, Lp, Ls, want):
    """A batch without a sequence has a route like any other, for every device, and nothing to merge."""
    page = lambda P, G: B.make_paged_desc(dtype, P, G, 28, 4, 128, Lp, 64, Ls // 64, 1, 0.1, block_table=1 << 20)
    of_pages = UNIT if 3 * Lp + Ls // 64 * 64 <= 3600 and Ls // 64 * 64 <= 2048 else SHARED
    tree = [(B.make_tree_desc(dtype, 0, 28, 4, 128, Ls, 0.1, lv), want) for lv in
            ([(None, None, None, 8, Lp)], [(None, None, None, 8, Lp), (None, None, None, 2, 0)])] if dtype == B.RLDA_BF16 else []
    for ds, route in [(desc(dtype, P, G, 28, 4, Lp=Lp, Ls=Ls), want) for P, G in ((0, 8), (3, 0), (0, 0))] + \
            [(page(P, G), of_pages) for P, G in ((0, 8), (3, 0))] + tree:
        for cus in (256, 304, 64, 32, 1):
            assert B.rl_decode_attn_debug_route(ds, cus) == route, (Lp, Ls, cus)
            assert B.rl_decode_attn_debug_merge(ds, cus) == B.RLDA_ERR_UNSUPPORTED
    for dt, d in ((B.RLDA_F32, 64), (B.RLDA_F32, 128), (dtype, 64)):      # not the shared-prefix path's
        assert B.rl_decode_attn_debug_route(desc(dt, 0, 8, 28, 4, d, Lp, Ls)) in (UNIT, SIMPLE)
        assert B.rl_decode_attn_debug_merge(desc(dt, 0, 8, 28, 4, d, Lp, Ls)) == B.RLDA_ERR_UNSUPPORTED


def test_how_the_partials_are_merged():
    """Teams by the parts that the unit counts give (256 / (P Hkv) + 2048 / (P G Hkv) on 256 pairs, a group of up to 64 rows), 16
    lanes from 128 prefix and 1024 suffix units on."""
    form = lambda P, G, Hkv, r=7, cus=256, **kw: B.rl_decode_attn_debug_merge(desc(P=P, G=G, Hq=r * Hkv, Hkv=Hkv, algo=SHARED, **kw), cus)
    assert [form(*u) for u in ((1, 1, 1), (1, 8, 1), (2, 4, 4), (4, 8, 4), (8, 8, 4), (16, 8, 4), (32, 8, 4))] == [32, 16, 8, 4, 2, 1, 0]
    assert form(64, 2, 2) == form(64, 7, 2) == form(63, 9, 2) == 1 and form(64, 8, 2) == 0
    assert form(64, 17, 1, 5) == 0 and form(63, 17, 1, 5) == 1              # two row halves a group: twice the prefix units
    assert form(64, 7, 2, cus=128) == 0                                      # follows the device
    tree = lambda n, Hkv, g: B.make_tree_desc(B.RLDA_BF16, n, 7 * Hkv, Hkv, 128, 4096, 0.1, [(None, None, None, g, 5000)])
    assert [B.rl_decode_attn_debug_merge(tree(*a)) for a in ((256, 8, 8), (32, 4, 8), (8, 1, 8))] == [1, 4, 16]
    assert B.rl_decode_attn_debug_merge(desc()) == B.RLDA_ERR_UNSUPPORTED    # one launch: nothing to merge
    assert B.rl_decode_attn_debug_merge(desc(P=0, algo=SHARED)) == B.RLDA_ERR_UNSUPPORTED
    assert B.rl_decode_attn_debug_merge(desc(d=64, algo=SHARED)) == B.RLDA_ERR_UNSUPPORTED
    assert B.rl_decode_attn_debug_merge(desc(algo=SHARED), 0) == B.RLDA_ERR_INVALID
    paged = B.make_paged_desc(B.RLDA_BF16, 32, 8, 28, 4, 128, 1280, 64, 40, 1000, 0.1, block_table=1 << 20)
    assert B.rl_decode_attn_debug_merge(paged) == 0


def test_which_kernel_a_prefill_runs_on():
    form = lambda P, Hq, Hkv, cap, cus=256, scale=0.1, **kw: B.rl_prefill_attn_debug_form(
        B.make_prefill_desc(kw.get("dtype", B.RLDA_BF16), P, Hq, Hkv, 128, cap, scale), cus)
    assert form(32, 28, 4, 1280) == 2 and form(8, 16, 2, 452) == 1                # many and few blocks of 128 rows
    assert form(8, 16, 2, 452, scale=0.0) == form(1, 8, 2, 2048, scale=-1.0) == 0
    # two teams from 640 rows of capacity on, and up to 8, 9, 10 and 12 blocks to six compute units from 640, 896, 1024, 1280
    assert form(1, 8, 2, 639) == 1 and form(1, 8, 2, 640) == 3
    for P, cap, want in ((4, 680, 3), (4, 688, 1), (3, 888, 3), (3, 896, 3), (3, 1016, 3), (3, 1024, 3), (3, 1136, 3), (3, 1144, 1),
                         (3, 1272, 1), (3, 1280, 3), (3, 1360, 3), (3, 1368, 1), (2, 2048, 3), (2, 2056, 1)):
        assert form(P, 8, 1, cap) == want, (P, cap)
    # what a full buffer loses by teams: 3 x 640 tokens of 16/4 heads 14.5 -> 16.9 us, 8 x 1024 of 4/1 20.0 -> 21.0
    assert form(3, 16, 4, 640) == form(8, 4, 1, 1024) == form(5, 7, 1, 640) == 1
    assert form(4, 8, 1, 344) == 1 and form(1, 8, 2, 2048, cus=128) == 3 and form(1, 8, 2, 2056, cus=128) == 1
    assert form(1, 8, 2, 640, cus=0) == B.RLDA_ERR_INVALID and form(1, 8, 2, 640, dtype=B.RLDA_F32) == B.RLDA_ERR_UNSUPPORTED
