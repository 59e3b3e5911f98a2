"""rl_kv_append_rope 16 bytes at a time (aligned buffers, unless the heads are few) against one element at a time
(buffers that are not): the same bits, for every element type, head size and store, around one pass of the workgroup
(256 chunks); and not the slower of the two.  The element path is compared with the oracle elsewhere.
"""
import pytest

from tests.test_gpu_unit_batches import us_per_call

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2512_21450_amd import binding
    return binding


def shifted(t, by):
    """a copy that starts `by` elements behind a 16-byte line"""
    import torch
    flat = torch.empty(t.numel() + 16, dtype=t.dtype, device=t.device)
    assert flat.data_ptr() % 16 == 0
    out = flat[by:by + t.numel()].view(t.shape)
    out.copy_(t)
    return out


CASES = [                       # Hq, Hkv, d: chunks of q and k in one workgroup
    (1, 1, 64),                 # 8 (bf16: one element at a time), 16 (fp32)
    (4, 1, 128),                # 40 (e4m3: one element at a time), 80
    (16, 2, 128),               # 144, 288
    (28, 4, 128),               # 256, 512
    (29, 4, 128),               # 264: a second pass of eight threads
    (56, 32, 64),               # 352; 256 chunks of values
    (64, 40, 128),              # several passes of both
]


@pytest.mark.parametrize("paged", [False, True], ids=["rows", "pages"])
@pytest.mark.parametrize("store", ["f32", "bf16", "e4m3"])
@pytest.mark.parametrize("heads", CASES, ids=str)
def test_same_bits(B, heads, store, paged):
    import torch
    Hq, Hkv, d = heads
    nB, cap, ps = 5, 96, 32
    g = torch.Generator(device="cuda").manual_seed(11)
    dt = torch.float32 if store == "f32" else torch.bfloat16
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).to(dt)
    q, kn, vn = rnd(nB, Hq, d), rnd(nB, Hkv, d), rnd(nB, Hkv, d)
    pos = torch.randint(0, 40000, (3, nB), device="cuda", generator=g, dtype=torch.int32)
    freq = 10000.0 ** (-torch.arange(d // 2, device="cuda", dtype=torch.float32) / (d // 2))
    lens = torch.tensor([0, ps - 1, ps, cap - 1, cap], dtype=torch.int32, device="cuda")
    act = torch.tensor([1, 1, 0, 1, 1], dtype=torch.uint8, device="cuda")
    table = torch.randperm(nB * cap // ps, device="cuda", generator=g).to(torch.int32).view(nB, cap // ps) if paged else None
    shape = (nB * cap // ps, Hkv, ps, d) if paged else (nB, Hkv, cap, d)
    if store == "e4m3":
        ks, vs = (torch.randint(0, 120, shape, device="cuda", generator=g, dtype=torch.uint8) for _ in range(2))
        scales = [torch.rand(Hkv, device="cuda", generator=g) + 0.01 for _ in range(2)]
    else:
        ks, vs, scales = rnd(*shape), rnd(*shape), [None, None]
    got = []
    for by in (0, 1):
        a = [shifted(t, by) for t in (q, kn, vn, ks, vs)]
        n = lens.clone()
        B.rl_kv_append_rope(a[0], a[1], a[2], pos, freq, (d // 4, d // 8, d // 8), a[3], a[4], n, block_table=table,
                            seq_active=act, k_scale=scales[0], v_scale=scales[1])
        torch.cuda.synchronize()
        got.append([t.clone() for t in (a[0], a[3], a[4], n)])
    for what, x, y in zip(("q", "keys", "values", "lengths"), *got):
        assert torch.equal(x, y), (what, (x != y).nonzero()[:8].tolist(), x[x != y][:8].tolist(), y[x != y][:8].tolist())
    assert not torch.equal(got[0][1], ks) and got[0][3].tolist() == [1, ps, ps, cap, cap]


@pytest.mark.parametrize("store", ["bf16", "e4m3"])
@pytest.mark.parametrize("nB,Hq,Hkv,d", [(1, 4, 1, 128), (64, 2, 2, 64), (128, 7, 1, 128), (128, 28, 4, 128), (4096, 4, 1, 64)])
def test_aligned_buffers_are_not_slower(B, nB, Hq, Hkv, d, store):
    """1.2 to 1.8 times as long for few heads on e4m3 stores when they went 16 bytes at a time."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).bfloat16()
    src = [rnd(nB, Hq, d), rnd(nB, Hkv, d), rnd(nB, Hkv, d)]
    stores = [torch.zeros(nB, Hkv, 512, d, device="cuda", dtype=torch.uint8 if store == "e4m3" else torch.bfloat16) for _ in range(2)]
    pos = torch.randint(0, 40000, (3, nB), device="cuda", generator=g, dtype=torch.int32)
    freq = 10000.0 ** (-torch.arange(d // 2, device="cuda", dtype=torch.float32) / (d // 2))
    scale = torch.full((Hkv,), 0.02, device="cuda") if store == "e4m3" else None
    t = []
    for by in (0, 1):
        a = [shifted(x, by) for x in src + stores]
        lens = torch.zeros(nB, dtype=torch.int32, device="cuda")      # room for every call below
        ds = B.kv_append_desc_from_tensors(a[0], a[1], a[2], pos, freq, (d // 4, d // 8, d // 8), a[3], a[4], lens, None, None,
                                           scale, scale)

        def call():
            assert B.rl_kv_append_rope_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
        t.append(us_per_call(call, n=50))
    print(f"\naligned {t[0]:.2f} us, not {t[1]:.2f}")
    assert t[0] <= 1.15 * t[1] + 0.1, t
