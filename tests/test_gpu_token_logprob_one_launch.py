"""Token statistics whose last workgroup merges a row's splits: with and without a reference, either side of the size from which a second kernel merges, rows of
three to 63 splits; workspaces that hold anything, and replays of a captured call.  Against the fp64 oracle at the tolerances of test_gpu_token_logprob."""
import numpy as np
import pytest

from oracle.token_stats_ref import token_stats_ref
from paper_2512_21450_amd import workloads as wl
from tests import test_gpu_token_logprob as base

pytestmark = pytest.mark.gpu
B = base.B


def rows(n, V, dtype, ref, k=6):
    """n rows that repeat k distinct ones, their ids and what the oracle says of them."""
    import torch
    x, at, wide = wl.make_logits(k, V, seed=V + n, dtype=dtype, with_ref=ref), np.arange(n) % k, -(-V // 8) * 8

    def put(a):
        t = torch.zeros((k, wide), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        t[:, :V] = base.dev(a)
        return t[torch.from_numpy(at).cuda()][:, :V]
    want = token_stats_ref(x["logits"], x["token_ids"], 1.0, x.get("ref_logits"))
    return put(x["logits"]), base.dev(x["token_ids"][at]), put(x["ref_logits"]) if ref else None, {k_: v[at] for k_, v in want.items()}


def check(got, want, what):
    for k, v in got.items():
        assert np.abs(v.cpu().numpy().astype(np.float64) - want[k]).max() <= base.TOL[k], (what, k)


# 48 000 KB of logits is the line
@pytest.mark.parametrize("ref", [False, True])
@pytest.mark.parametrize("n,V,dtype", [(1, 151936, "f32"), (3, 1000003, "bf16"), (63, 50001, "bf16"), (191, 33000, "f32"), (260, 40000, "bf16"),
                                       (161, 152000, "bf16"), (162, 152000, "bf16"), (80, 153600, "f32"), (81, 153600, "f32")])
def test_either_side_of_the_line(B, n, V, dtype, ref):  # noqa: F811
    z, ids, w, want = rows(n, V, dtype, ref)
    check(B.rl_token_logprob(z, ids, 1.0, w), want, (n, V, dtype, ref))


# 8 and 63 splits: a captured call merges the latter by a second kernel, to the same bits
@pytest.mark.parametrize("n,V,dtype", [(37, 40001, "bf16"), (2, 151936, "f32")])
@pytest.mark.parametrize("ref", [False, True])
def test_any_workspace_and_replays(B, ref, n, V, dtype):  # noqa: F811
    import torch
    z, ids, w, want = rows(n, V, dtype, ref)
    outs = {k: torch.full((n,), 7.0, device="cuda") for k in want}
    ds = B.token_logprob_desc_from_tensors(z, ids, 1.0, w, outs)
    need = B.rl_token_logprob_workspace_bytes(ds)
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    first, bits = None, lambda: [v.clone() for v in outs.values()]
    for fill, size in ((0, need), (0xFF, need), (0x5A, need), (None, need), (1, need + 256)):
        if fill is not None:
            ws.fill_(fill)
        ds.workspace, ds.workspace_bytes = ws.data_ptr(), size
        for v in outs.values():
            v.fill_(7.0)
        assert B.rl_token_logprob_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
        check(outs, want, fill)
        first = first or bits()
        assert all(torch.equal(a, b) for a, b in zip(bits(), first))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        for _ in range(2):
            assert B.rl_token_logprob_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
    for _ in range(4):
        for v in outs.values():
            v.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(bits(), first))
        assert B.rl_token_logprob_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
        assert all(torch.equal(a, b) for a, b in zip(bits(), first))
