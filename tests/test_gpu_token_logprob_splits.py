"""How the rows of the token statistics are cut: both sides of the lines between up to 64, 12, 8, 4 splits and none (rows 64, 192,
256, 320, 352, 376, 448, 512, 600, 640, vocabularies of 16384 logits and of more than 64 splits take in two rounds), vocabularies
that leave a short last split or fewer splits, and the splits that a caller with less workspace than asked for gets; against the
fp64 oracle at the tolerances of test_gpu_token_logprob."""
import numpy as np
import pytest

from oracle.token_stats_ref import token_stats_ref
from paper_2512_21450_amd import workloads as wl
from tests import test_gpu_token_logprob as base

pytestmark = pytest.mark.gpu
B = base.B


def run(B, n, V, ref, workspace=None):
    """n rows that repeat a few distinct ones (the oracle evaluates those)."""
    import torch
    k = min(n, 12)
    x = wl.make_logits(k, V, seed=V + n, with_ref=ref)
    at = np.arange(n) % k
    wide = -(-V // 8) * 8

    def rows(a):
        t = torch.zeros((k, wide), dtype=torch.bfloat16, device="cuda")
        t[:, :V] = base.dev(a)
        return t[torch.from_numpy(at).cuda()][:, :V]
    got = B.rl_token_logprob(rows(x["logits"]), base.dev(x["token_ids"][at]), 1.0, rows(x["ref_logits"]) if ref else None,
                             workspace=workspace)
    torch.cuda.synchronize()
    want = token_stats_ref(x["logits"], x["token_ids"], 1.0, x.get("ref_logits"))
    for name, v in got.items():
        assert np.abs(v.cpu().numpy().astype(np.float64) - want[name][at]).max() <= base.TOL[name], (n, V, name)
    return got


@pytest.mark.parametrize("ref", [False, True])
@pytest.mark.parametrize("n,V", [(1, 4095), (1, 8200), (3, 16385), (17, 50001), (191, 33000), (192, 33000), (256, 33000), (257, 33000),
                                 (352, 20003), (353, 20003), (300, 65535), (300, 65536), (448, 65536), (449, 65536), (513, 65536),
                                 (640, 65536), (641, 65536), (5, 151936), (2, 16383), (2, 16384), (1, 256001), (2, 1100003),
                                 (63, 33000), (64, 33000), (320, 50257), (321, 33000), (376, 70001), (377, 70001), (600, 65536),
                                 (601, 65536)])
def test_lines_between_the_splits(B, n, V, ref):  # noqa: F811
    run(B, n, V, ref)


@pytest.mark.parametrize("n,V", [(20, 60000), (100, 33000), (300, 70000)])
def test_less_workspace_than_asked_for(B, n, V):  # noqa: F811
    """20 rows of 60000: 14 splits asked for, 7 with less; 100: 8 and 3; 300 rows: 8, and none without workspace."""
    import torch
    whole = run(B, n, V, True)
    old = 0 if n >= 192 else n * min(-(-256 // n), V // 8192) * 24
    ds = B.make_token_logprob_desc(1, n, V, -(-V // 8) * 8, 1.0)
    assert B.rl_token_logprob_workspace_bytes(ds) > old
    less = run(B, n, V, True, workspace=torch.empty(max(old, 256), dtype=torch.uint8, device="cuda"))
    for k in whole:                                            # either within its tolerance of the oracle
        assert torch.allclose(whole[k], less[k], rtol=0, atol=2 * base.TOL[k])
