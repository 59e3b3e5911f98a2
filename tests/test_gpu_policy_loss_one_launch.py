"""The policy loss whose last workgroup reduces: sequence counts around the groups of 64 that the workgroups meet in and around the
most that are reduced so, against the fp64 oracle; workspaces that hold anything, and replays of a captured call."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests.test_gpu_policy_loss import B, check_loss, dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 191, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
def test_numbers_of_sequences(B, n, agg):  # noqa: F811
    x = wl.make_rollout_tokens(n, 300, 1, seed=n, lens=("uniform", 300))
    x["lens"][: n // 3: 5] = 0
    adv = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    check_loss(B, x, adv, 0.2, 0.28, beta_kl=0.04, beta_ent=0.01, agg=agg)


@pytest.mark.parametrize("n", [70, 1100, 4090])
def test_any_workspace_and_replays(B, n):  # noqa: F811
    import torch
    x = wl.make_rollout_tokens(n, 50, 1, seed=n, lens=("uniform", 50))
    t = {k: dev(x[k]) for k in ("logprob", "old_logprob", "kl", "entropy", "lens")}
    adv = torch.randn(n, generator=torch.Generator("cuda").manual_seed(n), device="cuda")
    stats, grad = torch.empty(8, device="cuda"), torch.empty((n, 50), device="cuda")
    ds = B.policy_loss_desc_from_tensors(t["logprob"], t["old_logprob"], adv, t["lens"], 0.2, 0.28, stats, t["kl"], t["entropy"], grad, 0.04, 0.01)
    ws = torch.empty(B.rl_policy_loss_workspace_bytes(ds), dtype=torch.uint8, device="cuda")
    ds.workspace, ds.workspace_bytes = ws.data_ptr(), ws.numel()
    want = B.rl_policy_loss(t["logprob"], t["old_logprob"], adv, t["lens"], 0.2, 0.28, t["kl"], t["entropy"], 0.04, 0.01)

    def same(what):
        assert torch.equal(stats, want[0]) and torch.equal(grad, want[1]), what
        stats.fill_(7.0), grad.fill_(7.0)
    for fill in (0, 0xFF, 0x5A, None, 1):
        if fill is not None:
            ws.fill_(fill)
        assert B.rl_policy_loss_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
        same(fill)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        for _ in range(2):
            assert B.rl_policy_loss_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
    for k in range(4):
        g.replay()
        torch.cuda.synchronize()
        same(k)
        assert B.rl_policy_loss_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
        same(k)
