"""The policy loss's token pass where its rows and its count end: rows of every remainder by four tokens, contiguous (so that
they start on four bytes only) and as views of padded rows, and sequence counts on both sides of the 1024 up to which the
token pass counts for itself, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests.test_gpu_policy_loss import B, check_loss, dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1024, 1025])
@pytest.mark.parametrize("T", [1, 2, 3, 5, 6, 1021, 1022, 1023, 1025, 1030])
def test_rows_of_every_remainder(B, T, n):  # noqa: F811
    import torch
    x = wl.make_rollout_tokens(n, T, 1, seed=T, drift=0.25, lens=("uniform", T))
    x["lens"][-1] = T
    if n > 8:
        x["lens"][:8] = [0, 1, T - 1, max(T - 2, 0), max(T - 3, 0), max(T - 4, 0), T, 0]
    adv = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    check_loss(B, x, adv, 0.2, 0.28, beta_kl=0.04, beta_ent=0.01, agg=n & 1)
    # the same rows one element into rows of T + 3, as views: the same bits, and what lies around the gradient's rows stays
    def view(a):
        wide = torch.full((n, T + 3), float("nan"), device="cuda")
        wide[:, 1:T + 1] = dev(a)
        return wide[:, 1:T + 1]
    names = ("logprob", "old_logprob", "kl", "entropy")
    one = B.rl_policy_loss(dev(x["logprob"]), dev(x["old_logprob"]), dev(adv), dev(x["lens"]), 0.2, 0.28, dev(x["kl"]),
                           dev(x["entropy"]), 0.04, 0.01)
    lp, old, kl, ent = (view(x[k]) for k in names)
    grad = view(x["kl"])
    around = grad._base
    stats = torch.empty(8, device="cuda")
    ds = B.policy_loss_desc_from_tensors(lp, old, dev(adv), dev(x["lens"]), 0.2, 0.28, stats, kl, ent, grad, 0.04, 0.01)
    ws = torch.empty(B.rl_policy_loss_workspace_bytes(ds), dtype=torch.uint8, device="cuda")
    ds.workspace, ds.workspace_bytes = ws.data_ptr(), ws.numel()
    a, l = dev(adv), dev(x["lens"])
    ds.advantages, ds.lens = a.data_ptr(), l.data_ptr()
    assert B.rl_policy_loss_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(grad, one[1]) and torch.equal(stats, one[0])
    assert around.shape == (n, T + 3) and around[:, 0].isnan().all() and around[:, T + 1:].isnan().all()


@pytest.mark.parametrize("T", [2**31 - 1, 2**31 - 4])
def test_the_longest_rows(B, T):  # noqa: F811
    """Rows whose last step of 1024 tokens ends behind 2^31: eight tokens and padding, the gradient zero to the last column."""
    import torch
    lp, grad = torch.zeros((1, T), device="cuda"), torch.full((1, T), 7.0, device="cuda")
    old = lp.clone()
    stats, adv, lens = torch.empty(8, device="cuda"), torch.ones(1, device="cuda"), torch.full((1,), 8, dtype=torch.int32, device="cuda")
    ds = B.policy_loss_desc_from_tensors(lp, old, adv, lens, 0.2, 0.28, stats, grad=grad)
    ws = torch.empty(B.rl_policy_loss_workspace_bytes(ds), dtype=torch.uint8, device="cuda")
    ds.workspace, ds.workspace_bytes = ws.data_ptr(), ws.numel()
    assert B.rl_policy_loss_raw(ds, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert stats[7].item() == 8 and (grad[0, :8] == -0.125).all() and torch.count_nonzero(grad).item() == 8
