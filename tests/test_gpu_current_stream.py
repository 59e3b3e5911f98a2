"""The stream a tensor function enqueues on: the caller's, or torch's current one, with torch's shortcut to its handle and without."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shortcut", [True, False])
def test_the_stream_of_a_call(shortcut, monkeypatch):
    import torch
    from paper_2512_21450_amd import binding as B
    if not shortcut:
        monkeypatch.setattr(B, "_current_raw_stream", None)
    t = torch.zeros(1, device="cuda")
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    assert B._stream_handle(None, t) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert B._stream_handle(None, t) == side.cuda_stream
        assert B._stream_handle(other, t) == other.cuda_stream
        # partials that the side stream makes, merged behind them on the same stream
        o = torch.randn((5, 1000, 64), device="cuda")
        lse = torch.randn((5, 1000), device="cuda")
        torch.cuda._sleep(1 << 20)
        o.mul_(2.0)
        out, l = B.rl_lse_combine(o, lse)
    side.synchronize()
    w = torch.softmax(lse.double(), 0)[:, :, None]
    assert (out - (w * o.double()).sum(0)).abs().max() < 1e-5
    assert (l - torch.logsumexp(lse.double(), 0)).abs().max() < 1e-5
