"""The one-launch decode kernel over paged stores whose sequences are finished in part: their rows are zeros and -inf whatever the
stores hold, and nothing of them is read (NaN in their q, their pages and the prefixes of prompts that have no live sequence; page
ids and lengths that are out of any range).  All wavefront forms, lengths of one, two and many tiles per wavefront.  Tolerances as
in test_gpu_unit."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests import util
from tests.test_gpu_unit import EXACT, LEAN, B, compare  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu


def nan_like(t):
    return 0x7FC0 if t.dtype == np.uint16 else (0x7F if t.dtype == np.uint8 else np.nan)


@pytest.mark.parametrize("which", ["none live", "one prompt live", "every third", "all but one"])
@pytest.mark.parametrize("page", [16, 32, 128])
@pytest.mark.parametrize("P,G,Lp,Ls", [(3, 4, 300, 290), (24, 8, 140, 700), (75, 4, 70, 200), (160, 8, 33, 40)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("e4m3", 64), ("bf16", 128), ("e4m3", 128)])
def test_finished_sequences(B, dtype, d, P, G, Lp, Ls, page, which):  # noqa: F811
    import torch
    n = P * G
    act = {"none live": np.zeros(n), "one prompt live": np.arange(n) // G == P - 1, "every third": np.arange(n) % 3 == 1,
           "all but one": np.arange(n) != G}[which].astype(np.uint8)
    x = util.random_case(P * d + Ls, P, G, 6, 2, d, Lp, Ls, "f32" if dtype == "f32" else "bf16")
    y = wl.to_pages(wl.kv_to_e4m3(x) if dtype == "e4m3" else x, page, seed=1)
    ro, rl = util.oracle_paged(y, 0.1, G, active=act)
    dead = act == 0
    y["q"][dead] = nan_like(y["q"])
    for b in np.flatnonzero(dead):
        used = y["block_table"][b, :-(-int(y["suffix_lens"][b]) // page)]
        y["k_pages"][used] = y["v_pages"][used] = nan_like(y["k_pages"])
    y["block_table"][dead], y["suffix_lens"][dead] = 1 << 30, 1 << 30
    for p in range(P):
        if dead[p * G:(p + 1) * G].all():
            y["k_prefix"][p] = y["v_prefix"][p] = nan_like(y["k_prefix"])
            y["prefix_lens"][p] = 1 << 30
    out, lse = util.gpu_run_paged(util.to_device(y), 0.1, G, active=torch.from_numpy(act).cuda())
    assert not out[torch.from_numpy(dead).cuda()].any()
    compare(out, lse, ro, rl, LEAN if d == 128 else EXACT, (dtype, d, P, page, which))
