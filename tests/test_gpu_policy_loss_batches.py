"""The one-workgroup kernels around the policy loss where their strides end: sequence counts around multiples of the
1024 threads and of what a thread takes per round (8 lengths, 4 rows of partial sums), against the fp64 oracle."""
import numpy as np
import pytest

from paper_2512_21450_amd import workloads as wl
from tests.test_gpu_policy_loss import B, check_loss  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg", [0, 1])
@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 4095, 4097, 8192, 8193])
def test_sequence_counts(B, n, agg):  # noqa: F811
    x = wl.make_rollout_tokens(n, 12, 1, seed=n, lens=("uniform", 12))
    x["lens"][-1] = 12
    x["lens"][: n // 3: 5] = 0
    adv = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    check_loss(B, x, adv, 0.2, 0.28, beta_kl=0.04, beta_ent=0.01, agg=agg)
