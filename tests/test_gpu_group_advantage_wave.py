"""rl_group_advantage around 64 samples a group: up to there one wavefront holds a prompt, beyond a workgroup does.

Against the oracle with the bars of test_gpu_policy_loss.py.
"""
import pytest

from tests.test_gpu_policy_loss import B, test_group_advantage as check  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("P,G,M", [(1, 2, 1), (3, 63, 2), (513, 64, 1), (9, 65, 3)])
def test_group_sizes(B, mode, P, G, M):  # noqa: F811
    check(B, mode, P, G, M)
