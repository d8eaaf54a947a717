"""Unmask calls of many rollouts: which of them take one launch, and one that a single launch would refuse."""
import numpy as np
import pytest
import torch

from tests.gpu_util import print_case
from tests.test_f32_limits import run_host


def test_calls_of_one_launch(tmp_path):
    assert "one launch: ok" in run_host("one_launch_main", tmp_path)


@pytest.mark.gpu
def test_more_rollouts_than_one_launch_holds():
    """2^23 blocks of one position: 2^32 work items at 512 a block.  A vocabulary of two, so that the token is the larger logit
    and the confidence 1 / (1 + 2^-d) with d the difference in powers of two."""
    import paper_2605_23163_amd as F
    N = 1 << 23
    print_case(test="unmask_many", N=N)
    rng = np.random.default_rng(3)
    token, d = rng.integers(0, 2, N, dtype=np.int32), rng.integers(1, 9, N)
    x = np.zeros((N, 1, 2), np.float32)
    x[np.arange(N), 0, token] = (d * np.log(2.0)).astype(np.float32)
    mask = rng.integers(0, 2, (N, 1)).astype(np.uint8)
    m, t = torch.from_numpy(mask.copy()).cuda(), torch.full((N, 1), -3, dtype=torch.int32, device="cuda")
    _, conf, count, committed = F.fdd_unmask_step(torch.from_numpy(x).cuda(), m, None, 2.0, t)
    torch.cuda.synchronize()
    live = mask == 1
    np.testing.assert_array_equal(t.cpu().numpy(), np.where(live, token[:, None], -3))
    np.testing.assert_array_equal(m.cpu().numpy(), np.zeros_like(mask))
    np.testing.assert_array_equal(committed.cpu().numpy(), mask)
    np.testing.assert_array_equal(count.cpu().numpy(), mask[:, 0])
    np.testing.assert_allclose(conf.cpu().numpy()[live], 1.0 / (1.0 + 0.5 ** d[live[:, 0]]), rtol=2e-5)
