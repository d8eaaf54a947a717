"""Unmask calls small enough for one launch: rows at every place of a vector, more positions than wavefronts and than lanes,
blocks without an eligible position, ties, banned tokens, the K/V refresh, and the first size beyond (two launches).  Tokens,
masks and counts bit for bit against the oracle; confidences to the 2e-5 of an fp32 sum."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, to_dev

pytestmark = pytest.mark.gpu


# N, B, V, dtype (8 wavefronts a rollout, 4 KB a wavefront; more than 32 positions with as many rollouts, 128 at most; more than 1024
# rollouts of 4 positions or more: both sides of each line)
@pytest.mark.parametrize("case", [(1, 8, 512, W.F32), (3, 7, 1, W.F32), (2, 9, 3, W.BF16), (5, 33, 129, W.BF16), (4, 65, 227, W.BF16), (2, 128, 64, W.F32),
                                  (1, 128, 128, W.BF16), (2, 129, 100, W.BF16), (2, 32, 512, W.BF16), (1, 8, 1024, W.F32), (1, 8, 1025, W.F32),
                                  (1, 1, 2048, W.BF16), (1, 1, 2049, W.BF16), (66, 65, 99, W.BF16), (128, 128, 31, W.F32), (1027, 5, 33, W.F32),
                                  (1025, 3, 40, W.BF16)])
@pytest.mark.parametrize("tau", [0.0, 0.5, 2.0])
def test_one_launch(oracle, case, tau):
    import paper_2605_23163_amd as F
    N, B, V, dtype = case
    print_case(test="unmask_small", case=case, tau=tau)
    rng = np.random.default_rng(N * 131 + B * 7 + V)
    x = np.round(rng.standard_normal((N, B, V)) * 4) / 2           # ties
    hit = rng.random((N, B)) < 0.5
    n, b = np.nonzero(hit)
    x[n, b, rng.integers(0, V, n.size)] += 30.0
    x[0, 0, : V // 2] = -np.inf
    logits = W.to_storage(x.astype(np.float32), dtype)
    mask = rng.integers(0, 2, (N, B)).astype(np.uint8)
    mask[N - 1] = 0 if N > 1 else mask[N - 1]
    scaffold = (rng.random((N, B)) < 0.3).astype(np.uint8)
    tokens = np.full((N, B), -3, np.int32)
    ref = oracle.unmask_step(logits, mask, scaffold, tokens, tau)
    tk, tv = (rng.standard_normal((11, 2, 64)).astype(np.float32) for _ in range(2))
    bk, bv = (rng.standard_normal((N, B, 2, 64)).astype(np.float32) for _ in range(2))
    d = [torch.from_numpy(z.copy()).cuda() for z in (tk, tv, bk, bv)]
    m, t = torch.from_numpy(mask.copy()).cuda(), torch.from_numpy(tokens.copy()).cuda()
    _, conf, nun, com = F.fdd_unmask_step(to_dev(logits), m, torch.from_numpy(scaffold).cuda(), tau, t, refresh=tuple(d))
    torch.cuda.synchronize()
    el = (mask == 1) & (scaffold == 0)
    c = conf.cpu().numpy()
    np.testing.assert_allclose(c[el], ref["confidences"][el], rtol=2e-5)
    assert np.all(np.isneginf(c[~el]))
    # (a forced commit among equal confidences, and confidences at tau, may fall either way in fp32)
    same = np.array([not el[i].any() or (np.abs(ref["confidences"][i][el[i]] - tau).min() > 1e-4 and
                     (tau < 1 or np.sum(ref["confidences"][i][el[i]] >= ref["confidences"][i][el[i]].max() * (1 - 1e-6)) == 1)) for i in range(N)])
    for name, got in (("tokens", t), ("mask", m), ("n_unmasked", nun), ("committed", com)):
        np.testing.assert_array_equal(got.cpu().numpy()[same], ref[name][same], err_msg=name)
    comm = com.cpu().numpy() == 1
    rk, rv = oracle.block_kv_update(t.cpu().numpy(), comm.astype(np.uint8), tk, tv, bk, bv)
    np.testing.assert_array_equal(d[2].cpu().numpy(), rk)
    np.testing.assert_array_equal(d[3].cpu().numpy(), rv)
