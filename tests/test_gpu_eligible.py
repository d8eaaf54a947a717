"""Vocabulary passes that deal their workgroups to eligible rows only: row counts at the ends of the range and at the 16
positions of a lane, every kind of mask, positions that start at odd addresses, one and several pieces per row, threads
per piece on both sides.  The sampled verifier deals rows of any length, the unmask step and the greedy verifier long ones
(32 KB a piece) only: the short cases are row by row for those two.  Tokens, masks and counts bit for bit against the oracle;
confidences to the 2e-5 of an fp32 sum."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, to_dev

pytestmark = pytest.mark.gpu

# N, B, V, dtype.  513, 514, 527, 528, 1009, 1023, 1024, 1025 rows of one piece; 172 rows of 5 pieces of 16 KB (row by row);
# 130 rows of 7 of 39 KB with sums and 8 of 34 KB without (910 and 1040 workgroups dealt)
CASES = [(513, 1, 40, W.BF16), (257, 2, 33, W.F32), (31, 17, 100, W.BF16), (33, 16, 64, W.F32), (1009, 1, 9, W.BF16),
         (93, 11, 500, W.BF16), (16, 64, 257, W.BF16), (41, 25, 31, W.F32), (43, 4, 41003, W.BF16), (26, 5, 70001, W.F32)]

# pieces of 32 KB and more.  513 rows of one piece of 32 KB; 514 and 1009 of one of 66 KB with sums (512 threads), two of 33 KB without
# (1028 and 2018 workgroups); 1024 of one of 32 KB (without sums row by row); 1025 (past the range); 250 of four of 68 KB with
# sums (512 threads), eight of 34 KB without
LONG = [(513, 1, 8200, W.F32), (257, 2, 17000, W.F32), (1009, 1, 17000, W.F32), (16, 64, 16500, W.BF16), (41, 25, 8300, W.F32), (10, 25, 70001, W.F32)]


def odd(a, by):
    """the array on the GPU, starting `by` bytes off an aligned address"""
    buf = torch.zeros(a.size + 64, dtype=torch.uint8, device="cuda")
    v = buf[by: by + a.size].view(a.shape)
    v.copy_(torch.from_numpy(a))
    return v


@pytest.mark.parametrize("case,kind", [(c, k) for c in CASES for k in ("random", "all", "none", "first", "last", "sparse", "no_scaffold")] +
                         [(c, k) for c in LONG for k in ("random", "last", "sparse")])
def test_rows_and_masks(oracle, case, kind):
    import paper_2605_23163_amd as F
    N, B, V, dtype = case
    print_case(test="eligible_rows", case=case, kind=kind)
    rng = np.random.default_rng(N * 31 + B + V)
    logits = W.to_storage((rng.standard_normal((N, B, V)) * 2).astype(np.float32), dtype)
    mask = rng.integers(0, 3, (N, B)).astype(np.uint8)           # (2 is not a mask)
    scaffold = (rng.random((N, B)) < 0.4).astype(np.uint8) * np.uint8(255)
    if kind == "no_scaffold":
        scaffold = None
    elif kind != "random":
        mask[:], scaffold[:] = 0, 0
        flat = mask.reshape(-1)
        if kind == "all":
            flat[:] = 1
        elif kind == "first":
            flat[0] = 1
        elif kind == "last":
            flat[-1] = 1
        elif kind == "sparse":
            flat[::97] = 1
    tokens = np.full((N, B), -3, np.int32)
    ref = oracle.unmask_step(logits, mask, scaffold, tokens, 0.0)        # tau = 0: every eligible position commits
    lg = to_dev(logits)
    by = N % 16 + 1
    m, t = odd(mask, by), torch.from_numpy(tokens.copy()).cuda()
    sc = None if scaffold is None else odd(scaffold, by + 2)
    _, conf, nun, com = F.fdd_unmask_step(lg, m, sc, 0.0, t)
    torch.cuda.synchronize()
    for name, got in (("tokens", t), ("mask", m), ("n_unmasked", nun), ("committed", com)):
        np.testing.assert_array_equal(got.cpu().numpy(), ref[name], err_msg=name)
    el = ref["committed"] == 1
    np.testing.assert_allclose(conf.cpu().numpy()[el], ref["confidences"][el], rtol=2e-5)
    # the verifiers on the same rows: half of the drafts are the greedy token
    draft = np.where(rng.random((N, B)) < 0.5, ref["candidates"], rng.integers(0, V, (N, B))).astype(np.int32)
    for temperature in (0.0, 0.8):
        if temperature and V > 5000:
            continue      # (the oracle's sampler is slow; its pieces are covered elsewhere)
        rv = oracle.verify_step(logits, mask, scaffold, draft, tokens, temperature=temperature, seed=5)
        m, t = odd(mask, by), torch.from_numpy(tokens.copy()).cuda()
        _, nacc, acc = F.fdd_verify_step(lg, m, sc, torch.from_numpy(draft).cuda(), t, temperature=temperature, seed=5)
        torch.cuda.synchronize()
        for name, got in (("tokens", t), ("mask", m), ("n_accepted", nacc), ("accepted", acc)):
            np.testing.assert_array_equal(got.cpu().numpy(), rv[name], err_msg=f"{name} at temperature {temperature}")
