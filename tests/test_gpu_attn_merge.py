"""Merge of the segments of an M-tile (bf16 path): segment counts on both sides of what a thread requests at once and of
every number of threads per chunk, M-tiles that are not full, and stream-K ranges (a different count per M-tile).

Tolerance: probabilities, averages and outputs are each rounded to bf16, 2^-9 of a value that is no larger than the
largest element of V: 3 x 2^-9 of that in all (the peaks leave rows that are one row of V, up to 4.5, so the 2e-2 that
averages of many keys meet does not hold here: 2.1e-2 seen at an output of 4)."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, rand_attn, to_dev, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
# N, B, Hq, Hkv, L, splits (0: the library's choice; 157 equal pieces for the third shape, free ranges for the last two)
@pytest.mark.parametrize("shape", [
    (1, 9, 3, 1, 640, 8), (1, 33, 1, 1, 640, 9), (1, 4, 1, 1, 20000, 0), (1, 5, 14, 2, 1100, 15), (1, 5, 14, 2, 1100, 16),
    (1, 32, 2, 2, 2200, 31), (1, 32, 2, 2, 2200, 32), (1, 3, 2, 1, 4100, 63), (1, 3, 2, 1, 4100, 64), (8, 40, 28, 4, 700, 9),
    (8, 40, 28, 4, 700, 3), (4, 64, 28, 4, 130, 2), (3, 43, 5, 1, 650, 0), (33, 40, 28, 4, 300, 0)])
def test_segment_counts(oracle, shape, D):
    import paper_2605_23163_amd as F
    N, B, Hq, Hkv, L, splits = shape
    print_case(test="attn_merge", shape=shape, D=D)
    rng = np.random.default_rng(N * 1009 + B * 31 + L + D + splits)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.BF16)
    # a few keys far above the rest: segments of very different weight
    d["prefix_k"][:: max(1, L // 5)] = W.to_storage(3.0 * rng.standard_normal((len(range(0, L, max(1, L // 5))), Hkv, D)).astype(np.float32), W.BF16)
    t = {k: to_dev(v) for k, v in d.items()}
    out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], splits=splits)
    torch.cuda.synchronize()
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"])
    err = np.abs(to_f64(out) - ref).max()
    v_max = max(np.abs(to_f64(t[k])).max() for k in ("prefix_v", "block_v"))
    assert np.isfinite(err) and err <= 3 * 2.0**-9 * v_max


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", [(1, 4, 1, 1, 20000, 0), (8, 40, 28, 4, 700, 9), (4, 64, 28, 4, 260, 2)])
def test_large_values(oracle, shape, D):
    """Values up to 2e36: a segment's sum of them still fits fp32, the sum over all keys does not; the average does.
    Probabilities are 1; averages and outputs are each rounded to bf16, by 2^-8 of themselves at most."""
    import paper_2605_23163_amd as F
    N, B, Hq, Hkv, L, splits = shape
    print_case(test="attn_merge_large", shape=shape, D=D)
    rng = np.random.default_rng(L + D)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.BF16)
    d["q"] = np.zeros_like(d["q"])             # equal weights
    for k in ("prefix_v", "block_v"):
        d[k] = W.to_storage(rng.uniform(1e36, 2e36, d[k].shape).astype(np.float32), W.BF16)
    t = {k: to_dev(v) for k, v in d.items()}
    out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], splits=splits)
    torch.cuda.synchronize()
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"])
    np.testing.assert_allclose(to_f64(out), ref, rtol=2 * 2.0**-8)
