"""Merge of the segments of an M-tile (bf16 path): segment counts on both sides of what a thread requests at once and of
every number of threads per chunk, M-tiles that are not full, and stream-K ranges (a different count per M-tile).

Tolerance: probabilities, averages and outputs are each rounded to bf16, 2^-9 of a value that is no larger than the
largest element of V: 3 x 2^-9 of that in all (the peaks leave rows that are one row of V, up to 4.5, so the 2e-2 that
averages of many keys meet does not hold here: 2.1e-2 seen at an output of 4).  Averages of many keys are far smaller than
that, so each row is also held to its own norm, and a test without a GPU shows that no tile can be missing within it."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import ROW_TOL, print_case, rand_attn, row_error, to_dev, to_f64


# N, B, Hq, Hkv, L, splits (0: the library's choice; 157 equal pieces for the third shape, free ranges for the last two)
SHAPES = [(1, 9, 3, 1, 640, 8), (1, 33, 1, 1, 640, 9), (1, 4, 1, 1, 20000, 0), (1, 5, 14, 2, 1100, 15), (1, 5, 14, 2, 1100, 16),
          (1, 32, 2, 2, 2200, 31), (1, 32, 2, 2, 2200, 32), (1, 3, 2, 1, 4100, 63), (1, 3, 2, 1, 4100, 64), (8, 40, 28, 4, 700, 9),
          (8, 40, 28, 4, 700, 3), (4, 64, 28, 4, 130, 2), (3, 43, 5, 1, 650, 0), (33, 40, 28, 4, 300, 0)]


def inputs(shape, D, peaks):
    """`peaks`: a few keys far above the rest, segments of very different weight.  Otherwise scores of less than one, so that
    every tile of keys has its share of every row."""
    N, B, Hq, Hkv, L, splits = shape
    rng = np.random.default_rng(N * 1009 + B * 31 + L + D + splits)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.BF16)
    if peaks:
        d["prefix_k"][:: max(1, L // 5)] = W.to_storage(3.0 * rng.standard_normal((len(range(0, L, max(1, L // 5))), Hkv, D)).astype(np.float32), W.BF16)
    else:
        d["q"] = W.to_storage(0.3 * rng.standard_normal((N, B, Hq, D)).astype(np.float32), W.BF16)
    return d


@pytest.mark.parametrize("shape", SHAPES)
def test_bound_sees_every_tile(shape):
    """The bound of the next test: the output without any one tile of 64 prefix keys is off by more than twice of it."""
    N, B, Hq, Hkv, L, splits = shape
    for D in (64, 128):
        d = {k: (v.astype(np.uint32) << 16).view(np.float32).astype(np.float64) for k, v in inputs(shape, D, False).items()}
        worst = np.zeros((L + 63) // 64)
        for b in range(min(B, 4)):
            k, v = (np.concatenate([d["prefix_" + x][:, 0], d["block_" + x][0, :, 0]]) for x in "kv")
            p = np.exp(k @ d["q"][0, b, 0] / np.sqrt(D))
            out = p @ v / p.sum()
            for t in range(worst.size):
                w = p[t * 64: min(L, t * 64 + 64)]
                without = (p @ v - w @ v[t * 64: min(L, t * 64 + 64)]) / (p.sum() - w.sum())
                worst[t] = max(worst[t], np.linalg.norm(without - out) / np.linalg.norm(out))
        assert worst.min() > 2 * ROW_TOL, (D, worst.argmin(), worst.min())


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", SHAPES)
def test_segment_counts(oracle, shape, D):
    import paper_2605_23163_amd as F
    splits = shape[-1]
    print_case(test="attn_merge", shape=shape, D=D)
    for peaks in (True, False):
        d = inputs(shape, D, peaks)
        t = {k: to_dev(v) for k, v in d.items()}
        out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], splits=splits)
        torch.cuda.synchronize()
        ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"])
        err = np.abs(to_f64(out) - ref).max()
        v_max = max(np.abs(to_f64(t[k])).max() for k in ("prefix_v", "block_v"))
        assert np.isfinite(err) and err <= 3 * 2.0**-9 * v_max
        assert row_error(to_f64(out), ref) <= ROW_TOL


@pytest.mark.gpu
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
