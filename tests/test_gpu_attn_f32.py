"""GPU parity of the fp32 attention path at the edges of its tiles: 32-row tiles,
16-key tiles, 8 wavefronts that share the key tiles of a row tile (more wavefronts
than tiles among them), split counts, and row tiles that span several rollouts.

Tolerance: the task's 1e-4 (sums of at most 3 000 terms of magnitude 1 in fp32 stay
below 3 000 * 2^-24 = 2e-4 of the largest term and near 1e-6 of the result in practice)."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, rand_attn, to_dev, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
# N, B, L, Hq, Hkv, E, splits
@pytest.mark.parametrize("shape", [
    (1, 1, 1, 1, 1, 0, 0), (1, 31, 15, 1, 1, 0, 0), (1, 32, 16, 2, 2, 0, 0), (1, 33, 17, 1, 1, 16, 0), (2, 16, 0, 1, 1, 0, 0),
    (4, 8, 127, 4, 2, 15, 0), (11, 3, 128, 1, 1, 17, 0), (3, 13, 129, 5, 1, 1, 2), (2, 17, 2047, 7, 1, 0, 64), (1, 4, 40, 8, 8, 3, 3),
    (1, 32, 2900, 7, 1, 0, 0),
])
@pytest.mark.parametrize("causal", [False, True])
def test_tile_edges(oracle, shape, D, causal):
    import paper_2605_23163_amd as F
    N, B, L, Hq, Hkv, E, splits = shape
    print_case(test="attn_f32_tile_edges", shape=shape, D=D, causal=causal)
    rng = np.random.default_rng(N * 1000003 + L * 101 + B * 7 + D)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.F32)
    ek, ev = (rng.standard_normal((N, E + 2, Hkv, D)).astype(np.float32) for _ in range(2))
    t = {k: to_dev(v) for k, v in d.items()}
    kw = dict(ext_k=to_dev(ek), ext_v=to_dev(ev), E=E) if E else {}
    okw = dict(ext_k=ek, ext_v=ev, E=E) if E else {}
    out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], causal_block=causal, splits=splits, **kw)
    torch.cuda.synchronize()
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"], causal_block=causal, **okw)
    got = to_f64(out)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 1e-4
