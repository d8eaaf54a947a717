"""GPU parity of fp32 attention in row tiles of 16, which calls take that leave half of the compute units idle, at the edges of
its tiles and on both sides of the rule.

Tolerance: fp32 arithmetic on scores of D products of size 1 and averages of values up to 5, a few 2^-24 of 5: 1e-5 is 30 of them."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, rand_attn, to_dev, to_f64

pytestmark = pytest.mark.gpu

TOL = 1e-5

# (N, B, L, Hq, Hkv, E, D): one row, a full tile, one row more; tiles of several rollouts; rollouts that cross tiles; keys of a
# single tile and of none; key ranges shared by workgroups; 448 workgroups of 32 rows, 96, 132 (32-row tiles, beyond 128) and 128
SHAPES = [(1, 1, 0, 1, 1, 0, 64), (1, 4, 15, 4, 1, 0, 64), (1, 17, 33, 4, 4, 0, 128), (7, 3, 100, 2, 1, 5, 64), (3, 11, 64, 6, 2, 17, 128),
          (1, 8, 5000, 4, 1, 0, 64), (5, 5, 900, 14, 2, 9, 128), (16, 32, 31, 28, 4, 0, 64), (2, 33, 48, 32, 32, 0, 128), (33, 32, 20, 4, 1, 0, 64),
          (32, 32, 20, 4, 1, 0, 64)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("causal", [False, True])
def test_tile_edges(oracle, shape, causal):
    import paper_2605_23163_amd as F
    print_case(test="f32_few_edges", shape=shape, causal=causal)
    N, B, L, Hq, Hkv, E, D = shape
    rng = np.random.default_rng(L + N)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.F32)
    ext = {}
    if E:
        d["ext_k"], d["ext_v"] = (rng.standard_normal((N, E + 2, Hkv, D)).astype(np.float32) for _ in range(2))
        ext = dict(ext_k=d["ext_k"], ext_v=d["ext_v"], E=E)
    t = {k: to_dev(v) for k, v in d.items()}
    dext = dict(ext_k=t["ext_k"], ext_v=t["ext_v"], E=E) if E else {}
    args = [t[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")]
    ref = oracle.block_attn(*(d[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")), causal_block=causal, **ext)
    for splits in (0, 3):      # (a forced cut leaves partial results of 16 rows to the merge)
        out = F.fdd_block_attn(*args, causal_block=causal, splits=splits, **dext)
        torch.cuda.synchronize()
        assert np.abs(to_f64(out) - ref).max() <= TOL, splits
    pos = np.sort(rng.permutation(N * B)[:(N * B + 2) // 3])
    out = torch.full_like(t["q"], 7.0)
    F.fdd_block_attn(*args, out=out, causal_block=causal, q_positions=torch.from_numpy(pos.astype(np.int32)).cuda(), **dext)
    torch.cuda.synchronize()
    got, ref = to_f64(out).reshape(N * B, Hq, D), ref.reshape(N * B, Hq, D)
    rest = np.ones(N * B, dtype=bool)
    rest[pos] = False
    assert np.all(got[rest] == 7.0) and np.abs(got[pos] - ref[pos]).max() <= TOL
