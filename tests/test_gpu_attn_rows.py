"""M-tiles that are not full: wavefronts without a stacked row only move tiles (bf16 path).

Row counts on both sides of a wavefront's 32 rows and of 256, key runs of 0..9 full tiles, with and without a ragged last
one, in one piece and in several.  Calls this short take M-tiles of 128 rows; those of 256 with idle wavefronts are in
test_gpu_attn_large_tiles.py.  Tolerance: 2e-2 for bf16 storage."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, rand_attn, to_dev, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("packed", [False, True])
# N, B, G (rows = N B G), L, splits
@pytest.mark.parametrize("shape", [(1, 1, 1, 64, 0), (1, 4, 8, 320, 1), (1, 33, 1, 256, 1), (1, 32, 4, 192, 1), (3, 43, 1, 577, 1),
                                   (1, 37, 7, 600, 3), (1, 65, 4, 130, 1), (2, 72, 2, 448, 2), (1, 32, 7, 40, 0), (1, 32, 7, 1024, 2)])
def test_wavefronts_without_rows(oracle, shape, packed, D):
    import paper_2605_23163_amd as F
    N, B, G, L, splits = shape
    print_case(test="attn_rows", shape=shape, packed=packed, D=D)
    rng = np.random.default_rng(N * 1009 + B * 31 + L + D)
    d = rand_attn(rng, N, B, L, 2 * G, 2, D, W.BF16)
    t = {k: to_dev(v) for k, v in d.items()}
    pk = F.fdd_prefix_pack(t["prefix_v"]) if packed else None
    out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], splits=splits, prefix_v_packed=pk)
    torch.cuda.synchronize()
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"])
    got = to_f64(out)
    assert np.isfinite(got).all() and np.abs(got - ref).max() <= 2e-2
