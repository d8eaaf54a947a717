"""Both M-tile sizes of the bf16 path, 256 rows (8 wavefronts, four ring slots per operand) and 128 (4 wavefronts, two slots or
four): row counts at the edges of a wavefront's 32 and of both tiles, key runs of 0 full tiles and more, ragged ends, several
pieces, and calls on both sides of the lines between them: more than 256 M-tiles of 128 rows; 9 units per compute unit at D = 128, 5
at D = 64 (64 KV heads of 34 / 35 and 18 / 19 prefix tiles); 6 units a workgroup, from which on it has four slots (20 KV heads of
29 / 30 tiles).  test_attn_plan.py checks on the host that these are the two sides.

Tolerance: probabilities, averages and outputs are each rounded to bf16, 2^-9 of a value that is no larger than the largest
element of V: 3 x 2^-9 of that in all; and each row to its own norm."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import ROW_TOL, print_case, rand_attn, row_error, to_dev, to_f64

pytestmark = pytest.mark.gpu

# N, B, Hkv (one query head each), L
LARGE = [(1, 300, 100, L) for L in (0, 40, 64, 130, 192, 256, 321, 600)] + \
        [(1, B, 100, 200) for B in (257, 287, 288, 289, 320, 384, 511)] + [(3, 100, 90, 300), (9, 31, 120, 128)]
SMALL = [(1, B, 3, L) for B in (1, 31, 32, 33, 127, 128, 129, 160) for L in (64, 500)] + \
        [(1, 70, 2, L) for L in (0, 10, 63, 65, 128, 129, 1024, 2049)] + [(5, 50, 2, 700), (7, 18, 1, 333)]
LINE = [(1, 2, 64, 64 * t) for t in (14, 15, 18, 19, 22, 23, 34, 35)]
SLOTS = [(1, 140, 20, 64 * t) for t in (29, 30)]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", LARGE + SMALL + LINE + SLOTS)
def test_rows_and_tiles(oracle, shape, D):
    import paper_2605_23163_amd as F
    N, B, Hkv, L = shape
    print_case(test="attn_tiles", shape=shape, D=D)
    rng = np.random.default_rng(N * 1009 + B * 31 + L + D)
    d = rand_attn(rng, N, B, L, Hkv, Hkv, D, W.BF16)
    t = {k: to_dev(v) for k, v in d.items()}
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"])
    v_max = max(np.abs(to_f64(t[k])).max() for k in (("prefix_v", "block_v") if L else ("block_v",)))
    for pk in (None, F.fdd_prefix_pack(t["prefix_v"]) if L >= 64 else None):
        out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], prefix_v_packed=pk)
        torch.cuda.synchronize()
        err = np.abs(to_f64(out) - ref).max()
        assert np.isfinite(err) and err <= 3 * 2.0**-9 * v_max
        assert row_error(to_f64(out), ref) <= ROW_TOL
