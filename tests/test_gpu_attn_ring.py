"""The bf16 loop's ring of tiles: workgroups of 4 wavefronts with two slots per operand (fewer than 6 units) and with four (6 and
more, several M-tiles), from no full tile to more than the ring holds, ragged ends, private tiles requested before, between and
after the full ones (a block and extensions of one tile and of several), segments that end inside an M-tile, and wavefronts
without rows.  Every row is compared; tolerance as derived in test_gpu_attn_tiles.py."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import ROW_TOL, print_case, rand_attn, row_error, to_dev, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("E,causal", [(0, False), (70, True)])
@pytest.mark.parametrize("splits", [1, 2, 3])
def test_ring(oracle, D, E, causal, splits):
    import paper_2605_23163_amd as F
    N, B, Hkv, G = 3, 44, 1, 2                      # 264 stacked rows: M-tiles of 128, 128 and 8
    for tiles in (0, 1, 2, 3, 4, 5, 6, 9, 14):
        for rest in (0, 13):
            L = 64 * tiles + rest
            if L == 0:
                continue
            print_case(test="attn_ring", D=D, E=E, splits=splits, L=L)
            rng = np.random.default_rng(L * 7 + D + E + splits)
            d = rand_attn(rng, N, B, L, Hkv * G, Hkv, D, W.BF16)
            t = {k: to_dev(v) for k, v in d.items()}
            kw, okw = {}, {}
            if E:
                e = [W.to_storage(rng.standard_normal((N, E + 2, Hkv, D)).astype(np.float32), W.BF16) for _ in "kv"]
                kw, okw = dict(ext_k=to_dev(e[0]), ext_v=to_dev(e[1]), E=E), dict(ext_k=e[0], ext_v=e[1], E=E)
            ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"], causal_block=causal, **okw)
            v_max = max(np.abs(to_f64(x)).max() for x in (t["prefix_v"], t["block_v"], *([kw["ext_v"]] if E else [])))
            for pk in (None, F.fdd_prefix_pack(t["prefix_v"]) if L >= 64 else None):
                out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], prefix_v_packed=pk,
                                       causal_block=causal, splits=splits, **kw)
                torch.cuda.synchronize()
                err = np.abs(to_f64(out) - ref).max()
                assert np.isfinite(err) and err <= 3 * 2.0**-9 * v_max
                assert row_error(to_f64(out), ref) <= ROW_TOL
