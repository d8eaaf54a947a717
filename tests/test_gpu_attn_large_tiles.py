"""M-tiles of 256 rows (bf16 path, 8 wavefronts): shapes that the plan keeps there, plain V and V laid out.  Several problems in a
launch with pieces weighted by XCD, the verify pass, extensions, M-tiles with one row and with all, every number of merge
threads per chunk, one piece and free ranges.  That the plan does keep them there is checked from the workspace, which holds
segments x 256 rows of averages (D bf16) and (m, l).

A few dozen rows of each are compared: the first and last of every problem, M-tile and wavefront edge, and random ones."""
import ctypes as C

import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import ROW_TOL, print_case, rand_attn, row_error, to_dev, to_f64

pytestmark = pytest.mark.gpu

# name: problems, N, B, Hq, Hkv, L, D, E, causal, segments of an M-tile (free ranges: at most)
CASES = {
    "batch, weighted pieces": (2, 10, 50, 16, 2, 8200, 128, 0, False, 4),
    "verify pass, weighted pieces": (1, 10, 50, 32, 4, 8200, 128, 0, True, 4),
    "extension and verify pass": (1, 7, 33, 28, 4, 5003, 128, 37, True, 9),
    "four rows, 8 merge threads": (1, 1, 4, 8, 8, 20000, 128, 0, False, 32),
    "four rows, 4 merge threads": (1, 1, 4, 10, 10, 15000, 128, 0, False, 24),
    "four rows, 2 merge threads": (1, 1, 4, 20, 20, 7700, 128, 0, False, 12),
    "33 rows, D = 64, 8 merge threads": (1, 1, 33, 8, 8, 12000, 64, 0, False, 32),
    "batch of extensions, D = 64": (3, 2, 40, 21, 3, 6000, 64, 70, False, 9),
    "free ranges": (1, 60, 80, 16, 2, 700, 128, 0, False, 2),
}


def rows_to_compare(rng, N, B, Hq, Hkv):
    G = Hq // Hkv
    R = N * B * G                                # stacked rows of a KV head: (n, b, head of the group)
    r = {0, R - 1} | {min(e + o, R - 1) for e in range(0, R, 256) for o in (0, 31, 32, 255)} | set(rng.integers(0, R, 16).tolist())
    r = np.array(sorted(r) if len(r) <= 60 else sorted(rng.choice(sorted(r), 60, replace=False)))
    kh = rng.integers(0, Hkv, r.size)
    return np.stack([r // G // B, r // G % B, kh * G + r % G], axis=1).astype(np.int32)


@pytest.mark.parametrize("name", CASES)
def test_rows_against_oracle(oracle, name):
    import paper_2605_23163_amd as F
    from paper_2605_23163_amd import binding as Bd
    P, N, B, Hq, Hkv, L, D, E, causal, segments = CASES[name]
    print_case(test="attn_large_tiles", name=name)
    rng = np.random.default_rng(L + D + P)
    d = [rand_attn(rng, N, B, L, Hq, Hkv, D, W.BF16) for _ in range(P)]
    ext = [[W.to_storage(rng.standard_normal((N, E + 3, Hkv, D)).astype(np.float32), W.BF16) for _ in "kv"] for _ in range(P)]
    t = {k: torch.stack([to_dev(x[k]) for x in d]) for k in d[0]}
    kw = dict(causal_block=causal)
    if E:
        kw.update(ext_k=torch.stack([to_dev(x[0]) for x in ext]), ext_v=torch.stack([to_dev(x[1]) for x in ext]), E=E)
    rows = rows_to_compare(rng, N, B, Hq, Hkv)
    ref = [oracle.block_attn(*(x[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")), rows=rows, causal_block=causal,
                             **(dict(ext_k=e[0], ext_v=e[1], E=E) if E else {})) for x, e in zip(d, ext)]
    for packed in (None, torch.stack([F.fdd_prefix_pack(v) for v in t["prefix_v"]])):
        p = Bd._batched_params(*(t[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")), None, None, 0, packed, causal,
                               kw.get("ext_k"), kw.get("ext_v"), E)
        m_tiles = P * Hkv * ((N * B * (Hq // Hkv) + 255) // 256)
        need = Bd.load_library().fdd_block_attn_workspace(C.byref(p))
        assert need == m_tiles * segments * 256 * (D * 2 + 8)
        out = F.fdd_block_attn_batched(*(t[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")), prefix_v_packed=packed, **kw)
        torch.cuda.synchronize()
        got = to_f64(out)
        assert np.isfinite(got).all()
        for i in range(P):
            assert row_error(got[i][tuple(rows.T)], ref[i]) <= ROW_TOL, (i, packed is not None)
