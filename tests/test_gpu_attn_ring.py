"""The bf16 loop's ring of tiles: workgroups of 4 wavefronts with two slots per operand (fewer than 6 units) and with four (6 and
more, several M-tiles), from no full tile to more than the ring holds, ragged ends, private tiles requested before, between and
after the full ones (a block and extensions of one tile and of several), segments that end inside an M-tile, and wavefronts
without rows.  Every row is compared; tolerance as derived in test_gpu_attn_tiles.py."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import ROW_TOL, print_case, rand_attn, row_error, to_dev, to_f64
from tests.test_attn_plan import DEALT

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


# N, B, Hkv, L, E: more private tiles than a workgroup's share of the units (they are dealt to several), up to more than are booked
# (64 units), a list of positions, and pieces without any tile
MANY = [(40, 1, 2, 300, 0), (130, 1, 1, 64, 0), (130, 1, 1, 0, 70), (24, 3, 2, 200, 130), (5, 40, 2, 700, 37), (33, 1, 8, 1408, 1), (9, 96, 1, 130, 192)]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", MANY)
def test_many_private_tiles(oracle, shape, D):
    import paper_2605_23163_amd as F
    N, B, Hkv, L, E = shape
    print_case(test="attn_private", shape=shape, D=D)
    rng = np.random.default_rng(N * 31 + L + E + D)
    d = rand_attn(rng, N, B, L, 2 * Hkv, Hkv, D, W.BF16)
    t = {k: to_dev(v) for k, v in d.items()}
    kw, okw = {}, {}
    if E:
        e = [W.to_storage(rng.standard_normal((N, E, Hkv, D)).astype(np.float32), W.BF16) for _ in "kv"]
        kw, okw = dict(ext_k=to_dev(e[0]), ext_v=to_dev(e[1]), E=E), dict(ext_k=e[0], ext_v=e[1], E=E)
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"], **okw).reshape(N * B, 2 * Hkv, D)
    v_max = max(np.abs(to_f64(x)).max() for x in (t["block_v"], *([t["prefix_v"]] if L else []), *([kw["ext_v"]] if E else [])))
    some = torch.arange(0, N * B, 3 if N * B > 50 else 2, dtype=torch.int32, device="cuda")
    for pos in (None, some):
        at = np.arange(N * B) if pos is None else pos.cpu().numpy()
        out = torch.zeros_like(t["q"])
        F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], out=out,
                         **kw, **({} if pos is None else dict(q_positions=pos)))
        torch.cuda.synchronize()
        got = to_f64(out).reshape(N * B, 2 * Hkv, D)[at]
        err = np.abs(got - ref[at]).max()
        assert np.isfinite(err) and err <= 3 * 2.0**-9 * v_max
        assert row_error(got, ref[at]) <= ROW_TOL


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shape", DEALT)
def test_every_form_of_plan(oracle, shape, causal):
    import paper_2605_23163_amd as F
    N, B, L, Hq, Hkv, D, E = shape
    print_case(test="attn_dealt", shape=shape, causal=causal)
    rng = np.random.default_rng(N + L + E + D)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.BF16)
    t = {k: to_dev(v) for k, v in d.items()}
    e = [W.to_storage(rng.standard_normal((N, E + 3, Hkv, D)).astype(np.float32), W.BF16) for _ in "kv"]
    kw = dict(ext_k=to_dev(e[0]), ext_v=to_dev(e[1]), E=E, causal_block=causal)
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"], causal_block=causal, ext_k=e[0], ext_v=e[1], E=E)
    v_max = max(np.abs(to_f64(x)).max() for x in (t["prefix_v"], t["block_v"], kw["ext_v"]))
    for pk in (None, F.fdd_prefix_pack(t["prefix_v"]) if L >= 64 else None):
        got = to_f64(F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], prefix_v_packed=pk, **kw))
        err = np.abs(got - ref).max()
        assert np.isfinite(err) and err <= 3 * 2.0**-9 * v_max
        assert row_error(got, ref) <= ROW_TOL


# N, B, Hq, Hkv, L, E, D, pieces of an M-tile (128 rows) with its private tiles in one place
LESS = [(20, 1, 28, 4, 138, 37, 128, 3), (40, 3, 8, 4, 300, 0, 64, 3)]


@pytest.mark.parametrize("shape", LESS)
def test_less_scratch(oracle, shape):
    # a call whose scratch is too small for the many pieces that its private tiles are dealt to, but enough for the few that there are
    # without, runs on those
    import ctypes as C

    import paper_2605_23163_amd.binding as b
    N, B, Hq, Hkv, L, E, D, pieces = shape
    print_case(test="attn_less_scratch", shape=shape)
    rng = np.random.default_rng(N + L)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.BF16)
    t = {k: to_dev(v) for k, v in d.items()}
    ext = [W.to_storage(rng.standard_normal((N, max(E, 1), Hkv, D)).astype(np.float32), W.BF16) for _ in "kv"]
    kw = dict(ext_k=ext[0], ext_v=ext[1], E=E) if E else {}
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"], **kw)
    dev_ext = [to_dev(x) for x in ext]
    out = torch.empty_like(t["q"])
    p = b._attn_params(*(t[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")), None, out, None, 0)
    p.stream = torch.cuda.current_stream().cuda_stream
    if E:
        p.ext_k, p.ext_v, p.E, p.ext_capacity = dev_ext[0].data_ptr(), dev_ext[1].data_ptr(), E, E
    lib, ok, refused = b.load_library(), 0, 5
    need = lib.fdd_block_attn_workspace(C.byref(p))
    small = Hkv * (-(-N * B * (Hq // Hkv) // 128)) * pieces * 128 * (2 * D + 8)
    assert small < need
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    for size, status in ((need, ok), (need - 1, refused), (need - 256, ok), (small, ok), (small - 256, refused), (0, refused)):
        out.fill_(7.0)
        p.workspace, p.workspace_bytes = ws.data_ptr(), size
        assert lib.fdd_block_attn(C.byref(p)) == status, size
        torch.cuda.synchronize()
        if status == ok:
            assert row_error(to_f64(out), ref) <= ROW_TOL
        else:
            assert bool((out == 7.0).all())
