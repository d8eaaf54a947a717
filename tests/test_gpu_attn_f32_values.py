"""fp32 attention away from small, finite scores: what the values of q, k and v may do to a result."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, rand_attn, to_dev, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import paper_2605_23163_amd as F
    F.load_library()
    return F


def run(F, d, scale=None, causal=False, splits=0, ext=None, E=0):
    t = {k: to_dev(v) for k, v in d.items()}
    kw = dict(ext_k=to_dev(ext[0]), ext_v=to_dev(ext[1]), E=E) if E else {}
    out = F.fdd_block_attn(t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"], scale=scale, causal_block=causal,
                           splits=splits, **kw)
    torch.cuda.synchronize()
    return out


# rows per rollout: a half, a quarter, an odd part and more than a whole row tile of 32; few tiles and several splits
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", [(2, 16, 1), (3, 8, 1), (5, 5, 3), (3, 40, 1), (2, 17, 4)])
@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_a_rollout_does_not_see_anothers_values(F, shape, splits, bad, D):
    N, B, G = shape
    L, Hkv, E = 50, 2, 19
    print_case(test="rollout_isolation", shape=shape, splits=splits, bad=bad, D=D)
    rng = np.random.default_rng(N * 100 + B + D)
    d = rand_attn(rng, N, B, L, G * Hkv, Hkv, D, W.F32)
    ek, ev = (rng.standard_normal((N, E, Hkv, D)).astype(np.float32) for _ in range(2))
    clean = to_f64(run(F, d, splits=splits, ext=(ek, ev), E=E))
    sick = 1
    others = [n for n in range(N) if n != sick]
    for name in ("block_v", "block_k", "ext_v", "ext_k"):
        x = dict(d, block_k=d["block_k"].copy(), block_v=d["block_v"].copy(), ext_k=ek.copy(), ext_v=ev.copy())
        x[name][sick, -1] = bad
        x[name][sick, 0, :, ::3] = bad
        e = (x.pop("ext_k"), x.pop("ext_v"))
        got = to_f64(run(F, x, splits=splits, ext=e, E=E))
        assert np.array_equal(got[others], clean[others]), name
        assert not np.isfinite(got[sick]).all(), name        # and the rollout itself does


def test_infinite_values_stay_infinite(F, oracle):
    # an infinity in the last key of a ragged run: every row that sees it is infinite there, not NaN, and finite elsewhere
    N, B, L, Hkv, D = 1, 21, 37, 1, 64
    print_case(test="infinite_value")
    rng = np.random.default_rng(3)
    d = rand_attn(rng, N, B, L, Hkv, Hkv, D, W.F32)
    for name in ("prefix_v", "block_v"):
        x = dict(d, **{name: d[name].copy()})
        x[name].reshape(-1, Hkv, D)[-1, :, 5] = np.inf
        got = to_f64(run(F, x))
        ref = oracle.block_attn(x["q"], x["prefix_k"], x["prefix_v"], x["block_k"], x["block_v"])
        assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and not np.isnan(got).any(), name
        fin = np.isfinite(ref)
        assert np.abs(got[fin] - ref[fin]).max() <= 1e-4


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_bad_query_row_spoils_itself_only(F, bad):
    N, B, L, Hq, Hkv, D = 2, 20, 100, 3, 1, 64
    print_case(test="bad_query", bad=bad)
    rng = np.random.default_rng(4)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.F32)
    clean = to_f64(run(F, d))
    x = dict(d, q=d["q"].copy())
    x["q"][1, 7, 2, :] = bad
    got = to_f64(run(F, x))
    keep = np.ones((N, B, Hq), dtype=bool)
    keep[1, 7, 2] = False
    assert np.array_equal(got[keep], clean[keep]) and np.isnan(got[1, 7, 2]).all()


def test_rows_of_block_keys_two_gigabytes_apart(F):
    # heads so many that the 16 keys of a tile span more than 2^31 bytes (15 x 580 000 heads x 64 x 4): every key must
    # count.  Checked against the same problem cut down to a few heads.
    B, Hkv, D = 16, 580000, 64
    print_case(test="wide_rows", Hkv=Hkv)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, bk, bv = (torch.randn((1, B, Hkv, D), device="cuda", generator=g) for _ in range(3))
    none = torch.empty((0, Hkv, D), device="cuda")
    out = F.fdd_block_attn(q, none, none, bk, bv)
    heads = torch.tensor([0, 1, 290000, Hkv - 1], device="cuda")
    cut = [x[:, :, heads].contiguous() for x in (q, bk, bv)]
    small = F.fdd_block_attn(cut[0], none[:, :4].contiguous(), none[:, :4].contiguous(), cut[1], cut[2])
    torch.cuda.synchronize()
    assert (out[:, :, heads] - small).abs().max().item() <= 1e-5
