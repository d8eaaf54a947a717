"""fp32 attention away from small, finite scores: what the values of q, k and v may do to a result.

Scores that are exact in fp32 (small integers and eighths) isolate the softmax: the error against the oracle is then that
of the exponentials and of the merges of wavefronts and splits alone."""
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


def levels(rng, n, kind, raw_per_bit):
    """Integer or eighth-valued scores of n consecutive keys."""
    r = rng.integers(-64, 65, n) / 8.0                                  # +-8, in eighths
    if kind == "plateau":                                               # one large level, a reference of its own per wavefront
        return 4096.0 + r
    if kind == "ramp":                                                  # rises by 3 bits per 16 keys: a raise every third tile
        return np.round((np.arange(n) // 16) * 3 * raw_per_bit) + r / 8
    if kind == "fall":                                                  # the first keys hold everything, later ones nothing
        return -np.round((np.arange(n) // 16) * 3 * raw_per_bit) + r / 8
    peaks = 4096.0 * (rng.random(n) < 0.02)                             # "peaks": a few keys 2^8 and more above the rest
    return peaks + r


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", ["plateau", "ramp", "fall", "peaks"])
def test_exact_scores_of_large_magnitude(F, oracle, kind, causal, splits, D):
    # q picks channel 0 (the level) with weight 1 or 1/2, so that rows of one tile need different references.  c = scale
    # log2 e = 0.36 per score unit; ramps stay within 2^100.  V carries 2^-(level) where the scores ramp, so that every key
    # tile has the same share in the result and a lost rescale shows.
    N, B, L, Hq, Hkv, E, scale = 3, 20, 600, 4, 2, 21, 0.25
    print_case(test="exact_scores", kind=kind, causal=causal, splits=splits, D=D)
    rng = np.random.default_rng(D + 7 * splits + len(kind))
    raw_per_bit = 1.0 / (scale * np.log2(np.e))
    if kind in ("ramp", "fall"):
        L = 16 * 28 + 5

    def kv(*shape):
        n, heads = int(np.prod(shape)), Hkv
        s = levels(rng, n, kind, raw_per_bit)
        k = np.zeros((n, heads, D), dtype=np.float32)
        k[:, :, 0] = s[:, None]
        v = rng.standard_normal((n, heads, D))
        if kind in ("ramp", "fall"):
            v *= np.exp2(-np.round(s / raw_per_bit))[:, None, None]
        return k.reshape(*shape, heads, D), v.astype(np.float32).reshape(*shape, heads, D)

    pk, pv = kv(L)
    bk, bv = kv(N, B)
    ek, ev = kv(N, E)
    q = np.zeros((N, B, Hq, D), dtype=np.float32)
    q[..., 0] = 1.0
    if kind not in ("ramp", "fall"):
        q[:, 1::2, :, 0] = 0.5
    d = dict(q=q, prefix_k=pk, prefix_v=pv, block_k=bk, block_v=bv)
    got = to_f64(run(F, d, scale, causal, splits, (ek, ev), E))
    ref = oracle.block_attn(q, pk, pv, bk, bv, scale=scale, causal_block=causal, ext_k=ek, ext_v=ev, E=E)
    size = oracle.block_attn(q, pk, np.abs(pv), bk, np.abs(bv), scale=scale, causal_block=causal, ext_k=ek, ext_v=np.abs(ev), E=E)
    assert np.isfinite(got).all()
    # Per term: the rounding of c (2^-24 of an exponent of at most 6 bits where the key counts, times ln 2: 2.5e-7; of 90
    # bits in a ramp: 3.7e-6), of the exponent (the same once more), of exp2 (one unit: 6e-8), and of 700 ordered sums
    # (2^-24 each, growing with the root at most: 1.6e-6 in a ramp, whose keys all count; far fewer reach the size of the
    # sum otherwise).
    rel = (np.abs(got - ref) / size).max()
    bound = 1e-6 if kind in ("plateau", "peaks") else 1e-5
    print(f"error over sum of absolute terms: {rel:.2e}")
    assert rel <= bound, rel


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("splits", [0, 1, 5])
@pytest.mark.parametrize("std", [3.0, 6.0])
def test_spread_out_scores(F, oracle, std, splits, D):
    # q, k of standard deviation `std`: scores of deviation std^2 sqrt(D), exponents of std^2 log2 e = 13 and 52 bits, keys
    # that grow with their index, references raised many times.  Tolerance: a score is a sum of D products of size std^2,
    # rounded at partial sums of size up to 5 std^2 sqrt(D): D^1/2 2^-24 5 std^2 after the scale, a few times that for a
    # probability near its maximum, and |V| <= 5.
    N, B, L, Hq, Hkv = 2, 24, 700, 6, 2
    print_case(test="spread_scores", std=std, splits=splits, D=D)
    rng = np.random.default_rng(int(std) * 10 + splits + D)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.F32, std=std)
    d["prefix_v"], d["block_v"] = d["prefix_v"] / np.float32(std), d["block_v"] / np.float32(std)
    d["prefix_k"] *= np.linspace(0.2, 1.5, L, dtype=np.float32)[:, None, None]
    got = to_f64(run(F, d, splits=splits))
    ref = oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"])
    err = np.abs(got - ref).max()
    print(f"max-abs error {err:.2e}")
    assert err <= 5 * 4 * 5 * std * std * np.sqrt(D) * 2.0 ** -24


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
