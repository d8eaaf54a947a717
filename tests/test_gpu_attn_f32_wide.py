"""GPU parity of fp32 attention on the bf16 matrix pipe (128-row tiles, every fp32 product as six bf16 products) at the edges
of its tiles, and what values that are not finite do there.

Tolerance: products are kept to 2^-24 and sums are rounded to fp32, so results agree with the oracle as fp32 arithmetic does:
a score of D products of size 1 is off by a few 2^-24 sqrt(D), scaled by 1/sqrt(D), a probability by as much, and the average
of values up to 5 by 5 * 2^-24 times a few: 1e-5 is 30 times 2^-24 * 5."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, rand_attn, to_dev, to_f64
from tests.test_gpu_attn_f32_values import levels

pytestmark = pytest.mark.gpu

TOL = 1e-5

# (N, B, L, Hq, Hkv, E, D): row tiles of several rollouts, a part of one row tile over a full one, the last tile of 32 keys
# nearly empty and nearly full, extensions and blocks of less and more than a tile, fewer tiles than pieces would like
SHAPES = [(12, 20, 1025, 14, 2, 0, 128), (5, 39, 2527, 28, 4, 37, 64), (3, 33, 5000, 16, 4, 1, 128), (9, 65, 2200, 8, 2, 96, 64),
          (40, 7, 2311, 28, 4, 0, 64), (3, 70, 3009, 8, 8, 31, 128)]


@pytest.fixture(scope="module")
def F():
    import paper_2605_23163_amd as F
    F.load_library()
    return F


def make(shape, seed=0):
    N, B, L, Hq, Hkv, E, D = shape
    rng = np.random.default_rng(seed + L)
    d = rand_attn(rng, N, B, L, Hq, Hkv, D, W.F32)
    if E:
        d["ext_k"], d["ext_v"] = (rng.standard_normal((N, E + 2, Hkv, D)).astype(np.float32) for _ in range(2))
    return d


def run(F, d, E, check_wide=True, **kw):
    t = {k: to_dev(v) for k, v in d.items()}
    args = (t["q"], t["prefix_k"], t["prefix_v"], t["block_k"], t["block_v"])
    ext = dict(ext_k=t["ext_k"], ext_v=t["ext_v"], E=E) if E else {}
    if check_wide:      # the partial results of 128-row tiles, and not of 32-row tiles
        N, B, Hq, D = d["q"].shape
        Hkv = d["block_k"].shape[2]
        rows, per = N * B * (Hq // Hkv), 4 * D + 8
        need = F.fdd_block_attn_workspace(*args, **ext)
        assert need > 0 and need % (Hkv * ((rows + 127) // 128) * 128 * per) == 0, need
        assert need % (Hkv * ((rows + 31) // 32) * 32 * per) != 0, need
    out = F.fdd_block_attn(*args, **ext, **kw)
    torch.cuda.synchronize()
    return out


def reference(oracle, d, E, **kw):
    ext = dict(ext_k=d["ext_k"], ext_v=d["ext_v"], E=E) if E else {}
    return oracle.block_attn(d["q"], d["prefix_k"], d["prefix_v"], d["block_k"], d["block_v"], **ext, **kw)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("causal", [False, True])
def test_tile_edges(F, oracle, shape, causal):
    print_case(test="f32_wide_edges", shape=shape, causal=causal)
    d, E = make(shape), shape[5]
    got = to_f64(run(F, d, E, causal_block=causal))
    assert np.abs(got - reference(oracle, d, E, causal_block=causal)).max() <= TOL


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1], SHAPES[5]])
def test_rows_behind_the_last_key_are_not_read(F, shape):
    # The rows that follow a run of keys in memory are NaN.  Had a tile read one, its wavefront would have done its keys
    # again with fp32 products, whose sums differ in their last bits.
    print_case(test="f32_wide_behind", shape=shape)
    d, E, L = make(shape), shape[5], shape[2]
    clean = run(F, d, E)
    t = {k: to_dev(v) for k, v in d.items()}
    for k in ("prefix_k", "prefix_v", "block_k", "block_v"):
        flat = t[k].reshape(-1, *t[k].shape[-2:])
        t[k] = torch.cat([flat, torch.full_like(flat[:40], float("nan"))])[:flat.shape[0]].reshape(t[k].shape)
    ext = {}
    if E:
        t["ext_k"][:, E:] = t["ext_v"][:, E:] = float("nan")
        ext = dict(ext_k=t["ext_k"], ext_v=t["ext_v"], E=E)
    got = F.fdd_block_attn(*(t[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")), **ext)
    torch.cuda.synchronize()
    assert torch.equal(got, clean)


def test_scores_that_grow_along_the_keys(F, oracle):
    # exponents of up to +-40 that rise with the key: the reference is raised again and again, in every piece
    shape = SHAPES[1]
    print_case(test="f32_wide_growing", shape=shape)
    d, E, D = make(shape), shape[5], shape[6]
    d["q"][..., 0] = 1.0
    d["prefix_k"][..., 0] = np.linspace(0, 40 * np.sqrt(D), shape[2], dtype=np.float32)[:, None]
    got, ref = to_f64(run(F, d, E)), reference(oracle, d, E)
    # (scores up to 40 sqrt(D), rounded to 2^-24 of that, are exponents off by 40 * 2^-24)
    assert np.abs(got - ref).max() <= 8 * TOL


@pytest.mark.parametrize("N,D", [(16, 64), (6, 128)])        # 3 and 7 or 8 pieces
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", ["plateau", "ramp", "fall", "peaks"])
def test_exact_scores_of_large_magnitude(F, oracle, kind, causal, N, D):
    # scores, values and bounds of the test of this name for the other tiles, on which see there; pieces chosen by the library
    B, L, Hq, Hkv, E, scale = 20, 600, 28, 4, 21, 0.25
    print_case(test="f32_wide_exact_scores", kind=kind, causal=causal, D=D)
    rng = np.random.default_rng(D + len(kind))
    raw_per_bit = 1.0 / (scale * np.log2(np.e))
    if kind in ("ramp", "fall"):
        L = 16 * 28 + 5

    def kv(*shape):
        n = int(np.prod(shape))
        s = levels(rng, n, kind, raw_per_bit)
        k = np.zeros((n, Hkv, D), dtype=np.float32)
        k[:, :, 0] = s[:, None]
        v = rng.standard_normal((n, Hkv, D))
        if kind in ("ramp", "fall"):
            v *= np.exp2(-np.round(s / raw_per_bit))[:, None, None]
        return k.reshape(*shape, Hkv, D), v.astype(np.float32).reshape(*shape, Hkv, D)

    d = {}
    d["prefix_k"], d["prefix_v"] = kv(L)
    d["block_k"], d["block_v"] = kv(N, B)
    d["ext_k"], d["ext_v"] = kv(N, E)
    d["q"] = np.zeros((N, B, Hq, D), dtype=np.float32)
    d["q"][..., 0] = 1.0
    if kind not in ("ramp", "fall"):
        d["q"][:, 1::2, :, 0] = 0.5
    got = to_f64(run(F, d, E, scale=scale, causal_block=causal))
    ref = reference(oracle, d, E, scale=scale, causal_block=causal)
    size = reference(oracle, {k: np.abs(v) if k.endswith("_v") else v for k, v in d.items()}, E, scale=scale, causal_block=causal)
    rel = (np.abs(got - ref) / size).max()
    print(f"error over sum of absolute terms: {rel:.2e}")
    assert np.isfinite(got).all() and rel <= (1e-6 if kind in ("plateau", "peaks") else 1e-5), rel


def wide_size(rows, Hkv, D, pieces):
    """Scratch of 128-row tiles in so many pieces."""
    up = lambda n: (n + 255) // 256 * 256
    return up(Hkv * -(-rows // 128) * 128 * pieces * D * 4) + up(Hkv * -(-rows // 128) * 128 * pieces * 8)


def test_listed_positions_and_a_batch(F, oracle):
    shape = (5, 39, 2527, 28, 4, 0, 64)
    print_case(test="f32_wide_list_batch", shape=shape)
    d = make(shape)
    N, B, L, Hq, Hkv, E, D = shape
    pos = np.sort(np.random.default_rng(1).permutation(N * B)[:149])
    full = to_f64(run(F, d, 0)).reshape(N * B, Hq, D)
    out = torch.full((N, B, Hq, D), 7.0, device="cuda")
    t = {k: to_dev(v) for k, v in d.items()}
    args = [t[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")]
    # (scratch of 128-row tiles and of no others: the rows of a list and of a batch are not multiples of 32)
    need = F.fdd_block_attn_workspace(*args, n_q_positions=149)
    assert need in [wide_size(149 * 7, Hkv, D, s) for s in range(2, 65)] and need % (Hkv * 33 * 32 * (4 * D + 8)) != 0
    F.fdd_block_attn(*args, out=out, q_positions=torch.from_numpy(pos.astype(np.int32)).cuda())
    torch.cuda.synchronize()
    got = to_f64(out).reshape(N * B, Hq, D)
    rest = np.ones(N * B, dtype=bool)
    rest[pos] = False
    assert np.all(got[rest] == 7.0) and np.abs(got[pos] - full[pos]).max() <= TOL
    e = make(shape, seed=1)
    both = [torch.stack([to_dev(d[k]), to_dev(e[k])]) for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")]
    need = F.fdd_block_attn_batched_workspace(*both)
    assert need in [wide_size(N * B * 7, 2 * Hkv, D, s) for s in range(2, 65)] and need % (2 * Hkv * 43 * 32 * (4 * D + 8)) != 0
    out = F.fdd_block_attn_batched(*both)
    torch.cuda.synchronize()
    for i, x in enumerate((d, e)):
        assert np.abs(to_f64(out[i]) - reference(oracle, x, 0)).max() <= TOL


# All variants of the merge: 5 pieces (a thread sums them all), 11 (two threads) and 22 to 26 (four), the last of which hold
# private keys only, for every row tile or all but one
PIECES = [(3, 64, 334, 28, 4, 32, 128), (3, 64, 732, 28, 4, 128, 64), (1, 64, 498, 28, 4, 128, 128), (1, 64, 505, 28, 4, 128, 64),
          (4, 20, 1005, 8, 8, 128, 128), (4, 20, 1006, 8, 8, 64, 64)]


@pytest.mark.parametrize("shape", PIECES)
def test_nan_keys_in_all_pieces_but_the_last(F, oracle, shape):
    # every score of a piece is NaN, so that nothing ever raises its reference: what it leaves is NaN all the same
    print_case(test="f32_wide_nan_pieces", shape=shape)
    d, E = make(shape), shape[5]
    got = to_f64(run(F, d, E))
    assert np.abs(got - reference(oracle, d, E)).max() <= TOL
    d["prefix_k"][..., 3] = np.nan
    assert np.isnan(to_f64(run(F, d, E))).all()


@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[0]])
@pytest.mark.parametrize("bad", [np.inf, np.nan, -np.inf])
def test_values_that_are_not_finite_reach_only_who_sees_them(F, oracle, shape, bad):
    # (rows that share a wavefront with a sick one are computed with fp32 products instead: the same up to rounding)
    print_case(test="f32_wide_not_finite", shape=shape, bad=bad)
    d, E = make(shape), shape[5]
    clean = to_f64(run(F, d, E))
    sick, others = 1, [n for n in range(shape[0]) if n != 1]
    for name in ("block_v", "block_k") + (("ext_v", "ext_k") if E else ()):
        x = dict(d, **{name: d[name].copy()})
        x[name][sick, 0, :, ::3] = bad
        got = to_f64(run(F, x, E))
        assert np.abs(got[others] - clean[others]).max() <= TOL, name
        assert not np.isfinite(got[sick]).all(), name


def test_an_infinite_value_stays_infinite(F, oracle):
    shape = SHAPES[0]
    print_case(test="f32_wide_infinite", shape=shape)
    d = make(shape)
    d["prefix_v"][-1, :, 5] = np.inf          # the last key, alone in its tile
    got, ref = to_f64(run(F, d, 0)), reference(oracle, d, 0)
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and not np.isnan(got).any()
    fin = np.isfinite(ref)
    assert np.abs(got[fin] - ref[fin]).max() <= TOL


# factors of V, Q and K (and of the scale, where the scores would not be those of the default one)
RANGES = [(1.0, 1.0, 1.0, 1.0), (1e-36, 1.0, 1.0, 1.0), (1e-37, 1.0, 1.0, 1.0), (1e-41, 1.0, 1.0, 1.0), (1e28, 1.0, 1.0, 1.0),
          (1e34, 1.0, 1.0, 1.0), (1.0, 1e-37, 1e37, 1.0), (1.0, 1e37, 1e-37, 1.0), (1.0, 1e-40, 1e37, 1e3), (1.0, 1e37, 1e-40, 1e3),
          (1.0, 2.0 ** -40, 1.0, 2.0 ** 40), (1.0, 1.0, 2.0 ** 40, 2.0 ** -40), (1.0, 1e22, 1e-34, 1e12)]


@pytest.mark.parametrize("factors", RANGES)
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1]])
def test_small_and_large_values_keep_their_bits(F, oracle, shape, factors):
    # Positive values, so nothing cancels: an average is off by 2^-24 for each of its weights' and its own few roundings, with
    # scores up to 5 off by 5 * 2^-24 a few times over, 2e-6 in all; below 2^-126 also by 2^-149 for the partial results and the
    # result.  The third part of 1e-36 would be below the smallest bf16 number, 3.4e38 has no nearest one.
    print_case(test="f32_wide_range", shape=shape, factors=factors)
    fv, fq, fk, fs = factors
    d, E, D = make(shape), shape[5], shape[6]
    with np.errstate(under="ignore"):
        for k in d:
            if k.endswith("_v"):
                d[k] = ((np.abs(d[k]) * 0.3 + 0.5) * np.float64(fv)).astype(np.float32)
            else:
                d[k] = (d[k] * np.float64(fq if k == "q" else fk)).astype(np.float32)
    scale = fs / np.sqrt(D)
    got = to_f64(run(F, d, E, scale=scale))
    ref = reference(oracle, d, E, scale=scale)
    err = np.abs(got - ref)
    print(f"relative error {(err / ref).max():.2e}, in norm {np.linalg.norm(err) / np.linalg.norm(ref):.2e}")
    assert (err <= 2e-6 * ref + 2 * 2.0 ** -149).all()


def test_a_value_without_a_nearest_bf16_number(F, oracle):
    shape = SHAPES[0]
    print_case(test="f32_wide_largest", shape=shape)
    d = make(shape)
    d["prefix_k"][700], d["prefix_v"][700, :, 3] = 0.0, np.float32(3.4e38)
    got, ref = to_f64(run(F, d, 0)), reference(oracle, d, 0)
    size = np.maximum(np.abs(ref), 1.0)
    assert np.isfinite(got).all() and (np.abs(got - ref) / size).max() <= TOL


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[5]])
def test_scores_far_below_zero(F, oracle, shape, causal):
    # every score a row sees is -2^86 and less, so that it overflows with the factor on the queries: the last prefix key is the
    # largest by 2^74, 2^44 after the scale, and holds the row
    print_case(test="f32_wide_far_below", shape=shape, causal=causal)
    d, E, L = make(shape), shape[5], shape[2]
    for k in ("q", "prefix_k", "block_k") + (("ext_k",) if E else ()):
        d[k][...] = 0.0
        d[k][..., 0] = 2.0 ** 44 if k == "q" else -2.0 ** 43
    d["prefix_k"][..., 0] = (-2.0 ** 42 - 2.0 ** 30 * np.arange(L)[::-1])[:, None]
    got = to_f64(run(F, d, E, scale=2.0 ** -30, causal_block=causal))
    ref = reference(oracle, d, E, scale=2.0 ** -30, causal_block=causal)
    assert np.array_equal(got, ref)


def test_calls_with_less_scratch_run_on_smaller_tiles(F, oracle):
    # 32-row tiles that are not cut need no scratch: such a call may bring none, too little or a misaligned one
    import ctypes as C

    import paper_2605_23163_amd.binding as b
    lib, ok, refused = F.load_library(), 0, 5

    def call(shape, splits=0):
        d = make(shape)
        t = {k: to_dev(v) for k, v in d.items()}
        args = [t[k] for k in ("q", "prefix_k", "prefix_v", "block_k", "block_v")]
        out = torch.empty_like(t["q"])
        p = b._attn_params(*args, None, out, None, splits)
        p.stream = torch.cuda.current_stream().cuda_stream
        return p, out, (d, t)

    def run_with(p, ptr, size):
        p.workspace, p.workspace_bytes = ptr, size
        return lib.fdd_block_attn(C.byref(p))

    shape = (7, 64, 190, 28, 4, 0, 64)
    print_case(test="f32_wide_less_scratch", shape=shape)
    p, out, keep = call(shape)
    need, ref = lib.fdd_block_attn_workspace(C.byref(p)), reference(oracle, keep[0], 0)
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    assert need > 0 and ws.data_ptr() % 256 == 0
    got = {}
    for name, ptr, size in (("none", None, 0), ("none, a size", None, need), ("short", ws.data_ptr(), need - 256),
                            ("misaligned", ws.data_ptr() + 16, need), ("enough", ws.data_ptr(), need)):
        out.fill_(7.0)
        assert run_with(p, ptr, size) == ok, name
        torch.cuda.synchronize()
        got[name] = out.clone()
        assert np.abs(to_f64(out) - ref).max() <= TOL, name
    assert torch.equal(got["none"], got["short"]) and torch.equal(got["none"], got["misaligned"])
    assert torch.equal(got["none"], got["none, a size"]) and not torch.equal(got["none"], got["enough"])

    # where the 32-row tiles are cut, what they need is still asked for
    shape = (2, 40, 3000, 28, 4, 0, 128)
    print_case(test="f32_wide_less_scratch", shape=shape)
    p, out, keep = call(shape)
    ref = reference(oracle, keep[0], 0)
    ws = torch.empty(lib.fdd_block_attn_workspace(C.byref(p)), dtype=torch.uint8, device="cuda")
    assert run_with(p, None, 0) == refused
    for splits in range(2, 12):
        forced, forced_out, keep2 = call(shape, splits)
        size = lib.fdd_block_attn_workspace(C.byref(forced))
        assert size < ws.numel()
        assert run_with(p, ws.data_ptr(), size - 256) == refused
        if run_with(p, ws.data_ptr(), size) == ok:
            break
    else:
        assert False, "no cut of 32-row tiles was enough"
    assert run_with(forced, ws.data_ptr(), size) == ok
    torch.cuda.synchronize()
    assert torch.equal(out, forced_out) and np.abs(to_f64(out) - ref).max() <= TOL
