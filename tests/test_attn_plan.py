"""How bf16 attention calls are cut (make_attn_plan): which keep one workgroup for each M-tile and need no scratch, and what calls with
less scratch than they are asked for run on.  Host arithmetic, checked without a GPU."""
import collections
import os

import pytest

from tests.test_f32_limits import ROOT, run_host

Plan = collections.namedtuple("Plan", "rows slots W pieces units prefix need small_need finished small_finished")

# N, B, L, Hq, Hkv, D, E: more private tiles than prefix tiles, cut inside the units booked for them, in every form of plan: (rows of
# an M-tile, ring slots, equal pieces or 0: ranges).  tests/test_gpu_attn_ring.py runs them.
DEALT = {(33, 1, 1408, 8, 8, 128, 1): (128, 2, 29), (33, 2, 64, 32, 8, 128, 130): (128, 4, 10), (33, 2, 64, 32, 8, 64, 130): (128, 4, 10),
         (77, 8, 40, 28, 4, 128, 37): (128, 4, 0), (33, 8, 64, 32, 8, 128, 130): (256, 4, 6), (96, 4, 64, 56, 8, 128, 37): (256, 4, 0),
         (96, 4, 64, 56, 8, 64, 37): (256, 4, 0)}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    from paper_2605_23163_amd import binding, build
    if not os.path.exists(binding.library_path()):
        build.build()
    lib = os.path.join(ROOT, "paper_2605_23163_amd")

    def run(shapes):
        """Plans of calls (N, B, L, Hq, Hkv, D[, E[, length of the list[, splits]]])."""
        args = [str(x) for s in shapes for x in (*s, 0, 0, 0)[:9]]
        out = run_host("attn_plan_main", tmp_path_factory.mktemp("plan"), ["-L" + lib, "-lfdd", "-Wl,-rpath," + lib], args)
        return [Plan(*map(int, line.split())) for line in out.splitlines()]
    return run


def test_short_prefixes_need_no_scratch(plans):
    # (two launches and an average rounded to bf16 on its way through the workspace would cost more than the shorter workgroups save)
    shapes = [(N, B, L, Hq, Hkv, D) for Hq, Hkv in ((28, 4), (14, 2)) for D in (64, 128) for B in (32, 64) for N in (1, 2, 4)
              for L in (0, 1, 32, 64)] + [(8, 32, L, 28, 4, 128) for L in (0, 32, 64)] + [(16, 32, 0, 28, 4, 128), (130, 1, 64, 2, 1, 128)]
    for shape, p in zip(shapes, plans(shapes)):
        assert p.need == 0 and p.pieces == 1, (shape, p)


def test_private_tiles_are_dealt_out_where_that_pays(plans):
    # One unit less in the longest of the 128-row pieces, two if there are more of them, three if the merge then needs another round;
    # more of them in pieces of 256 rows and in ranges, where fewer do not pay; pieces do not become ranges.  (pieces, units, prefix units)
    want = {(1, 32, 192, 28, 4, 128): (3, 5, 3), (4, 32, 1024, 28, 4, 128): (7, 20, 16), (33, 1, 1408, 8, 8, 128, 1): (29, 86, 22),
            (41, 32, 151, 14, 2, 64): (3, 6, 3), (9, 65, 585, 28, 4, 128, 65, 409): (5, 25, 10), (41, 32, 326, 28, 4, 128): (0, 8, 6),
            (1, 40, 3968, 28, 4, 128, 37): (17, 66, 62), (2, 20, 716, 8, 8, 128): (8, 16, 12), (1, 32, 2360, 32, 8, 128): (19, 38, 37),
            (1, 1, 943, 14, 2, 128): (8, 16, 15), (4, 32, 855, 28, 4, 128): (8, 16, 14), (8, 31, 365, 4, 1, 128): (4, 8, 6),
            (24, 65, 4864, 14, 2, 128, 130): (0, 94, 76), (14, 64, 75, 14, 2, 128): (2, 5, 2), (44, 40, 94, 14, 2, 128): (2, 5, 2)}
    got = plans(list(want))
    for (shape, w), p in zip(want.items(), got):
        assert (p.pieces, p.units, p.prefix) == w, (shape, p)


def test_every_form_of_plan_deals_private_tiles_out(plans):
    for (shape, form), p in zip(DEALT.items(), plans(list(DEALT))):
        m_tiles = shape[4] * -(-shape[0] * shape[1] * (shape[3] // shape[4]) // p.rows)
        booked, longest = p.units - p.prefix, -(-m_tiles * p.units // p.W)
        assert (p.rows, p.slots, p.pieces) == form and booked > longest > 2, (shape, p)


def test_ring_slots(plans):
    # four slots per operand for workgroups of 256 rows, and of 128 with 6 units or more where several M-tiles share a prefix and there are
    # no more workgroups than compute units (two of four slots do not fit one)
    want = {(1, 32, 2048, 28, 4, 128): 2, (8, 32, 4096, 28, 4, 128): 4, (2, 64, 14976, 8, 8, 128): 2, (1, 16, 14976, 28, 4, 128): 2,
            (3, 44, 64 * 4, 2, 1, 128, 0, 0, 1): 4, (3, 44, 64 * 3, 2, 1, 128, 0, 0, 1): 2, (8, 32, 1024, 28, 4, 64): 2, (8, 32, 2048, 28, 4, 64): 4,
            (8, 32, 4096, 28, 4, 128, 0, 0, 4): 4, (8, 32, 4096, 28, 4, 128, 0, 0, 5): 2, (8, 32, 4096, 28, 4, 128, 0, 0, 8): 2,
            (16, 64, 16384, 28, 4, 128): 4, (16, 64, 16384, 28, 4, 128, 0, 0, 4): 4}
    want.update({(1, 140, 64 * t, 20, 20, D): slots for D in (64, 128) for t, slots in ((29, 2), (30, 4))})
    for (shape, slots), p in zip(want.items(), plans(list(want))):
        assert p.slots == slots and (p.rows == 256) == (shape[0] == 16), (shape, p)


def test_rows_of_an_m_tile(plans):
    # 128 up to 9 units per compute unit of the plan with 256 rows at D = 128, 5 at D = 64 (64 KV heads of one M-tile, 2 units for the block)
    want = {(1, 2, 64 * t, 64, 64, D): rows for D, t, rows in ((64, 18, 128), (64, 19, 256), (128, 34, 128), (128, 35, 256))}
    for (shape, rows), p in zip(want.items(), plans(list(want))):
        assert p.rows == rows, (shape, p)


def test_ranges_that_end_with_their_m_tiles(plans):
    # dealt out, the ranges of these calls would be three to thirteen units shorter and end inside more M-tiles, whose averages are
    # rounded to bf16 on their way through the workspace
    shapes = [(32, 65, 72, 32, 8, 64, 65), (43, 40, 64, 28, 4, 64, 80), (25, 96, 575, 28, 4, 64), (36, 70, 284, 28, 4, 128, 70)]
    for shape, p in zip(shapes, plans(shapes)):
        assert p.pieces == 0 and p.finished == p.small_finished > 0, (shape, p)


def test_no_call_needs_scratch_or_cuts_m_tiles_for_the_sake_of_its_private_tiles(plans):
    import random
    rng = random.Random(4)
    shapes = []
    for _ in range(2000):
        Hq, Hkv = rng.choice(((28, 4), (14, 2), (32, 8), (16, 4), (8, 8), (4, 1), (64, 64)))
        N, B = int(2 ** rng.uniform(0, 8)), rng.choice((1, 3, 8, 32, 40, 65, 200))
        shapes.append((N, B, rng.choice((0, rng.randrange(400), int(2 ** rng.uniform(6, 15)))), Hq, Hkv, rng.choice((64, 128)),
                       rng.choice((0, 0, B, 37, 300)), rng.choice((0, 0, max(1, N * B // 3))), rng.choice((0, 0, 0, 3))))
    for shape, p in zip(shapes, plans(shapes)):
        assert (p.need == 0) == (p.small_need == 0) and p.finished >= p.small_finished, (shape, p)
