// C ABI entry points: host-side validation, planning and launches.
#include <cmath>
#include <cstdint>
#include <cstdarg>
#include <cstdio>
#include <numeric>

#include "fdd_internal.h"
#include <algorithm>

namespace fdd {
namespace {

thread_local char g_err[384] = "";
thread_local hipEvent_t g_ev_start = nullptr;
thread_local hipEvent_t g_ev_stop = nullptr;

}  // namespace

fdd_status set_error(fdd_status code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

namespace {

#define fail set_error

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

fdd_status check_attn_shape(const fdd_attn_params* p)
{
    if (!p) return fail(FDD_ERR_NULL, "fdd_block_attn: params is NULL");
    if (p->N <= 0 || p->B <= 0 || p->L < 0 || p->Hq <= 0 || p->Hkv <= 0 || p->D <= 0)
        return fail(FDD_ERR_SHAPE, "fdd_block_attn: N, B, Hq, Hkv, D must be positive and L >= 0 (got N=%d B=%d L=%d Hq=%d Hkv=%d D=%d)",
                    p->N, p->B, p->L, p->Hq, p->Hkv, p->D);
    if (p->Hq % p->Hkv) return fail(FDD_ERR_SHAPE, "fdd_block_attn: Hq=%d is not a multiple of Hkv=%d", p->Hq, p->Hkv);
    if (p->dtype != FDD_F32 && p->dtype != FDD_BF16) return fail(FDD_ERR_DTYPE, "fdd_block_attn: dtype %d is neither FDD_F32 nor FDD_BF16", p->dtype);
    if (p->D != 64 && p->D != 128) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_attn: head size D=%d not supported (64 or 128)", p->D);
    if (p->splits < 0 || p->splits > 64) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_attn: splits=%d outside [0, 64]", p->splits);
    if (p->flags & ~FDD_ATTN_CAUSAL_BLOCK) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_attn: unknown bits in flags (0x%x)", p->flags);
    // (every product below is bounded before the next factor is multiplied in: no 64-bit overflow for any int32 input)
    const long long nb = (long long)p->N * p->B;
    if (nb > (1ll << 30) || nb * (p->Hq / p->Hkv) > (1ll << 30) || nb * p->Hq > (1ll << 33))
        return fail(FDD_ERR_SHAPE, "fdd_block_attn: N*B*Hq too large");
    if ((long long)p->L * p->Hkv >= (1ll << 31) || (long long)p->L * p->Hkv * p->D * 4 >= (1ll << 31))
        return fail(FDD_ERR_SHAPE, "fdd_block_attn: prefix K (L*Hkv*D elements) must stay below 2 GiB");
    if (nb * p->Hkv >= (1ll << 32) || nb * p->Hkv * p->D * 4 >= (1ll << 32))
        return fail(FDD_ERR_SHAPE, "fdd_block_attn: block K (N*B*Hkv*D elements) must stay below 4 GiB");
    if (p->batch < 0 || p->batch > 65535 / p->Hkv) return fail(FDD_ERR_SHAPE, "fdd_block_attn: batch=%d outside [0, 65535 / Hkv]", p->batch);
    {
        // work units of the bf16 path: (KV head, 256-row M-tile, 64-key prefix tile)
        const long long mt = (nb * (p->Hq / p->Hkv) + 255) / 256;            // <= 2^22
        const long long tpu = (p->L + 63) / 64 + 64;          // prefix tiles plus the units booked for private tiles (bounded by 64 here)
        const long long heads = (long long)p->Hkv * (p->batch > 1 ? p->batch : 1);                 // <= 2^16
        if (heads * mt >= (1ll << 31) || heads * mt * tpu >= (1ll << 31)) return fail(FDD_ERR_SHAPE, "fdd_block_attn: batch*N*B*Hq*L too large");
    }
    if (std::isnan(p->scale) || std::isinf(p->scale)) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_attn: scale is not finite");
    if (p->n_q_positions < 0 || (long long)p->n_q_positions > (long long)p->N * p->B)
        return fail(FDD_ERR_SHAPE, "fdd_block_attn: n_q_positions=%d outside [0, N*B]", p->n_q_positions);
    if (p->batch > 1) {
        const long long es = p->dtype == FDD_BF16 ? 2 : 4;
        struct { const char* name; long long stride, need; } st[] = {
            {"q_batch_stride", p->q_batch_stride, (long long)p->N * p->B * p->Hq * p->D},
            {"out_batch_stride", p->out_batch_stride, (long long)p->N * p->B * p->Hq * p->D},
            {"block_batch_stride", p->block_batch_stride, (long long)p->N * p->B * p->Hkv * p->D},
            {"prefix_batch_stride", p->prefix_batch_stride, (long long)p->L * p->Hkv * p->D},
            {"ext_batch_stride", p->ext_batch_stride, p->E > 0 ? (long long)p->N * p->ext_capacity * p->Hkv * p->D : 0},
        };
        for (const auto& x : st)
            if (x.stride < x.need || (x.stride * es) % 16)
                return fail(FDD_ERR_SHAPE, "fdd_block_attn: %s=%lld must be at least %lld elements and a multiple of 16 bytes",
                            x.name, x.stride, x.need);
        if (p->prefix_v_packed && (p->packed_batch_stride % 256 ||
                                   p->packed_batch_stride < (size_t)p->Hkv * (p->L / 64) * 64 * p->D * 2))
            return fail(FDD_ERR_SHAPE, "fdd_block_attn: packed_batch_stride must be a multiple of 256 and hold one packed prefix V");
    }
    if (p->E < 0 || p->ext_capacity < 0 || p->E > p->ext_capacity)
        return fail(FDD_ERR_SHAPE, "fdd_block_attn: need 0 <= E <= ext_capacity (got E=%d, ext_capacity=%d)", p->E, p->ext_capacity);
    if ((long long)p->N * p->ext_capacity * p->Hkv * p->D * 4 >= (1ll << 32))
        return fail(FDD_ERR_SHAPE, "fdd_block_attn: extension K (N*ext_capacity*Hkv*D elements) must stay below 4 GiB");
    return FDD_OK;
}

}  // namespace

// Workgroups per row tile of the fp32 path, and the time that is expected of them.
//   32-row tiles (attn_f32_kernel): a round of workgroups takes ceil(tiles / (8 S)) tiles per wavefront, two wavefronts per
// SIMD at 36 D cycles a tile (32 D of them matrix pipe; 4.0 us per pair at D = 128 and 2.3 GHz), after about 4 us of start,
// first loads and LDS merge; S > 1 adds the merge kernel (about 4 us, and the partials' way to memory and back).
//   128-row tiles (attn_f32_wide_kernel): ceil(tiles / S) tiles of 32 keys a workgroup, 2.3 us each at D = 128 (2.0 with half of the
// compute units, which clock higher), 1.3 at D = 64, after 8 us of start, queries and first tiles; S > 1 adds 3 us and the partials.
// The smallest estimate wins, fewer splits on ties.
struct F32Cut {
    int splits;
    double us;
};
static F32Cut f32_cut(bool wide, long long row_tiles, long long tiles, int D, int s_min)
{
    const double tile_us = wide ? (D == 128 ? 2.3 : 1.3) : 2.0 * 36 * D / 2300.0, start_us = wide ? 8.0 : 4.0, merge_us = wide ? 3.0 : 4.0;
    const int sharers = wide ? 1 : kF32Waves;                    // of a workgroup's keys
    const double partial_us = (wide ? (double)kF32WideRowTile * D * 4.0 / 4e6 : (double)kF32RowTile * D * 8.0 / 4e6);
    F32Cut best = {1, HUGE_VAL};                                 // (kept where s_min is above the most splits)
    for (int s = s_min; s <= 64 && (s == s_min || (long long)(s - 1) * sharers < tiles); ++s) {
        const long long rounds = (row_tiles * s + kNumCU - 1) / kNumCU;
        const long long per = (tiles + (long long)s * sharers - 1) / ((long long)s * sharers);
        double us = (double)rounds * ((double)per * tile_us + start_us);
        if (s > 1) us += merge_us + (double)row_tiles * s * partial_us;
        if (us < best.us) best = {s, us};
        if (row_tiles * s >= 4 * kNumCU) break;      // more rounds gain nothing
    }
    return best;
}

bool make_attn_plan(const fdd_attn_params& p, AttnPlan* plan, bool ample)
{
    AttnPlan pl;
    pl.slots = 0;
    pl.G = p.Hq / p.Hkv;
    pl.R = (p.n_q_positions > 0 ? p.n_q_positions : p.N * p.B) * pl.G;
    pl.key_tile = p.dtype == FDD_BF16 ? 64 : 16;
    pl.TP = (p.L + pl.key_tile - 1) / pl.key_tile;
    const int batch = p.batch > 1 ? p.batch : 1;
    long long NM;
    auto set_rows = [&](int rows) {
        pl.mtile_rows = rows;
        pl.MT = (pl.R + rows - 1) / rows;
        NM = (long long)p.Hkv * batch * pl.MT;
    };
    bool partials;
    // Cuts for M-tiles of `rows` rows, with the private tiles of an M-tile at the workgroup that ends its units or (`deal`) wherever
    // their units lie.  `longest`: units of the longest workgroup; `booked_all`: dealing them out would be the same cut.
    long long longest;
    bool booked_all;
    auto cut_units = [&](int rows, bool deal) {
        set_rows(rows);
        // The private tiles of an M-tile (extension and block of every rollout its rows belong to) go through the masked path at
        // about 1.8 times the cost of a pipelined prefix tile.  They are booked as `wt` extra units behind the M-tile's prefix tiles
        // (up to 64) and go to the workgroups that these units go to.
        // (with a list of query positions a rollout contributes fewer rows: its average share stands in for B)
        const long long BG = p.n_q_positions > 0 ? std::max(1ll, (long long)p.n_q_positions * pl.G / p.N) : (long long)p.B * pl.G;
        const long long span_lo = (pl.mtile_rows + BG - 1) / BG;                 // rollouts an M-tile spans at least
        const long long span = span_lo + ((pl.mtile_rows % BG) != 0 && BG < (long long)pl.R ? 1 : 0);
        const long long per_rollout = (p.E + pl.key_tile - 1) / pl.key_tile + (p.B + pl.key_tile - 1) / pl.key_tile;
        const long long private_tiles = (span < p.N ? span : p.N) * per_rollout;
        const long long cost = std::max((private_tiles * 9 + 4) / 5, 1ll);
        long long wt = std::min(cost, 64ll);
        auto pieces_for = [&](long long tpu) {
            // equal pieces per M-tile, of two units or more (one of them may have less); the fewest pieces that reach the shortest critical path
            long long smax = NM > 0 ? kNumCU / NM : 0;
            if (smax > (tpu + 1) / 2) smax = (tpu + 1) / 2;
            if (smax < 1) return 0ll;
            const long long crit = (tpu + smax - 1) / smax;
            long long sbest = smax;
            while (sbest > 1 && (tpu + (sbest - 1) - 1) / (sbest - 1) == crit) --sbest;
            return sbest;
        };
        long long w;
        pl.uniform = 0;
        if (p.splits > 0) {
            if (wt > 2) wt = 2;
            pl.TPU = pl.TP + (int)wt;
            pl.uniform = p.splits < pl.TPU ? p.splits : pl.TPU;
            w = NM * pl.uniform;
        } else {
            // Equal pieces per M-tile when that fills at least 4/5 of the compute
            // units: the workgroups of an XCD then walk the same K/V tiles in step
            // and the prefix is fetched from HBM once.  So are calls of fewer than two units per compute unit, which
            // leave some idle either way: a range that crosses into the next M-tile does two set-ups and two partial
            // results for its two units (us per call, ranges / pieces: N=1, L=64 13.5/9.3; N=8, L=64 17.3/11.7; N=1, L=700
            // 13.5/12.6).  Otherwise equal contiguous unit ranges (stream-K).
            long long s = pieces_for(pl.TP + wt);
            if (s >= 1 && !deal) {
                const long long per = (pl.TP + wt) / s;       // a piece must not lie inside the booked units only
                if (wt > per) wt = per > 1 ? per : 1;
                s = pieces_for(pl.TP + wt);
            }
            pl.TPU = pl.TP + (int)wt;
            long long smax = NM > 0 ? kNumCU / NM : 0;
            if (smax > (pl.TPU + 1) / 2) smax = (pl.TPU + 1) / 2;
            if (s >= 1 && (NM * smax * 5 >= (long long)kNumCU * 4 || NM * pl.TPU < 2 * kNumCU)) {
                w = NM * s;
                pl.uniform = (int)s;
            } else {
                // (ranges are short here: book at most two units, so that no range lies inside them only)
                if (wt > 2 && !deal) wt = 2;
                pl.TPU = pl.TP + (int)wt;
                const long long U = NM * pl.TPU;
                w = U < 2 * kNumCU ? (U + 1) / 2 : kNumCU;
                if (w > U) w = U;
                if (w <= NM && NM <= kNumCU) {   // nothing to gain from cutting M-tiles: one workgroup each
                    w = NM;
                    pl.uniform = 1;
                }
            }
        }
        pl.U = NM * pl.TPU;
        pl.W = (int)w;
        pl.splits = 0;
        const long long upw = pl.U / pl.W;
        pl.max_seg = pl.uniform > 0 ? pl.uniform : (int)((pl.TPU + upw - 1) / upw) + 1;
        partials = pl.W != NM;
        // (What is not booked comes on top, with every M-tile that ends in a range; of the rollouts that an M-tile can span: the
        // first row's place in its rollout is a multiple of what row counts of both have in common.)
        longest = (pl.U + w - 1) / w;
        if (!deal) {
            const long long most = p.n_q_positions > 0 ? span : (BG - std::gcd(BG, (long long)rows) + rows - 1) / BG + 1;
            const long long units = (std::min(most, (long long)p.N) * per_rollout * 9 + 4) / 5;
            longest += std::max(0ll, units - wt) * ((longest + pl.TPU - 1) / pl.TPU);
        }
        booked_all = wt == std::min(cost, 64ll);
    };
    // Private tiles are dealt out where that shortens the longest workgroup by more than the further segments cost: pieces of 128 rows by
    // a unit, one more if there are more of them than two and than before, and one more if the merge kernel then needs another round of
    // loads; four for pieces of 256, whose wavefronts pass over the private tiles of
    // other rollouts, so that these cost less than they are booked with; three for ranges, some of which then end in one more
    // M-tile.  Never if equal pieces would become ranges.  us per call, one place / dealt, in brackets the units of the longest workgroup and
    // the pieces, Hq = 28, Hkv = 4, D = 128 unless said:
    //   pieces of 128 rows, dealt: N=1, B=32, L=192 [3/2, 2/3] 9.9/8.5; N=8, L=128 [4/2, 2/3] 10.4/10.7; N=1, B=40, L=3968, E=37 [5/4, 17/17]
    //   14.6/13.7; Hkv = Hq = 8, N=2, B=20, L=716 [4/2, 7/8] 10.6/9.9; D = 64: Hq = 32, Hkv = 8, B=72, L=1197 [5/3, 7/8] 12.2/10.0; Hq = 14,
    //   Hkv = 2, N=8, B=40, L=3008, E=40 [9/8] 15.3/14.4; many rollouts, Hq = Hkv = 8, N=33, B=1, L=1408, E=1 [119/3] 93.4/12.9;
    //   in one place: Hq = 32, Hkv = 8, N=1, B=32, L=2360 [3/2, 19/20] 12.2/13.0; another round of the merge: Hq = 14, Hkv = 2, B=1, L=943
    //   [3/2, 8/9] 9.7/10.3, N=4, B=32, L=855 [4/2, 8/9] 13.3/13.9, Hq = 4, Hkv = 1, N=8, B=31, L=365 [4/2, 4/6] 10.5/11.6, but Hq = 32,
    //   Hkv = 8, N=2, B=1, L=384 [4/2, 4/5] 9.3/8.7;
    //   478 drawn calls: 451 dealt (1.36 in the geometric mean, ten of them slower by more than 2 %), 27 in one place (0.99);
    //   pieces of 256: Hq = 14, Hkv = 2, N=41, B=32, L=151, D = 64 [5/3] 11.9/12.5; half of the positions of N=31, B=32, L=24 [6/3] 17.2/18.4;
    //   N=50, B=8, L=108 [11/3] 18.2/18.4; N=9, B=65, L=585, E=65, listed [13/5] 20.2/18.4; N=7, B=70, L=320, Hq = 32, Hkv = 8, E=140, listed
    //   [24/7] 26.0/21.7;
    //   ranges: N=55, B=32, L=64 [7/6] 25.6/28.2; N=41, B=32, L=326 [9/7] 28.5/29.4; Hq = 32, Hkv = 8, N=15, B=70, L=100 [9/6] 29.4/27.8;
    //   Hq = 32, Hkv = 8, N=41, B=64, L=1152, E=128 [34/31] 82.4/79.2;
    //   Hq = 14, Hkv = 2, N=24, B=65, L=4864, E=130 [43/32] 74.5/64.4; a gain of one unit or two
    //   0.97 (17 drawn calls), of three or four 1.04 (11);
    //   pieces to ranges: Hq = 14, Hkv = 2, N=14, B=64, L=75 13.4/15.1; N=44, B=40, L=94 20.5/23.9.
    auto cut_bf16 = [&](int rows, bool may_deal) {
        cut_units(rows, false);
        if (!may_deal || booked_all) return;
        const long long whole = longest;
        const int pieces = pl.uniform;
        cut_units(rows, true);
        long long least = 3;
        if (pieces > 0) {
            const long long chunks = (long long)p.Hkv * batch * pl.R * (p.D / 8);
            const MergeCut a = merge_cut(chunks, pieces), b = merge_cut(chunks, pl.uniform);
            least = rows == 256 ? 4 : 1 + (pieces > 2 && pl.uniform > pieces) + (b.rounds > a.rounds);
        }
        if (longest + least > whole || (pieces > 0 && pl.uniform == 0)) cut_units(rows, false);
    };
    auto cut_rows = [&](bool may_deal) {
        cut_bf16(256, may_deal);
        // M-tiles of 128 rows (workgroups of 4 wavefronts, one per SIMD) while the call is short: alone in a compute unit such a
        // workgroup takes 0.68 us a tile where one of 8 takes 1.09 (D = 128), starts on fewer tiles, and its segments are half as
        // large; long calls fetch K and V twice as often.  Up to 9 units per compute unit of the 256-row plan, D = 64 5; not where only the
        // larger tiles cut into equal pieces that fill the chip.  By the figures below 128 rows would be 1 to 6 % ahead up to 11 units at
        // D = 128, and within 3 % either way up to 8 at D = 64.  The lines stand lower because these few shapes are all that was measured
        // beyond them, and because the tests of the 256-row kernels have their shapes there (9.2 to 9.9 units): they would have to grow
        // first.  us per call,
        // prefixes from memory (30 calls in rotation), 256 / 128 rows, Hq = 28, Hkv = 4, B = 32, in brackets the units per compute unit:
        //   D = 128, V laid out: N=8, L=2048 [3.9] 19.8/17.1; L=4096 [7.7] 25.6/23.6; N=4, L=8192 [8.4] 25.8/24.2; N=2, L=18000 [8.9]
        //   27.3/26.2; N=12, L=3000 [9.1] 27.4/25.8; N=4, L=9500 [9.7] 27.6/26.3; N=8, L=6000 [10.9] 31.0/30.8; N=16, L=4096 [15]
        //   37.2/38.0;
        //   D = 128, plain V: N=1, L=2048 12.5/10.4; N=8, L=512 14.6/12.4; N=8, L=4096 25.7/23.8; N=12, L=3000 27.6/25.9; N=16, L=2048
        //   [8.3] 26.2/24.8; no equal pieces of 128 rows: N=24, L=1024 [7.2] 24.8/26.7;
        //   D = 64: N=1, L=2048 9.5/8.3; N=8, L=2048 [3.9] 13.8/12.5, plain 13.9/12.8; N=1, L=20000 [4.9] 15.3/14.4; N=8, L=4096 [7.7]
        //   17.2/16.7, plain 17.3/17.5; N=8, L=6000 [10.9] 20.3/22.2; N=16, L=4096 [15], plain 24.9/27.5.
        const int uniform256 = pl.uniform;
        if (pl.U <= (p.D == 128 ? 9 : 5) * (long long)kNumCU) {
            cut_bf16(128, may_deal);
            if (pl.uniform == 0 && (uniform256 > 0 || NM > kNumCU)) cut_bf16(256, may_deal);
        }
    };
    // Stacked rows, over all KV heads, of M-tiles that several workgroups work on.  (Ranges, 256 at most, are walked without a division
    // each: for both plans of such a call 2 us of the host's, 3.2 with divisions; the call takes 17 and more on the GPU.)
    auto shared_rows = [&](const AttnPlan& a) -> long long {
        if (a.uniform > 0) return a.uniform == 1 ? 0 : (long long)p.Hkv * batch * a.R;
        const int last_rows = a.R - (a.MT - 1) * a.mtile_rows, rem = (int)(a.U % a.W);
        const long long base = a.U / a.W;
        const int tiles = (int)(base / a.TPU), units = (int)(base % a.TPU), tiles_in_head = tiles % a.MT;
        long long n = 0, shared = -1, m = 0;     // the last shared M-tile; the one that range w begins in
        int mt = 0, u = 0;                       // its place in its KV head, the unit in it
        for (int w = 1; w < a.W; ++w) {
            u += units + (w <= rem ? 1 : 0);
            const int over = u >= a.TPU ? 1 : 0;
            u -= over ? a.TPU : 0;
            m += tiles + over;
            mt += tiles_in_head + over;
            mt -= mt >= a.MT ? a.MT : 0;
            const bool cut = (u != 0) & (m != shared);
            const int rows = mt == a.MT - 1 ? last_rows : a.mtile_rows;
            n += cut ? rows : 0;
            shared = cut ? m : shared;
        }
        return n;
    };
    if (p.dtype == FDD_BF16) {
        // Calls that have one workgroup for each M-tile with its private tiles in one place stay so: their sums are in fp32 up to the one
        // rounding of the output (off from 64 bits by 2.0e-3 in norm, with averages that go through the workspace in bf16 2.6e-3), and
        // they need neither scratch nor a merge.  With short prefixes the second launch costs what the shorter workgroups save: us per
        // call, one workgroup / dealt, Hq = 28, Hkv = 4, B = 32: L=64, N=2 9.7/8.9, N=8 10.0/10.9; L=0, N=4 8.5/9.2, N=16 9.2/12.3; D = 64,
        // Hq = 14, Hkv = 2, L=64, N=4 7.4/8.2.  (With many rollouts an M-tile it would not: B=1, L=8, N=10 18.4/10.5.)
        // Nor do ranges that end with their M-tiles move into them: as many rows as before have fp32 sums.  (One call in 120 of a sweep;
        // us per call, one place / dealt: N=27, B=96, L=91, Hq=32, Hkv=8 38.6/44.7; D = 64: N=45, B=96, L=74, Hq=32, Hkv=8 33.8/37.3, N=43,
        // B=40, L=64, E=80 22.5/24.4, N=32, B=65, L=72, Hq=32, Hkv=8, E=65 33.4/30.7; N=36, B=70, L=284, E=70 49.9/48.5, off from 64 bits by
        // 2.47e-3/2.66e-3.)
        cut_rows(false);
        if (ample && p.splits == 0 && partials && !booked_all) {
            const AttnPlan one_place = pl;
            cut_rows(true);
            const bool other = pl.TPU != one_place.TPU || pl.mtile_rows != one_place.mtile_rows;
            if (other && shared_rows(pl) > shared_rows(one_place)) cut_rows(false);
        }
        // Ring slots per operand: four hide more of the memory's latency, two start earlier, with fewer requests in flight, do better
        // where nearly every request goes to memory (one M-tile per KV head), and leave room for a second workgroup on a compute unit
        // (D = 128: 80 KB of LDS against 144), which a call of more workgroups than compute units has.  us per call, prefixes from
        // memory, 4 / 2 slots, in brackets the units per workgroup:
        //   several M-tiles, D = 128, N=1, L=2048 [2] 10.4/10.1; N=3, L=1279, Hq=32, Hkv=8 [2] 12.9/12.5; N=1, L=6518 [3.2] 13.6/13.1;
        //   B=70, L=3008, Hq=32, Hkv=8 [4.4] 16.1/15.7; N=2, L=6239 [6.1] 16.3/16.1; B=40, L=14464, Hq=16 [7.1] 17.2/18.2; N=2, L=18304,
        //   Hq=16 [8.9] 20.6/21.9; N=3, B=8, L=24960 [12] 21.3/24.4; N=8, L=4096, V laid out [16] 23.6/28.7; D = 64, N=8, L=1024 [4]
        //   10.2/10.1, L=2048 [8] 12.5/13.2, N=1, L=20000 [10] 14.4/16.1;
        //   one M-tile, D = 128, plain / V laid out: Hq = Hkv = 8, N=2, B=64, L=8000 [4.0] 19.9/17.3, 18.7/16.1, L=14976 [7.4] 24.5/23.0,
        //   21.7/20.8, B=8, L=8000 13.9/14.1, 13.3/13.6, L=14976 19.1/20.1, 17.0/16.7; Hq = 28, Hkv = 4, N=1, B=16, L=14976 [3.7] 19.5/16.1,
        //   18.1/15.2, L=30000 [7.4] 24.1/22.9, 20.4/20.0; Hq = Hkv = 16, N=1, B=32, L=2000 [2.1] 11.4/10.7, L=8000 [7.9] 19.6/20.5,
        //   17.2/18.2; D = 64 within 4 % of each other (longer ones, from 9 and 5 units on, have 256 rows);
        //   more workgroups than compute units (`splits`): N=8, L=4096 in 5 pieces 37.1/30.1, 6 34.0/27.4, 8 32.4/26.3; N=16, L=2000 in 4
        //   31.1/26.8; D = 64, Hq = 14, Hkv = 2, N=16, L=2000 in 5 16.6/16.0.
        pl.slots = pl.mtile_rows == 128 && (pl.MT == 1 || pl.U < 6ll * pl.W || pl.W > kNumCU) ? 2 : 4;
    } else {
        auto cut_f32 = [&](int rows, int key_tile) {
            set_rows(rows);
            pl.key_tile = key_tile;
            pl.TP = (p.L + key_tile - 1) / key_tile;
            const long long rows_per_rollout = std::max(1ll, (long long)pl.R / p.N);
            const long long span = std::min<long long>(p.N, (rows + rows_per_rollout - 1) / rows_per_rollout + 1);
            return pl.TP + span * ((p.E + key_tile - 1) / key_tile + (p.B + key_tile - 1) / key_tile);
        };
        // Products on the bf16 pipe (128-row tiles) where they are expected to be faster and the keys are cut at least once more:
        // a row's sum is rounded twice per 32 keys of a workgroup there, four times per 4 keys of a wavefront here, and with that
        // many pieces the error against 64 bits in norm was 0.53 to 0.86 of that of 32-row tiles in the 33 of 60 drawn calls that
        // take them (N to 33, L = 200 to 16384, six head counts, both D, deviations 0.09 to 2).  us per call, replayed, 32-row tiles / 128-row
        // tiles (pieces): D = 128, Hq = 28, Hkv = 4, B = 32: N=1, L=2048 22.1 / 19.3 (22); N=1, L=16384 71.0 / 51.5 (31); N=2, L=1024
        // 24.2 / 20.6 (12); N=4, L=4096 76.5 / 49.2 (9); N=8, L=4096 135.1 / 85.5 (4); N=16, L=4096 268 / 157 (2); D = 64: N=8, L=4096
        // 73.7 / 51.5 (4); N=5, B=40, L=5003, Hq=14, Hkv=2 47.8 / 29.9 (11).
        long long tiles = cut_f32(kF32RowTile, 16);
        int s = p.splits;
        if (s == 0) {
            const F32Cut narrow = f32_cut(false, NM, tiles, p.D, 1);
            s = narrow.splits;
            const long long wide_tiles = cut_f32(kF32WideRowTile, kF32WideKeyTile);
            const F32Cut wide = f32_cut(true, NM, wide_tiles, p.D, narrow.splits + 1);
            // (short calls that are cut take 2 to 5 us more than the estimate for 32-row tiles says)
            // (up to a GiB of partials: beyond it the chip is full many times over, and the narrow tiles need none)
            const bool fits = NM * wide.splits * (kF32WideRowTile * p.D * 4ll) <= (1ll << 30);
            // (a larger scale multiplies what those products lose of keys below 2^-110; a smaller one gives weight to scores that
            // overflow with their factor on Q)
            const bool usual_scale = !(p.scale > 0.f) || (p.scale >= 0x1p-30f && p.scale <= 0x1p10f);
            if (ample && usual_scale && fits && wide_tiles >= 2 * wide.splits && wide.us < narrow.us + (narrow.splits > 1 ? 3.0 : 0.0)) {
                s = wide.splits;
                tiles = wide_tiles;
            } else {
                tiles = cut_f32(kF32RowTile, 16);
            }
        }
        if (s > tiles) s = (int)tiles;
        if (s < 1) s = 1;
        // Tiles of 16 rows, cut alike, where twice the workgroups still find a compute unit each: half of the matrix work for
        // every wavefront, the same sums per row.  us per call, replayed, 32 rows / 16 rows (workgroups of 32 rows): D = 64, Hq = 4,
        // Hkv = 1, N=1, B=8, L=256 10.4 / 7.1 (1), L=20000 16.4 / 12.6 (53); D = 64, Hq = 28, Hkv = 4, N=1, B=64, L=100 8.8 / 6.5 (56); D = 128,
        // Hq = 28, Hkv = 4, N=1, B=32, L=256 15.3 / 11.9 (84), N=2, B=32, L=128 16.3 / 11.0 (56); Hq = 8, Hkv = 8, B=8, L=1000 13.0 / 11.0 (64).
        // With more workgroups a second round costs more than the halves save: D = 128, Hq = 28, Hkv = 4, N=8, B=32, L=40 12.5 / 15.5
        // (224), N=9, L=64 12.8 / 16.3 (252), Hq = 4, Hkv = 1, N=2, B=31, L=10559 25.6 / 30.7 (208); at D = 64 it is 10 % either way.
        if (pl.mtile_rows == kF32RowTile && 2 * NM * s <= kNumCU) cut_f32(kF32FewRowTile, 16);
        pl.TPU = pl.TP > 0 ? pl.TP : 1;
        pl.U = NM * pl.TPU;
        pl.splits = s;
        pl.W = 0;
        pl.uniform = 0;
        pl.max_seg = s;
        partials = s > 1;
    }
    if (partials) {
        const size_t prow = (size_t)NM * pl.max_seg * pl.mtile_rows;
        pl.ws_o_bytes = (prow * p.D * (p.dtype == FDD_BF16 ? 2 : sizeof(float)) + 255) & ~(size_t)255;
        pl.ws_ml_bytes = (prow * 2 * sizeof(float) + 255) & ~(size_t)255;
    } else {
        pl.ws_o_bytes = 0;
        pl.ws_ml_bytes = 0;
    }
    // The kernel reads V repacked when the caller brings it that way (fdd_prefix_pack, once per prefix).
    // Repacking inside the call is a launch and a pass over V of its own, and the kernel that reads V as it
    // lies (transposing LDS reads) is 2 to 5 % slower: measured, the in-call pass pays from about
    // the size of N=16, B=64, L=16384 on (28 M-tiles x 256 tiles per KV head), and costs 3..5 us below it.
    pl.ws_vt_bytes = 0;
    pl.packed = p.dtype == FDD_BF16 && p.L >= pl.key_tile && (p.prefix_v_packed || (long long)pl.MT * pl.TP >= 8192);
    if (pl.packed && !p.prefix_v_packed)
        pl.ws_vt_bytes = (((size_t)p.Hkv * batch * (p.L / pl.key_tile) * pl.key_tile * p.D * 2) + 255) & ~(size_t)255;
    *plan = pl;
    return true;
}

}  // namespace fdd

using namespace fdd;

static fdd_status check_unmask_shape(const fdd_unmask_params* p, const char* fn)
{
    if (!p) return fail(FDD_ERR_NULL, "%s: params is NULL", fn);
    if (p->N <= 0 || p->B <= 0 || p->V <= 0) return fail(FDD_ERR_SHAPE, "%s: N, B, V must be positive (got N=%d B=%d V=%lld)", fn, p->N, p->B, (long long)p->V);
    if (p->V >= (1ll << 31)) return fail(FDD_ERR_SHAPE, "%s: V must be below 2^31", fn);
    if ((long long)p->N * p->B > (1ll << 24)) return fail(FDD_ERR_SHAPE, "%s: N*B too large", fn);
    if (p->dtype != FDD_F32 && p->dtype != FDD_BF16) return fail(FDD_ERR_DTYPE, "%s: dtype %d is neither FDD_F32 nor FDD_BF16", fn, p->dtype);
    if (std::isnan(p->tau)) return fail(FDD_ERR_UNSUPPORTED, "%s: tau is NaN", fn);
    return FDD_OK;
}


// shape, type and pointer checks shared by the entry points of the unmask step (everything but the workspace)
fdd_status fdd::check_unmask_args(const fdd_unmask_params* p, const char* fn)
{
    fdd_status st = check_unmask_shape(p, fn);
    if (st != FDD_OK) return st;
    if (!p->logits || !p->mask || !p->tokens || !p->confidences)
        return fail(FDD_ERR_NULL, "%s: logits, mask, tokens and confidences must not be NULL", fn);
    if (!aligned16(p->logits)) return fail(FDD_ERR_UNSUPPORTED, "%s: logits must be 16-byte aligned", fn);
    if (p->refresh_table_k || p->refresh_table_v || p->refresh_block_k || p->refresh_block_v) {
        if (!p->refresh_table_k || !p->refresh_table_v || !p->refresh_block_k || !p->refresh_block_v)
            return fail(FDD_ERR_NULL, "%s: the K/V refresh needs refresh_table_k, refresh_table_v, refresh_block_k and refresh_block_v", fn);
        if (p->refresh_Hkv <= 0 || p->refresh_D <= 0 || p->refresh_T <= 0)
            return fail(FDD_ERR_SHAPE, "%s: refresh_Hkv, refresh_D, refresh_T must be positive", fn);
        if (p->refresh_dtype != FDD_F32 && p->refresh_dtype != FDD_BF16)
            return fail(FDD_ERR_DTYPE, "%s: refresh_dtype %d is neither FDD_F32 nor FDD_BF16", fn, p->refresh_dtype);
        const long long row = (long long)p->refresh_Hkv * p->refresh_D * (p->refresh_dtype == FDD_BF16 ? 2 : 4);
        if (row % 16 || row > (1ll << 24)) return fail(FDD_ERR_UNSUPPORTED, "%s: a refreshed K/V row must be a multiple of 16 bytes (and at most 16 MiB)", fn);
        if (!aligned16(p->refresh_table_k) || !aligned16(p->refresh_table_v) || !aligned16(p->refresh_block_k) || !aligned16(p->refresh_block_v))
            return fail(FDD_ERR_UNSUPPORTED, "%s: refresh tables and block K/V must be 16-byte aligned", fn);
    }
    return FDD_OK;
}

extern "C" {

size_t fdd_block_attn_workspace(const fdd_attn_params* p)
{
    if (check_attn_shape(p) != FDD_OK) return 0;
    AttnPlan plan;
    make_attn_plan(*p, &plan);
    size_t partials = plan.ws_o_bytes + plan.ws_ml_bytes;
    if (p->dtype == FDD_BF16) {      // enough for the same call with V laid out and with V as it lies, which may be cut differently
        fdd_attn_params other = *p;
        other.prefix_v_packed = p->prefix_v_packed ? nullptr : p;      // (only whether it is set counts)
        AttnPlan o;
        make_attn_plan(other, &o);
        partials = std::max(partials, o.ws_o_bytes + o.ws_ml_bytes);
    }
    return partials + plan.ws_vt_bytes;
}

fdd_status fdd_block_attn(const fdd_attn_params* p)
{
    fdd_status st = check_attn_shape(p);
    if (st != FDD_OK) return st;
    if (!p->q || !p->block_k || !p->block_v || !p->out) return fail(FDD_ERR_NULL, "fdd_block_attn: q, block_k, block_v and out must not be NULL");
    if (p->L > 0 && (!p->prefix_k || !p->prefix_v)) return fail(FDD_ERR_NULL, "fdd_block_attn: prefix_k / prefix_v is NULL with L=%d", p->L);
    if (p->E > 0 && (!p->ext_k || !p->ext_v)) return fail(FDD_ERR_NULL, "fdd_block_attn: ext_k / ext_v is NULL with E=%d", p->E);
    if (p->n_q_positions > 0 && !p->q_positions) return fail(FDD_ERR_NULL, "fdd_block_attn: q_positions is NULL with n_q_positions=%d", p->n_q_positions);
    if (p->n_q_positions > 0 && (reinterpret_cast<uintptr_t>(p->q_positions) & 3u)) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_attn: q_positions must be 4-byte aligned");
    const void* ptrs[] = {p->q, p->prefix_k, p->prefix_v, p->block_k, p->block_v, p->out, p->prefix_v_packed,
                          p->E > 0 ? p->ext_k : nullptr, p->E > 0 ? p->ext_v : nullptr};
    for (const void* x : ptrs)
        if (x && !aligned16(x)) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_attn: data pointers must be 16-byte aligned");
    if (p->out == p->q) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_attn: out must not alias q");
    AttnPlan plan;
    make_attn_plan(*p, &plan);
    size_t need = plan.ws_o_bytes + plan.ws_ml_bytes + plan.ws_vt_bytes;
    const size_t given = p->workspace && (reinterpret_cast<uintptr_t>(p->workspace) & 255u) == 0 ? p->workspace_bytes : 0;
    if (need >= given + 256 && (p->dtype == FDD_BF16 || plan.mtile_rows == kF32WideRowTile)) {
        // A call that brings less than the query says, which asks for the fastest plan, but what the plan without 128-row tiles (fp32,
        // which always leave partial results) or with an M-tile's private tiles in one place (bf16: fewer segments, often one)
        // needs, runs on that.  (Sizes come in steps of 256 bytes: one that misses the query's by less is a slip of the
        // caller's and refused, as it always was.)
        AttnPlan small;
        make_attn_plan(*p, &small, false);
        const size_t small_need = small.ws_o_bytes + small.ws_ml_bytes + small.ws_vt_bytes;
        if (small_need <= given) {
            plan = small;
            need = small_need;
        }
    }
    if (need > 0) {
        if (!p->workspace) return fail(FDD_ERR_WORKSPACE, "fdd_block_attn: workspace is NULL, %zu bytes needed", need);
        if (reinterpret_cast<uintptr_t>(p->workspace) & 255u) return fail(FDD_ERR_WORKSPACE, "fdd_block_attn: workspace must be 256-byte aligned");
        if (p->workspace_bytes < need) return fail(FDD_ERR_WORKSPACE, "fdd_block_attn: workspace has %zu bytes, %zu needed", p->workspace_bytes, need);
    }
    const float scale = p->scale > 0.f ? p->scale : 1.f / std::sqrt((float)p->D);
    hipStream_t s = static_cast<hipStream_t>(p->stream);
    const bool timed = g_ev_start && g_ev_stop;
    hipError_t e;
    if (p->dtype == FDD_BF16) {
        e = launch_attn_bf16(*p, plan, scale, s, timed ? g_ev_start : nullptr);
    } else {
        if (timed && hipEventRecord(g_ev_start, s) != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_block_attn: cannot record the start event");
        e = launch_attn_f32(*p, plan, scale, s);
    }
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_block_attn: launch failed: %s", hipGetErrorString(e));
    if (timed && hipEventRecord(g_ev_stop, s) != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_block_attn: cannot record the stop event");
    if (plan.ws_o_bytes > 0) {
        e = p->dtype == FDD_BF16 ? launch_attn_merge_bf16(*p, plan, scale, s) : launch_attn_combine(*p, plan, scale, s);
        if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_block_attn: merge launch failed: %s", hipGetErrorString(e));
    }
    return FDD_OK;
}

size_t fdd_prefix_pack_bytes(int32_t L, int32_t Hkv, int32_t D, int32_t dtype)
{
    if (dtype != FDD_BF16 || L < 64 || Hkv <= 0 || (D != 64 && D != 128)) return 0;
    return (((size_t)Hkv * (L / 64) * 64 * D * 2) + 255) & ~(size_t)255;
}

fdd_status fdd_prefix_pack(const void* prefix_v, int32_t L, int32_t Hkv, int32_t D, int32_t dtype, void* packed,
                           size_t packed_bytes, void* stream)
{
    if (dtype != FDD_BF16) return fail(FDD_ERR_DTYPE, "fdd_prefix_pack: only FDD_BF16 prefixes are packed");
    if (L < 0 || Hkv <= 0) return fail(FDD_ERR_SHAPE, "fdd_prefix_pack: L must be >= 0 and Hkv positive");
    if (D != 64 && D != 128) return fail(FDD_ERR_UNSUPPORTED, "fdd_prefix_pack: head size D=%d not supported (64 or 128)", D);
    if ((long long)L * Hkv >= (1ll << 31) || (long long)L * Hkv * D * 4 >= (1ll << 31))
        return fail(FDD_ERR_SHAPE, "fdd_prefix_pack: prefix V (L*Hkv*D elements) must stay below 2 GiB");
    const size_t need = fdd_prefix_pack_bytes(L, Hkv, D, dtype);
    if (need == 0) return FDD_OK;
    if (!prefix_v || !packed) return fail(FDD_ERR_NULL, "fdd_prefix_pack: prefix_v and packed must not be NULL");
    if (!aligned16(prefix_v) || !aligned16(packed)) return fail(FDD_ERR_UNSUPPORTED, "fdd_prefix_pack: pointers must be 16-byte aligned");
    if (packed_bytes < need) return fail(FDD_ERR_WORKSPACE, "fdd_prefix_pack: packed buffer has %zu bytes, %zu needed", packed_bytes, need);
    hipError_t e = launch_prefix_pack(prefix_v, L, Hkv, D, packed, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_prefix_pack: launch failed: %s", hipGetErrorString(e));
    return FDD_OK;
}

size_t fdd_unmask_workspace(const fdd_unmask_params* p)
{
    if (check_unmask_shape(p, "fdd_unmask_workspace") != FDD_OK) return 0;
    UnmaskPlan plan;
    make_unmask_plan(*p, &plan);
    return plan.ws_bytes;
}

fdd_status fdd_unmask_step(const fdd_unmask_params* p)
{
    fdd_status st = check_unmask_args(p, "fdd_unmask_step");
    if (st != FDD_OK) return st;
    UnmaskPlan plan;
    make_unmask_plan(*p, &plan);
    if (!p->workspace) return fail(FDD_ERR_WORKSPACE, "fdd_unmask_step: workspace is NULL, %zu bytes needed", plan.ws_bytes);
    if (reinterpret_cast<uintptr_t>(p->workspace) & 255u) return fail(FDD_ERR_WORKSPACE, "fdd_unmask_step: workspace must be 256-byte aligned");
    if (p->workspace_bytes < plan.ws_bytes) return fail(FDD_ERR_WORKSPACE, "fdd_unmask_step: workspace has %zu bytes, %zu needed", p->workspace_bytes, plan.ws_bytes);
    hipError_t e = launch_unmask(*p, plan, static_cast<hipStream_t>(p->stream));
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_unmask_step: launch failed: %s", hipGetErrorString(e));
    return FDD_OK;
}

size_t fdd_verify_workspace(const fdd_verify_params* p)
{
    UnmaskPlan plan;
    if (!p || p->V >= (1ll << 31) || (long long)p->N * p->B > (1ll << 24) ||
        (p->dtype != FDD_F32 && p->dtype != FDD_BF16) || !make_vocab_plan(p->N, p->B, p->V, p->dtype, !(p->temperature > 0.f), &plan))
        return 0;
    return plan.ws_bytes;
}

fdd_status fdd_verify_step(const fdd_verify_params* p)
{
    if (!p) return fail(FDD_ERR_NULL, "fdd_verify_step: params is NULL");
    if (p->N <= 0 || p->B <= 0 || p->V <= 0) return fail(FDD_ERR_SHAPE, "fdd_verify_step: N, B, V must be positive (got N=%d B=%d V=%lld)", p->N, p->B, (long long)p->V);
    if (p->V >= (1ll << 31)) return fail(FDD_ERR_SHAPE, "fdd_verify_step: V must be below 2^31");
    if ((long long)p->N * p->B > (1ll << 24)) return fail(FDD_ERR_SHAPE, "fdd_verify_step: N*B too large");
    if (p->dtype != FDD_F32 && p->dtype != FDD_BF16) return fail(FDD_ERR_DTYPE, "fdd_verify_step: dtype %d is neither FDD_F32 nor FDD_BF16", p->dtype);
    if (!(p->temperature >= 0.f) || std::isinf(p->temperature))
        return fail(FDD_ERR_UNSUPPORTED, "fdd_verify_step: temperature must be 0 (greedy) or positive and finite");
    if (!p->ar_logits || !p->draft || !p->mask || !p->tokens)
        return fail(FDD_ERR_NULL, "fdd_verify_step: ar_logits, draft, mask and tokens must not be NULL");
    if (!aligned16(p->ar_logits)) return fail(FDD_ERR_UNSUPPORTED, "fdd_verify_step: ar_logits must be 16-byte aligned");
    UnmaskPlan plan;
    make_vocab_plan(p->N, p->B, p->V, p->dtype, !(p->temperature > 0.f), &plan);
    if (!p->workspace) return fail(FDD_ERR_WORKSPACE, "fdd_verify_step: workspace is NULL, %zu bytes needed", plan.ws_bytes);
    if (reinterpret_cast<uintptr_t>(p->workspace) & 255u) return fail(FDD_ERR_WORKSPACE, "fdd_verify_step: workspace must be 256-byte aligned");
    if (p->workspace_bytes < plan.ws_bytes) return fail(FDD_ERR_WORKSPACE, "fdd_verify_step: workspace has %zu bytes, %zu needed", p->workspace_bytes, plan.ws_bytes);
    hipError_t e = launch_verify(*p, plan, static_cast<hipStream_t>(p->stream));
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_verify_step: launch failed: %s", hipGetErrorString(e));
    return FDD_OK;
}

fdd_status fdd_fork_block(int32_t N, size_t bytes, const void* src, void* dst, void* stream)
{
    if (!src || !dst) return fail(FDD_ERR_NULL, "fdd_fork_block: src and dst must not be NULL");
    if (N <= 0 || bytes == 0) return fail(FDD_ERR_SHAPE, "fdd_fork_block: N and bytes must be positive");
    if (bytes % 4 || (reinterpret_cast<uintptr_t>(src) & 3u) || (reinterpret_cast<uintptr_t>(dst) & 3u))
        return fail(FDD_ERR_UNSUPPORTED, "fdd_fork_block: bytes and pointers must be multiples of 4");
    if (bytes > (SIZE_MAX >> 1) / (size_t)N) return fail(FDD_ERR_SHAPE, "fdd_fork_block: N*bytes too large");
    const uintptr_t s0 = reinterpret_cast<uintptr_t>(src), d0 = reinterpret_cast<uintptr_t>(dst);
    const uintptr_t total = (uintptr_t)N * bytes;
    if (s0 > UINTPTR_MAX - bytes || d0 > UINTPTR_MAX - total) return fail(FDD_ERR_SHAPE, "fdd_fork_block: address range wraps around");
    if (s0 < d0 + total && d0 < s0 + bytes) return fail(FDD_ERR_UNSUPPORTED, "fdd_fork_block: src and dst overlap");
    hipError_t e = launch_fork_block(N, bytes, src, dst, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_fork_block: launch failed: %s", hipGetErrorString(e));
    return FDD_OK;
}

fdd_status fdd_block_commit(const fdd_commit_params* p)
{
    if (!p) return fail(FDD_ERR_NULL, "fdd_block_commit: params is NULL");
    if (p->N <= 0 || p->B <= 0 || p->Hkv <= 0 || p->D <= 0 || p->E < 0 || p->ext_capacity <= 0)
        return fail(FDD_ERR_SHAPE, "fdd_block_commit: N, B, Hkv, D, ext_capacity must be positive and E >= 0");
    if ((long long)p->E + p->B > p->ext_capacity)
        return fail(FDD_ERR_SHAPE, "fdd_block_commit: E + B = %lld exceeds ext_capacity = %d", (long long)p->E + p->B, p->ext_capacity);
    if (p->dtype != FDD_F32 && p->dtype != FDD_BF16) return fail(FDD_ERR_DTYPE, "fdd_block_commit: dtype %d is neither FDD_F32 nor FDD_BF16", p->dtype);
    if (p->reserved != 0) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_commit: reserved field must be 0");
    if (!p->block_k || !p->block_v || !p->ext_k || !p->ext_v) return fail(FDD_ERR_NULL, "fdd_block_commit: block_k, block_v, ext_k and ext_v must not be NULL");
    const size_t es = p->dtype == FDD_BF16 ? 2 : 4;
    if (((size_t)p->Hkv * p->D * es) % 16) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_commit: a K/V row must be a multiple of 16 bytes");
    const void* ptrs[] = {p->block_k, p->block_v, p->ext_k, p->ext_v};
    for (const void* x : ptrs)
        if (!aligned16(x)) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_commit: pointers must be 16-byte aligned");
    hipError_t e = launch_block_commit(*p, static_cast<hipStream_t>(p->stream));
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_block_commit: launch failed: %s", hipGetErrorString(e));
    return FDD_OK;
}

fdd_status fdd_traj_mean(int32_t N, int32_t P, const float* traj, float* out, void* stream)
{
    if (!traj || !out) return fail(FDD_ERR_NULL, "fdd_traj_mean: traj and out must not be NULL");
    if (N <= 0 || P <= 0) return fail(FDD_ERR_SHAPE, "fdd_traj_mean: N and P must be positive (got N=%d P=%d)", N, P);
    if ((reinterpret_cast<uintptr_t>(traj) & 3u) || (reinterpret_cast<uintptr_t>(out) & 3u))
        return fail(FDD_ERR_UNSUPPORTED, "fdd_traj_mean: pointers must be 4-byte aligned");
    hipError_t e = launch_traj_mean(N, P, traj, out, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_traj_mean: launch failed: %s", hipGetErrorString(e));
    return FDD_OK;
}

fdd_status fdd_block_kv_update(const fdd_kv_update_params* p)
{
    if (!p) return fail(FDD_ERR_NULL, "fdd_block_kv_update: params is NULL");
    if (p->N <= 0 || p->B <= 0 || p->Hkv <= 0 || p->D <= 0 || p->T <= 0)
        return fail(FDD_ERR_SHAPE, "fdd_block_kv_update: N, B, Hkv, D, T must be positive");
    if (p->dtype != FDD_F32 && p->dtype != FDD_BF16) return fail(FDD_ERR_DTYPE, "fdd_block_kv_update: dtype %d is neither FDD_F32 nor FDD_BF16", p->dtype);
    if (!p->tokens || !p->committed || !p->table_k || !p->table_v || !p->block_k || !p->block_v)
        return fail(FDD_ERR_NULL, "fdd_block_kv_update: all pointers must be non-NULL");
    const size_t es = p->dtype == FDD_BF16 ? 2 : 4;
    if (((size_t)p->Hkv * p->D * es) % 16) return fail(FDD_ERR_UNSUPPORTED, "fdd_block_kv_update: a K/V row (Hkv*D elements) must be a multiple of 16 bytes");
    if (!aligned16(p->table_k) || !aligned16(p->table_v) || !aligned16(p->block_k) || !aligned16(p->block_v))
        return fail(FDD_ERR_UNSUPPORTED, "fdd_block_kv_update: tables and block K/V must be 16-byte aligned");
    hipError_t e = launch_kv_update(*p, static_cast<hipStream_t>(p->stream));
    if (e != hipSuccess) return fail(FDD_ERR_LAUNCH, "fdd_block_kv_update: launch failed: %s", hipGetErrorString(e));
    return FDD_OK;
}

fdd_status fdd_profile_attn_events(void* start, void* stop)
{
    if ((start == nullptr) != (stop == nullptr)) return fail(FDD_ERR_NULL, "fdd_profile_attn_events: pass two events or two NULLs");
    g_ev_start = static_cast<hipEvent_t>(start);
    g_ev_stop = static_cast<hipEvent_t>(stop);
    return FDD_OK;
}

const char* fdd_last_error(void) { return g_err; }

int fdd_version(void) { return 100; }

}  // extern "C"
