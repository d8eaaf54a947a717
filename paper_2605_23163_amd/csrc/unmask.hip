// Confidence-threshold unmasking of one block per rollout.
//
// One iteration of "iteratively unmasks value positions" (paper, "Section
// Diffusion (SD)"): masked, non-scaffold positions are the only ones touched
// (Eq. 2; visible tokens stay fixed).  For each such position the row of V
// logits is reduced to (arg max, largest softmax probability); a position
// commits when that probability reaches tau, and a block that would commit
// nothing commits its most confident eligible position.
//
// Two kernels, or in very small calls one (block_unmask_small):
//   vocab_reduce  streams the logits rows of eligible positions once.  A row
//                 is cut into `vsplits` pieces so that a few hundred rows
//                 still fill 256 CUs; each piece is reduced by one workgroup
//                 to (max, lowest arg max, sum exp(x - max)) with a one-pass
//                 running-maximum sum.  (value, index) pairs are ordered by
//                 value descending then index ascending through every
//                 in-thread, cross-lane and cross-wave stage, so ties of
//                 stored values (frequent in bf16) always resolve to the
//                 lowest id.  Workgroups of non-eligible rows exit at once
//                 and read nothing.
//   vocab_sample  the sampled verifier's sibling of vocab_reduce: the value
//                 reduced is the Gumbel-max key of every vocabulary entry
//                 (a Philox-4x32-10 word per entry, two polynomial log2, one
//                 fused multiply-add), worked out only where a cheap upper bound
//                 of it reaches the largest key met so far.
//   block_select  one workgroup per rollout: merges the pieces of each
//                 position in a fixed order (sum finished in fp64), applies
//                 the tau test and the forced single commit, and writes
//                 tokens / mask / confidences.
#include <algorithm>
#include <type_traits>

#include "fdd_internal.h"

namespace fdd {
namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr int PIECE_KB = 64;         // a row is cut into pieces of at least this size ...
constexpr int PIECE_KB_ARGMAX = 32;  // ... and of this size in the pass that takes no sums (measured: 8 pieces of a
                                     // 297 KB row are 1.5 us per call faster there than 4, and 1..2 us slower with the sums)
constexpr int PIECE_KB_FEW = 16;     // a call of few rows takes up to 8 pieces a row, of at least this size and up to
constexpr int kFewPieces = 1024;     // this number in all.  us per call with a fork, replayed, unmask / sampled verifier:
                                     // V = 152064 bf16, N=4, B=32, 4 pieces 13.5/28.0, 8 13.1/20.5, 16 14.9/25.9; N=1, 1 piece
                                     // 19.4/43.8, 4 11.2/19.7, 8 11.2/14.8, 16 12.6/17.0; V = 50001, 200 rows, 1 piece 12.5/28.8,
                                     // 5 11.5/21.5, 8 12.6/24.5; V = 32768, 128 rows, 1 10.4/17.4, 4 8.7/13.4, 8 9.8/12.7.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Partial {
    float m;
    int32_t arg;
    float s;
    int32_t pad;
};

struct Args {
    const void* logits;
    const uint8_t* scaffold;
    uint8_t* mask;
    int32_t* tokens;
    float* conf;
    int32_t* n_unmasked;
    uint8_t* committed;
    Partial* ws;
    const int32_t* draft;   // verify pass only
    // K/V refresh of the committed positions (unmask step only): row (token mod T) of the tables, or no refresh
    const u32x4* rf_tk;
    const u32x4* rf_tv;
    u32x4* rf_bk;
    u32x4* rf_bv;
    int rf_T, rf_row_vecs;  // table rows; 16-byte pieces per K/V row (0: no refresh)
    int N, B, vsplits;
    int units;              // workgroups of a vocabulary pass: N B pieces
    int pieces;             // pieces per row: vsplits, or twice as many whose (key, id) pairs share a record
    int per;                // vocabulary entries per piece (the last pieces of a row may be shorter or empty)
    FastDiv dVs;            // division by pieces
    long long V;
    float tau;
    float c;                // sampled verifier: log2(e) / temperature
    uint32_t seed_lo, seed_hi;
};

struct Run {
    float m;      // running maximum
    int idx;      // lowest index attaining it
    float s;      // sum of 2^((x - m) log2 e) over what was seen
};

// A thread's running sum takes its terms as 2^(x c - fl(m c)), c = log2 e, with one fused
// multiply-add each.  fl(m c) is off from m c by up to half an ulp, which scales every term
// by the same 2^(m c - fl(m c)): harmless as long as the whole sum is relative to the same
// fl(m c).  So a new maximum rescales the sum by 2^(fl(m_old c) - fl(m_new c)), the
// difference of the rounded products, and the common factor is taken out once, by
// `settle`, before sums of different threads meet.
struct ThreadRun {
    Run r;
    float mc;     // fl(r.m * log2 e)
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Reductions over the 64 lanes, result in every lane: DPP moves within rows of 16 (pairs, quads, then mirrors, which
// pair up what the steps before have made uniform), gfx950 lane swaps across rows.  A shuffle through LDS takes 60
// cycles and more per step, and a workgroup of the vocabulary pass ended with 18 of them in six dependent steps (pass
// with sums 41.0 -> 39.1 us, without 36.6 -> 34.1 at N=16, B=64, V=152064; 16.5 -> 15.6 and 13.9 -> 13.0 at N=8, B=32).
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t x, Op op)
{
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true));    // quad_perm 1 0 3 2
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true));    // quad_perm 2 3 0 1
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true));   // row_half_mirror
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true));   // row_mirror
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = op(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return op(b[0], b[1]);
}
__device__ __forceinline__ float wave_max(float x)
{
    return __uint_as_float(wave_reduce(__float_as_uint(x), [](uint32_t p, uint32_t q) {
        return __float_as_uint(fmaxf(__uint_as_float(p), __uint_as_float(q)));
    }));
}
__device__ __forceinline__ float wave_sum(float x)
{
    return __uint_as_float(wave_reduce(__float_as_uint(x), [](uint32_t p, uint32_t q) {
        return __float_as_uint(__uint_as_float(p) + __uint_as_float(q));
    }));
}
__device__ __forceinline__ int wave_min(int x)
{
    return (int)wave_reduce((uint32_t)x, [](uint32_t p, uint32_t q) { return (uint32_t)min((int)p, (int)q); });
}

// `b` is merged into `a`; on equal maxima the lower index wins.
__device__ __forceinline__ void merge(Run& a, const Run& b)
{
    const bool take_b = (b.m > a.m) || (b.m == a.m && b.idx < a.idx);
    const float M = fmaxf(a.m, b.m);
    const float sa = (a.m == M) ? a.s : a.s * fast_exp2((a.m - M) * LOG2E);
    const float sb = (b.m == M) ? b.s : b.s * fast_exp2((b.m - M) * LOG2E);
    a.s = sa + sb;
    a.m = M;
    if (take_b) a.idx = b.idx;
}

// SUM = false: only (max, arg max) are kept (the greedy verifier needs no probabilities)
template <int VEC, bool SUM>
__device__ __forceinline__ void absorb(ThreadRun& t, const float (&x)[VEC], int v0)
{
    Run& r = t.r;
    float cm = x[0];
#pragma unroll
    for (int j = 1; j < VEC; ++j) cm = fmaxf(cm, x[j]);
    if (cm > r.m) {
        // this thread walks the row in ascending order, so a strictly larger
        // value is the only way its arg max can move
        if (SUM) {
            const float mc_new = cm * LOG2E;
            r.s *= fast_exp2(t.mc - mc_new);      // (-inf - finite at the start: the sum is still 0)
            t.mc = mc_new;
        }
        r.m = cm;
        int first = VEC - 1;
#pragma unroll
        for (int j = VEC - 2; j >= 0; --j) first = (x[j] == cm) ? j : first;
        r.idx = v0 + first;
    }
    if (!SUM) return;
    // (a thread that has only met -inf so far takes its terms against 0: 2^(-inf) = 0, never inf - inf)
    const float mc = (t.mc == -INFINITY) ? 0.f : t.mc;
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc += fast_exp2(fmaf(x[j], LOG2E, -mc));
    r.s += acc;
}

// the sum as taken against m itself (see ThreadRun)
__device__ __forceinline__ Run settle(const ThreadRun& t)
{
    Run r = t.r;
    if (r.m != -INFINITY) r.s *= fast_exp2(-fmaf(r.m, LOG2E, -t.mc));
    return r;
}

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// Which (row, piece) a workgroup of a vocabulary pass takes: workgroup u the piece u mod vsplits of the (u / vsplits)-th
// ELIGIBLE row, so that the live workgroups come first and together, and the dispatcher deals them out evenly.  (With
// row = u / vsplits, workgroups of rows that are not eligible left at once, but not before they had been dealt a place:
// a scaffold pattern, which all rollouts share, left some compute units with several live workgroups and others with
// none.)  Every wavefront counts for itself: a lane looks at 16 positions, ballots give the counts before it, no LDS and no
// barrier; mask and scaffold are read in one round trip.  Returns -1 past the last eligible row.  Up to LIVE_ROWS rows, which a
// wavefront reads at once; `deal_to_eligible` has the calls it pays for, the others go by `unit_of_workgroup` below.
constexpr int LIVE_ROWS = 1024;
__device__ __forceinline__ int eligible_row(const uint8_t* mask, const uint8_t* scaffold, int rows, int target)
{
    const int lane = thread_id_x() & 63;
    const int at = lane * 16, p = min(at, rows - 16), drop = at - p;         // (drop: positions the lanes below have already)
    const uint8_t* const sc = scaffold ? scaffold : mask;
    const uint32_t use_sc = scaffold ? ~0u : 0u;
    uint32_t m[4], s[4];
    __builtin_memcpy(m, mask + p, 16);    // (positions start anywhere: the loads need no alignment)
    __builtin_memcpy(s, sc + p, 16);
    uint32_t z[4];                        // 0x80 in the bytes of eligible positions
    int c = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t t = (m[w] ^ 0x01010101u) | (s[w] & use_sc);                    // zero bytes: mask 1, no scaffold
        const uint32_t e = ~(((t & 0x7f7f7f7fu) + 0x7f7f7f7fu) | t | 0x7f7f7f7fu);
        z[w] = drop >= 4 * w + 4 ? 0u : drop <= 4 * w ? e : e & (~0u << (8 * (drop - 4 * w)));
        c += __builtin_popcount(z[w]);
    }
    int before = 0;                       // eligible positions of the lanes below
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        const uint64_t has = __builtin_amdgcn_ballot_w64((c >> b) & 1);
        before += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u)) << b;
    }
    const uint64_t here = __builtin_amdgcn_ballot_w64(before <= target && target < before + c);
    if (here == 0) return -1;
    const int l = __builtin_ctzll(here);
    int left = target - __builtin_amdgcn_readlane(before, l);
    const int first = __builtin_amdgcn_readlane(p, l);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)z[w], l);
        const int n = __builtin_popcount(e);
        if (left < n) {
            for (; left > 0; --left) e &= e - 1;
            return first + 4 * w + (__builtin_ctz(e) >> 3);
        }
        left -= n;
    }
    return -1;
}

// Other calls: each group of 8 consecutive launch indices (workgroups are dealt to the 8 XCDs round-robin) is
// rotated, by an amount that changes from group to group, from 8 groups to the next 8 and from 64 to the next, so that a
// scaffold pattern that repeats from rollout to rollout does not load the XCDs unequally.
__device__ __forceinline__ unsigned unit_of_workgroup(unsigned n_units)
{
    const unsigned u = wg_id_x(), g = u >> 3;
    if ((g << 3) + 8u > n_units) return u;           // a last, incomplete group stays as it is
    return (g << 3) + ((u + g + (g >> 3) + (g >> 6) + (g >> 9)) & 7u);
}

// the row and the piece of this workgroup; false: nothing to do.  COMPACT: workgroups are dealt to eligible rows only (a
// template argument: with the choice inside one kernel every workgroup waited for one more round of its arguments, 5 % of a
// call of 131072 short rows)
template <bool COMPACT>
__device__ __forceinline__ bool unit_of(const Args& a, int* row, int* piece)
{
    if (COMPACT) {
        const int u = (int)wg_id_x(), t = fast_div(u, a.dVs);
        *piece = u - t * a.pieces;
        *row = eligible_row(a.mask, a.scaffold, a.N * a.B, t);
        return *row >= 0;
    }
    const int u = (int)unit_of_workgroup((unsigned)a.units);
    *row = fast_div(u, a.dVs);
    *piece = u - *row * a.pieces;
    return a.mask[*row] == 1 && !(a.scaffold && a.scaffold[*row]);
}

// T = uint16_t (bf16 bits) or float; SUM = false leaves (max, arg max) only and a sum of 0
template <typename T, bool SUM, int THREADS, bool COMPACT>
__global__ __launch_bounds__(THREADS) void vocab_reduce_kernel(Args a)
{
    constexpr int VEC = 16 / sizeof(T);
    constexpr int UNROLL = THREADS == 512 ? 5 : 6;      // 16-byte loads in flight per thread
    int row, piece;
    if (!unit_of<COMPACT>(a, &row, &piece)) return;
    const long long v_lo = (long long)piece * a.per;
    const long long v_hi = min(a.V, v_lo + a.per);
    const T* base = static_cast<const T*>(a.logits) + (size_t)row * (size_t)a.V;
    const int tid = thread_id_x();

    ThreadRun tr;
    tr.r.m = -INFINITY;
    tr.r.idx = 0x7fffffff;
    tr.r.s = 0.f;
    tr.mc = -INFINITY;

    if (v_lo < v_hi) {
        // leading elements up to the first 16-byte boundary, then whole
        // vectors, then the remainder; each thread visits ascending indices
        const size_t e_lo = (size_t)row * (size_t)a.V + (size_t)v_lo;
        long long head = (long long)((VEC - (e_lo % VEC)) % VEC);
        if (head > v_hi - v_lo) head = v_hi - v_lo;
        const long long body0 = v_lo + head;
        const long long nvec = (v_hi - body0) / VEC;
        const long long tail0 = body0 + nvec * VEC;

        if (tid < head) {
            float x[1] = {sizeof(T) == 2 ? bf16_to_f32(((const uint16_t*)base)[v_lo + tid]) : ((const float*)base)[v_lo + tid]};
            absorb<1, SUM>(tr, x, (int)(v_lo + tid));
        }
        const u32x4* vp = reinterpret_cast<const u32x4*>(base + body0);
        auto widen = [&](const u32x4& raw, float (&x)[VEC]) {
            if (sizeof(T) == 2) {
                const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[2 * j] = __uint_as_float(w[j] << 16);
                    x[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
                }
            } else {
                x[0] = __uint_as_float(raw.x);
                x[1] = __uint_as_float(raw.y);
                x[2] = __uint_as_float(raw.z);
                x[3] = __uint_as_float(raw.w);
            }
        };
        // UNROLL independent 16-byte loads in flight per thread, absorbed in ascending order
        long long i = tid;
        for (; i + (UNROLL - 1) * THREADS < nvec; i += UNROLL * THREADS) {
            u32x4 raw[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) raw[u] = __builtin_nontemporal_load(vp + i + u * THREADS);
            // all of them are requested before the first is waited for (left to itself the scheduler waits
            // for the first after two requests and only then issues the rest: two latencies per group)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                float x[VEC];
                widen(raw[u], x);
                absorb<VEC, SUM>(tr, x, (int)(body0 + (i + u * THREADS) * VEC));
            }
        }
        if (i < nvec) {
            // the ragged last group: its loads are requested together as well
            u32x4 raw[UNROLL - 1];
#pragma unroll
            for (int u = 0; u < UNROLL - 1; ++u)
                if (i + u * THREADS < nvec) raw[u] = __builtin_nontemporal_load(vp + i + u * THREADS);
#pragma unroll
            for (int u = 0; u < UNROLL - 1; ++u) {
                if (i + u * THREADS < nvec) {
                    float x[VEC];
                    widen(raw[u], x);
                    absorb<VEC, SUM>(tr, x, (int)(body0 + (i + u * THREADS) * VEC));
                }
            }
        }
        const long long ntail = v_hi - tail0;
        if (tid < ntail) {
            float x[1] = {sizeof(T) == 2 ? bf16_to_f32(((const uint16_t*)base)[tail0 + tid]) : ((const float*)base)[tail0 + tid]};
            // tail indices are larger than anything this thread saw before
            absorb<1, SUM>(tr, x, (int)(tail0 + tid));
        }
    }

    // wavefront reduction, then across the wavefronts through LDS
    Run r = SUM ? settle(tr) : tr.r;
    const float m_wave = wave_max(r.m);
    if (SUM) r.s = wave_sum(r.m == m_wave ? r.s : r.s * fast_exp2((r.m - m_wave) * LOG2E));
    r.idx = wave_min(r.m == m_wave ? r.idx : 0x7fffffff);
    r.m = m_wave;
    __shared__ Run part[THREADS / 64];
    if ((tid & 63) == 0) part[tid >> 6] = r;
    __syncthreads();
    if (tid == 0) {
        Run t = part[0];
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) merge(t, part[w]);
        Partial p;
        p.m = t.m;
        p.arg = t.idx;
        p.s = t.s;
        p.pad = 0;
        a.ws[(size_t)row * a.vsplits + piece] = p;
    }
}

// ---- sampled verifier ------------------------------------------------------
// The arithmetic below is the definition of the sampler (see fdd_verify_step
// in the public header): every operation is written out as one exactly
// rounded binary32 operation and must not be contracted or reassociated.

// Philox-4x32 with 10 rounds (Salmon, Moraes, Dror, Shaw: "Parallel random
// numbers: as easy as 1, 2, 3", SC'11): counter (c0, c1, 0, 0), key (k0, k1).
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
    uint32_t c2 = 0u, c3 = 0u;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint32_t hi0 = mul_hi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = mul_hi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// log2 of a positive normal float: x = m 2^e, m in [1/sqrt 2, sqrt 2), e + f P(f) with f = m - 1
__device__ __forceinline__ float flog2_def(float x)
{
    const uint32_t bits = __float_as_uint(x);
    int e = (int)((bits >> 23) & 255u) - 127;
    float m = __uint_as_float((bits & 0x7fffffu) | 0x3f800000u);
    if (m > 1.41421354f) { m = __fmul_rn(m, 0.5f); e += 1; }
    const float f = __fsub_rn(m, 1.0f);
    float p = 0.12614846229553223f;
    p = __fmaf_rn(p, f, -0.20742103457450867f);
    p = __fmaf_rn(p, f, 0.21566985547542572f);
    p = __fmaf_rn(p, f, -0.23892034590244293f);
    p = __fmaf_rn(p, f, 0.2879183292388916f);
    p = __fmaf_rn(p, f, -0.36070483922958374f);
    p = __fmaf_rn(p, f, 0.48091059923171997f);
    p = __fmaf_rn(p, f, -0.7213473320007324f);
    p = __fmaf_rn(p, f, 1.4426950216293335f);
    return __fmaf_rn(f, p, (float)e);
}

__device__ __forceinline__ float gumbel_key(float x, float c, uint32_t r)
{
    const float u = __fmul_rn(__fadd_rn((float)(r >> 9), 0.5f), 1.1920928955078125e-07f);
    const float a = -flog2_def(u);
    const float g = -flog2_def(a);
    return __fmaf_rn(x, c, g);
}

struct Best {
    float k;
    int idx;
};
__device__ __forceinline__ void take(Best& a, float k, int idx)
{
    if (k > a.k || (k == a.k && idx < a.idx)) { a.k = k; a.idx = idx; }
}

// Upper bound of the noise of generator word r, for a fifth of its cost.  With w = 2^23 - 1/2 - (r >> 9) the uniform is
// u = 1 - w 2^-23, and -log2 u >= (1 - u) log2 e, so the noise -log2(-log2 u) is at most 23 - log2(log2 e) - log2 w;
// log2 w in turn is at least exponent + mantissa fraction, i.e. the bits of the float w read as a fixed-point number.
// The slack added to the constant (1e-3) is a hundred times what flog2_def and the roundings here are off by; the bound
// exceeds the noise by less than 0.092 for u > 0.99, where most winners lie, by 0.16 above 7/8, 0.48 above 1/2 and more below.  fma is monotonic, so
// fma(x, c, noise_bound(r)) is never below the entry's key.
constexpr float NOISE_C = 149.47223f;          // 23 + 127 - log2(log2 e) + 1e-3
constexpr float NOISE_MAX = 23.47223f;         // the bound at its largest (r >> 9 = 2^23 - 1)
__device__ __forceinline__ float noise_bound(uint32_t r)
{
    const float w = (float)(~r >> 9) + 0.5f;
    return fmaf((float)__float_as_uint(w), -1.1920928955078125e-07f, NOISE_C);
}

constexpr int VTHREADS = 256;
constexpr int VUNROLL = 5;       // sampled verifier: 16-byte loads in flight per thread

// Same work split as vocab_reduce; leaves (largest key, lowest id attaining it) per piece.
// Bound by the vector ALUs: the definition of a key takes 64 operations per entry (20 of them the generator, 40 the two
// logarithms), but only entries that can still win need theirs.  The key of the drafted token (the verifier mostly
// agrees with it) and any key a thread of the workgroup has worked out in full are lower bounds of the row's largest: an
// entry whose own upper bound lies below them is dropped, first by its logit alone (no generator word drawn: rows with a
// clear winner end here), then with the bound above in place of the logarithms.  What is left (a few entries per
// wavefront) is worked out as defined, and the row's winner is never dropped, so the verifier's token is the same bit for
// bit.
// Measured, bf16, 70 % of the rows live, V = 152064 (in brackets every entry worked out in full): N=8, B=32 27 us (87) with
// a clear winner in 4 of 5 rows, 37 (87) with none; N=16, B=64 68 (231) and 115 (230); N=5, B=40, V=50001 21 (211: rows
// that start inside a generator block took a block per entry).  Without a winner the generator's 32 x 32 bit products
// are what is left.
template <typename T, bool COMPACT>
__global__ __launch_bounds__(VTHREADS) void vocab_sample_kernel(Args a)
{
    constexpr int VEC = 16 / sizeof(T);
    constexpr int NW = VEC + 4;               // generator words that cover VEC entries starting anywhere
    int row, piece;
    if (!unit_of<COMPACT>(a, &row, &piece)) return;
    const long long v_lo = (long long)piece * a.per;
    const long long v_hi = min(a.V, v_lo + a.per);
    const T* base = static_cast<const T*>(a.logits) + (size_t)row * (size_t)a.V;
    const int tid = thread_id_x();
    Best r;
    r.k = -INFINITY;
    r.idx = 0x7fffffff;

    // largest key worked out by any thread of the workgroup so far, as an integer of the same order
    __shared__ int s_floor;
    auto ordered = [](float k) { const int b = __float_as_int(k); return b ^ ((b >> 31) & 0x7fffffff); };
    auto from_ordered = [](int o) { return __int_as_float(o ^ ((o >> 31) & 0x7fffffff)); };
    if (tid == 0) s_floor = ordered(-INFINITY);
    __syncthreads();

    auto logit = [&](long long v) { return sizeof(T) == 2 ? bf16_to_f32(((const uint16_t*)base)[v]) : ((const float*)base)[v]; };
    auto key_of = [&](float x, long long v) {     // a single entry: its own generator block
        uint32_t w[4];
        philox4x32_10((uint32_t)(v >> 2), (uint32_t)row, a.seed_lo, a.seed_hi, w);
        const uint32_t lo = (v & 1) ? w[1] : w[0], hi = (v & 1) ? w[3] : w[2];
        return gumbel_key(x, a.c, (v & 2) ? hi : lo);
    };
    auto one = [&](long long v) { take(r, key_of(logit(v), v), (int)v); };
    // the drafted token's logit is requested first: its key is a lower bound for every piece of the row
    const int d = a.draft[row];
    const bool d_ok = d >= 0 && d < a.V;
    const float x_d = d_ok ? logit(d) : -INFINITY;
    // the wavefront's largest key so far joins the workgroup's (by shuffles: with the lane moves of wave_max this pass is
    // 3 % slower where rows have a clear winner, 33.5 against 32.3 us at N=8, B=32)
    auto publish = [&]() {
        float k = r.k;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) k = fmaxf(k, __shfl_xor(k, off, 64));
        if ((tid & 63) == 0) atomicMax(&s_floor, ordered(k));
        return k;
    };
    if (v_lo < v_hi) {
        const size_t e_lo = (size_t)row * (size_t)a.V + (size_t)v_lo;
        int head = (int)((VEC - (e_lo % VEC)) % VEC);
        if (head > v_hi - v_lo) head = (int)(v_hi - v_lo);
        const long long body0 = v_lo + head;
        const int nvec = (int)((v_hi - body0) / VEC);
        const long long tail0 = body0 + (long long)nvec * VEC;
        const u32x4* vp = reinterpret_cast<const u32x4*>(base + body0);
        const int shift = (int)(body0 & 3);       // place of a vector's first entry in its generator block (the same for all)

        float floor = -INFINITY;                  // lower bound of the row's largest key, as far as the wavefront knows
        for (int i0 = 0; i0 < nvec; i0 += VUNROLL * VTHREADS) {
            u32x4 raw[VUNROLL];
#pragma unroll
            for (int u = 0; u < VUNROLL; ++u) {
                const int i = i0 + u * VTHREADS + tid;
                raw[u] = __builtin_nontemporal_load(vp + min(i, nvec - 1));    // (a repeated vector changes nothing)
            }
            __builtin_amdgcn_sched_barrier(0);    // all requested before the first is waited for
            if (i0 == 0) {
                // a first lower bound: every thread's largest logit of this group, with its noise
                float xm = -INFINITY;
                int at = 0;
#pragma unroll
                for (int u = 0; u < VUNROLL; ++u) {
                    const uint32_t q[4] = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
#pragma unroll
                    for (int j = 0; j < VEC; ++j) {
                        const float x = sizeof(T) == 4 ? __uint_as_float(q[j % 4])
                                      : (j & 1) ? __uint_as_float(q[j / 2] & 0xffff0000u) : __uint_as_float(q[j / 2] << 16);
                        if (x > xm) { xm = x; at = u * 8 + j; }
                    }
                }
                const long long v = body0 + (long long)min((at >> 3) * VTHREADS + tid, nvec - 1) * VEC + (at & 7);
                take(r, key_of(xm, v), (int)v);
                floor = publish();
                if (d_ok) floor = fmaxf(floor, key_of(x_d, d));
            }
#pragma unroll
            for (int u = 0; u < VUNROLL; ++u) {
                if (i0 + u * VTHREADS >= nvec) break;
                const int i = min(i0 + u * VTHREADS + tid, nvec - 1);
                const long long v0 = body0 + (long long)i * VEC;
                const uint32_t q[4] = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
                float x[VEC];
#pragma unroll
                for (int j = 0; j < VEC; ++j)
                    x[j] = sizeof(T) == 4 ? __uint_as_float(q[j % 4])
                         : (j & 1) ? __uint_as_float(q[j / 2] & 0xffff0000u) : __uint_as_float(q[j / 2] << 16);
                float xm = x[0];
#pragma unroll
                for (int j = 1; j < VEC; ++j) xm = fmaxf(xm, x[j]);
                floor = fmaxf(floor, from_ordered(__builtin_amdgcn_readfirstlane(*(volatile int*)&s_floor)));
                if (!__any(!(__fmaf_rn(xm, a.c, NOISE_MAX) < floor))) continue;

                uint32_t w[NW];
#pragma unroll
                for (int b = 0; b < NW / 4; ++b) {
                    if (b == VEC / 4 && shift == 0) break;        // (aligned: the last block is not touched)
                    uint32_t o[4];
                    philox4x32_10((uint32_t)(v0 >> 2) + b, (uint32_t)row, a.seed_lo, a.seed_hi, o);
#pragma unroll
                    for (int j = 0; j < 4; ++j) w[b * 4 + j] = o[j];
                }
                if (shift) {
#pragma unroll
                    for (int j = 0; j < VEC; ++j) w[j] = shift == 1 ? w[j + 1] : shift == 2 ? w[j + 2] : w[j + 3];
                }
                float kb[VEC];
                float km = -INFINITY;
#pragma unroll
                for (int j = 0; j < VEC; ++j) {
                    kb[j] = __fmaf_rn(x[j], a.c, noise_bound(w[j]));
                    km = j == 0 ? kb[0] : fmaxf(km, kb[j]);
                }
                if (!__any(!(km < floor))) continue;
                const float before = r.k;
#pragma unroll
                for (int j = 0; j < VEC; ++j)
                    if (__any(!(kb[j] < floor))) take(r, gumbel_key(x[j], a.c, w[j]), (int)(v0 + j));
                if (__any(r.k > before)) floor = fmaxf(floor, publish());
            }
        }
        if (tid < head) one(v_lo + tid);
        if (tid < v_hi - tail0) one(tail0 + tid);
    }
    const float k_wave = wave_max(r.k);
    r.idx = wave_min(r.k == k_wave ? r.idx : 0x7fffffff);
    r.k = k_wave;
    __shared__ Best part[VTHREADS / 64];
    if ((tid & 63) == 0) part[tid >> 6] = r;
    __syncthreads();
    if (tid == 0) {
        Best t = part[0];
#pragma unroll
        for (int w = 1; w < VTHREADS / 64; ++w) take(t, part[w].k, part[w].idx);
        Best* const ws = reinterpret_cast<Best*>(a.ws) + (size_t)row * a.vsplits * 2;     // two pairs per record
        if (a.pieces > a.vsplits) {
            ws[piece] = t;
        } else {
            ws[2 * piece] = t;
            ws[2 * piece + 1] = Best{-INFINITY, 0};
        }
    }
}

constexpr int STHREADS = 64;   // one wavefront per rollout: no LDS, no workgroup barrier
constexpr int SMALL_THREADS = kOneLaunchWaves * 64;   // small calls: threads per rollout

// The decisions for rollout n, by one wavefront (lane `tid`), on vsplits records per position in the workspace (the first PRE
// of them requested together with the mask bytes), or, OWN, on one record each in LDS (small calls, see below).
template <int PRE, bool OWN>
__device__ __forceinline__ void select_block(const Args& a, int n, int tid, const Partial* own)
{
    const double tau = (double)a.tau;

    int count = 0;
    double best_conf = -1.0;     // confidences are positive
    int best_b = 0x7fffffff;
    int best_tok = -1;

    // the wavefront refreshes the K/V rows of up to RB positions at once (see fdd_block_kv_update): all loads are on
    // their way before the first store, so the rows share one memory latency (one by one, K before V, each row took two)
    constexpr int RB = 4;
    auto refresh_rows = [&](int n_rows, const size_t (&pos)[RB], const int (&tok)[RB]) {
        for (int c = tid; c < a.rf_row_vecs; c += STHREADS) {
            u32x4 k[RB], v[RB];
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                if (u < n_rows) {
                    int t = tok[u] % a.rf_T;
                    if (t < 0) t += a.rf_T;
                    k[u] = a.rf_tk[(size_t)t * a.rf_row_vecs + c];
                    v[u] = a.rf_tv[(size_t)t * a.rf_row_vecs + c];
                }
            }
#pragma unroll
            for (int u = 0; u < RB; ++u) {
                if (u < n_rows) {
                    a.rf_bk[pos[u] * a.rf_row_vecs + c] = k[u];
                    a.rf_bv[pos[u] * a.rf_row_vecs + c] = v[u];
                }
            }
        }
    };

    for (int b0 = 0; b0 < a.B; b0 += STHREADS) {     // lane `tid` takes position b0 + tid (ascending per lane)
        const int b = b0 + tid;
        const size_t i = (size_t)n * a.B + (b < a.B ? b : 0);
        // The first pieces' records are requested together with the mask bytes, not after them: whether the
        // position is eligible is known one memory round trip later, and the records are then already there.
        // (records of positions that are not eligible hold whatever an earlier call left; they are not used)
        const int vsplits = OWN ? 1 : a.vsplits;
        const Partial* const p = OWN ? own + (b < a.B ? b : 0) : a.ws + i * vsplits;
        u32x4 rec[PRE];
#pragma unroll
        for (int s = 0; s < PRE; ++s) rec[s] = s < vsplits ? reinterpret_cast<const u32x4*>(p)[s] : u32x4{0u, 0u, 0u, 0u};
        const bool eligible = b < a.B && a.mask[i] == 1 && !(a.scaffold && a.scaffold[i]);
        float conf_out = -INFINITY;
        uint8_t com = 0;
        int arg = -1;
        if (eligible) {
            auto unpack = [](const u32x4& r) {
                Partial q;
                q.m = __uint_as_float(r.x); q.arg = (int)r.y; q.s = __uint_as_float(r.z); q.pad = 0;
                return q;
            };
            // pieces cover ascending index ranges: strict '>' keeps the lowest id
            float M = unpack(rec[0]).m;
            arg = unpack(rec[0]).arg;
#pragma unroll
            for (int s = 1; s < PRE; ++s) {
                const Partial q = unpack(rec[s]);
                if (s < vsplits && q.m > M) { M = q.m; arg = q.arg; }
            }
            for (int s = PRE; s < vsplits; ++s)
                if (p[s].m > M) { M = p[s].m; arg = p[s].arg; }
            // sum of the pieces' fp32 sums, rescaled to the row maximum, finished in fp64
            double z = 0.0;
#pragma unroll
            for (int s = 0; s < PRE; ++s) {
                const Partial q = unpack(rec[s]);
                if (s < vsplits && q.s > 0.f) z += (double)(q.s * fast_exp2((q.m - M) * LOG2E));
            }
            for (int s = PRE; s < vsplits; ++s)
                if (p[s].s > 0.f) z += (double)(p[s].s * fast_exp2((p[s].m - M) * LOG2E));
            const double conf = 1.0 / z;
            conf_out = (float)conf;
            if (conf >= tau) {
                a.tokens[i] = arg;
                a.mask[i] = 0;
                com = 1;
                ++count;
            }
            if (conf > best_conf) { best_conf = conf; best_b = b; best_tok = arg; }   // ascending b per thread
        }
        if (b < a.B) {
            a.conf[i] = conf_out;
            if (a.committed) a.committed[i] = com;
        }
        if (a.rf_row_vecs > 0) {
            unsigned long long m = __ballot(com != 0);
            while (m) {
                size_t pos[RB] = {};
                int tok[RB] = {}, n_rows = 0;
#pragma unroll
                for (int u = 0; u < RB; ++u) {
                    if (m) {
                        const int j = __builtin_ctzll(m);
                        m &= m - 1;
                        pos[u] = (size_t)n * a.B + b0 + j;
                        tok[u] = __builtin_amdgcn_readlane(arg, j);
                        n_rows = u + 1;
                    }
                }
                refresh_rows(n_rows, pos, tok);
            }
        }
    }
    // wavefront reduction: commits are summed; the best candidate is the one of highest confidence, lowest position on
    // ties (a confidence is positive, so its 64 bits order as an integer: upper half, then lower half, then position)
    count = (int)wave_reduce((uint32_t)count, [](uint32_t p, uint32_t q) { return p + q; });
    auto larger = [](uint32_t p, uint32_t q) { return p > q ? p : q; };
    const uint64_t bits = best_conf > 0.0 ? (uint64_t)__double_as_longlong(best_conf) : 0u;
    const uint32_t hi = (uint32_t)(bits >> 32), lo = (uint32_t)bits;
    const uint32_t hi_best = wave_reduce(hi, larger);
    const uint32_t lo_best = wave_reduce(hi == hi_best ? lo : 0u, larger);
    const int b_lane = best_b;
    best_b = wave_min(hi == hi_best && lo == lo_best ? b_lane : 0x7fffffff);
    best_tok = __builtin_amdgcn_readlane(best_tok, __builtin_ctzll(__ballot(b_lane == best_b)));
    // (count and the best candidate are now the same in every lane)
    if (count == 0 && best_tok >= 0) {
        // nothing reached tau: commit the most confident eligible position
        const size_t i = (size_t)n * a.B + best_b;
        if (tid == 0) {
            a.tokens[i] = best_tok;
            a.mask[i] = 0;
            if (a.committed) a.committed[i] = 1;
        }
        if (a.rf_row_vecs > 0) {
            const size_t pos[RB] = {i};
            const int tok[RB] = {best_tok};
            refresh_rows(1, pos, tok);
        }
        count = 1;
    }
    if (tid == 0 && a.n_unmasked) a.n_unmasked[n] = count;
}

template <int PRE>
__global__ __launch_bounds__(STHREADS) void block_select_kernel(Args a) { select_block<PRE, false>(a, (int)wg_id_x(), thread_id_x(), nullptr); }

// Small calls in one launch: a workgroup per rollout, a wavefront per position in turn, decisions by the first wavefront on
// records in LDS.  Bound by latency and launches either way.  The same values as the two kernels: a row's lanes walk it in
// ascending order and meet in the same reductions (their sums in another order: confidences differ by 1e-7).
template <typename T>
__global__ __launch_bounds__(SMALL_THREADS) void block_unmask_small_kernel(Args a)
{
    constexpr int VEC = 16 / sizeof(T);
    __shared__ __align__(16) Partial part[kOneLaunchB];
    const int n = (int)wg_id_x(), tid = thread_id_x(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int V = (int)a.V;
    for (int b = wave; b < a.B; b += SMALL_THREADS / 64) {
        const int row = n * a.B + b;
        const uint8_t m = a.mask[row], sc = a.scaffold ? a.scaffold[row] : (uint8_t)0;
        if (m != 1 || sc) continue;
        const T* x0 = static_cast<const T*>(a.logits) + (size_t)row * V;
        ThreadRun t;
        t.r.m = -INFINITY;
        t.r.idx = 0x7fffffff;
        t.r.s = 0.f;
        t.mc = -INFINITY;
        auto at = [&](int v) { return sizeof(T) == 2 ? bf16_to_f32(((const uint16_t*)x0)[v]) : ((const float*)x0)[v]; };
        const int head = min((int)((VEC - ((size_t)row * V) % VEC) % VEC), V), nvec = (V - head) / VEC;
        if (lane < head) {
            const float x[1] = {at(lane)};
            absorb<1, true>(t, x, lane);
        }
        const u32x4* vp = reinterpret_cast<const u32x4*>(x0 + head);
        for (int i = lane; i < nvec; i += 64) {
            const u32x4 raw = vp[i];
            const uint32_t q[4] = {raw.x, raw.y, raw.z, raw.w};
            float x[VEC];
#pragma unroll
            for (int j = 0; j < VEC; ++j)
                x[j] = sizeof(T) == 4 ? __uint_as_float(q[j % 4]) : (j & 1) ? __uint_as_float(q[j / 2] & 0xffff0000u) : __uint_as_float(q[j / 2] << 16);
            absorb<VEC, true>(t, x, head + i * VEC);
        }
        const int tail = head + nvec * VEC + lane;
        if (tail < V) {
            const float x[1] = {at(tail)};
            absorb<1, true>(t, x, tail);
        }
        Run r = settle(t);
        const float m_wave = wave_max(r.m);
        const float sum = wave_sum(r.m == m_wave ? r.s : r.s * fast_exp2((r.m - m_wave) * LOG2E));
        const int idx = wave_min(r.m == m_wave ? r.idx : 0x7fffffff);
        if (lane == 0) part[b] = Partial{m_wave, idx, sum, 0};
    }
    __syncthreads();
    if (wave == 0) select_block<1, true>(a, n, lane, part);
}

// Accept scan of scaffold speculative decoding: one wavefront per rollout.
// Draft positions are visited in ascending order; drafts equal to the AR arg
// max are accepted up to the first mismatch, which takes the AR token; later
// drafts are left masked.
// PAIRS: a record holds the (key, id) pairs of two pieces (sampled verifier), else one piece's (max, id) and no second one.
template <bool PAIRS>
__global__ __launch_bounds__(STHREADS) void verify_scan_kernel(Args a)
{
    const int n = wg_id_x();
    const int tid = thread_id_x();
    // pass 1: position of the first mismatch, and the AR token there.  A position's records and its draft are
    // requested together with its mask bytes (one memory round trip instead of three); what was requested for
    // a position that is no draft is not used.
    constexpr int PRE = 8;
    int first_bad = 0x7fffffff;
    int bad_tok = 0;            // AR token at this lane's lowest mismatch
    for (int b = tid; b < a.B; b += STHREADS) {
        const size_t i = (size_t)n * a.B + b;
        const u32x4* pr = reinterpret_cast<const u32x4*>(a.ws + i * a.vsplits);
        u32x4 rec[PRE];
#pragma unroll
        for (int s = 0; s < PRE; ++s) rec[s] = s < a.vsplits ? pr[s] : u32x4{0u, 0u, 0u, 0u};
        const int d = a.draft[i];
        const bool is_draft = a.mask[i] == 1 && !(a.scaffold && a.scaffold[i]);
        if (!is_draft) continue;
        // ascending pieces: strict '>' keeps the lowest id on ties
        float M = __uint_as_float(rec[0].x);
        int arg = (int)rec[0].y;
        auto larger = [&](uint32_t m, uint32_t id) {
            if (__uint_as_float(m) > M) { M = __uint_as_float(m); arg = (int)id; }
        };
        if (PAIRS) larger(rec[0].z, rec[0].w);
#pragma unroll
        for (int s = 1; s < PRE; ++s) {
            if (s >= a.vsplits) continue;
            larger(rec[s].x, rec[s].y);
            if (PAIRS) larger(rec[s].z, rec[s].w);
        }
        for (int s = PRE; s < a.vsplits; ++s) {
            const u32x4 r = pr[s];
            larger(r.x, r.y);
            if (PAIRS) larger(r.z, r.w);
        }
        if (arg != d && b < first_bad) { first_bad = b; bad_tok = arg; }
    }
    first_bad = wave_min(first_bad);
    // pass 2: accept up to it, replace at it, leave the rest
    int count = 0;
    for (int b = tid; b < a.B; b += STHREADS) {
        const size_t i = (size_t)n * a.B + b;
        const bool is_draft = a.mask[i] == 1 && !(a.scaffold && a.scaffold[i]);
        uint8_t acc = 0;
        if (is_draft && b <= first_bad) {
            acc = (b == first_bad) ? 2 : 1;
            // (the lane that visits position first_bad met no mismatch below it: bad_tok is the token there)
            a.tokens[i] = (b == first_bad) ? bad_tok : a.draft[i];
            a.mask[i] = 0;
            ++count;
        }
        if (a.committed) a.committed[i] = acc;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) count += __shfl_xor(count, off, 64);
    if (tid == 0 && a.n_unmasked) a.n_unmasked[n] = count;
}

}  // namespace

bool make_unmask_plan(const fdd_unmask_params& p, UnmaskPlan* plan)
{
    return make_vocab_plan(p.N, p.B, p.V, p.dtype, false, plan);
}

bool make_vocab_plan(int N, int B, long long V, int dtype, bool argmax_only, UnmaskPlan* plan)
{
    struct { int N, B; long long V; int dtype; } p = {N, B, V, dtype};
    if (p.N <= 0 || p.B <= 0 || p.V <= 0) return false;
    const long long rows = (long long)p.N * p.B;
    const long long es = p.dtype == FDD_BF16 ? 2 : 4;
    long long by_size = (p.V * es) / ((argmax_only ? PIECE_KB_ARGMAX : PIECE_KB) * 1024);     // keep pieces at this size or more
    if (by_size < 1) by_size = 1;
    long long want = (8192 + rows - 1) / rows;  // enough workgroups to fill 256 CUs several times
    if (want < 1) want = 1;
    long long vs = want < by_size ? want : by_size;
    const long long small = std::min({(p.V * es) / (PIECE_KB_FEW * 1024), kFewPieces / rows, 8ll});
    if (vs < small) vs = small;
    if (vs > 64) vs = 64;
    plan->vsplits = (int)vs;
    plan->ws_bytes = (size_t)rows * (size_t)vs * sizeof(Partial);
    return true;
}

// Entries per piece: a multiple of 64 (128 bytes of bf16), so that the pieces of an aligned row start on whole cache
// lines and have no entries outside whole 16-byte vectors but the row's own last ones.
static void set_pieces(Args& a, int vsplits, long long V, int pieces)
{
    a.vsplits = vsplits;
    a.pieces = pieces;
    a.units = a.N * a.B * pieces;
    a.V = V;
    const long long per = (V + pieces - 1) / pieces;
    a.per = (int)std::min<long long>((per + 63) / 64 * 64, V);
    a.dVs = make_fastdiv((uint32_t)pieces);
}

// Whether workgroups are dealt to eligible rows only (see eligible_row).  It costs each of them 0.3 us at its start, so not
// where it has little to do, and nothing is gained up to 512 pieces, two to a compute unit, or from about 3000 on, where so
// many even out.  us per call, replayed, row by row / dealt, at shares of 0.5 and 0.9 of the rows live:
//   with sums N=8, B=32, V=152064 (pieces of 74 KB) 18.6/15.4, 20.0/20.5; N=16, B=64, V=50001 (98 KB) 21.4/17.6, 23.9/24.5, V=20000
//   (39 KB) 13.8/12.7, 14.5/15.1, V=9973 (20 KB) 11.1/10.7, 11.7/12.1, V=2000 8.4/8.7, 8.4/9.4;
//   without N=8, B=32, V=152064 (37 KB, 2048 pieces) 16.0/15.1, 18.4/19.0; N=16, B=64, V=20000 (39 KB, 1024 pieces) 12.4/11.7,
//   13.4/14.0; N=4, B=40, V=50001 (16 KB) 9.8/10.1, 10.5/11.1;
//   sampled verifier N=8, B=32, V=152064 39.1/29.4, 43.6/44.6; N=16, B=64, V=2000 12.9/11.6, 13.2/13.9.
enum class Pass { SUMS, ARGMAX, SAMPLE };
static bool deal_to_eligible(const Args& a, Pass pass, long long piece_bytes)
{
    if (a.N * a.B < 16 || a.N * a.B > LIVE_ROWS || a.units <= 512 || a.units > 2560) return false;
    return pass == Pass::SAMPLE || (piece_bytes >= 32 * 1024 && (pass == Pass::SUMS || a.units > 1024));
}

// Threads per piece: 512 from 60 KB on (its loads in two groups instead of four), 256 below, where the second group of 512 is
// nearly empty.  us per call, replayed, half of the rows live, 256 / 512 threads, and in brackets the mean of their ratio over
// shares of live rows from 0.2 to 1 (a last round of workgroups that is nearly empty moves a single point by 10 %):
//   with sums, pieces of 49 KB, 4096 rows 27.0/28.2 (0.97); 55 KB 29.1/29.6 (1.00); 61 KB 32.4/31.3 (1.02); 70 KB 36.3/34.2
//   (1.09); 64 KB, two a row 51.0/52.0 (1.01), fp32, 2048 rows 32.1/29.8 (1.08); 74 KB, four a row 1024 rows 36.7/36.1 (1.04), 2048
//   63.2/69.3 (0.97), 4096 105/101 (1.04);
//   without, 49 KB, 4096 rows in two 42.0/48.7 (0.91), 2048 in four 38.8/40.5 (0.96); 54 KB 42.3/45.9 (0.97); 63 KB 46.5/46.4
//   (1.01); 64 KB 48.7/46.9 (1.03); 74 KB 57.2/59.2 (1.00), 100/95.7 (1.04).
template <bool SUM>
static void launch_reduce(const Args& a, int dtype, hipStream_t s)
{
    const long long piece_bytes = (long long)a.per * (dtype == FDD_BF16 ? 2 : 4);
    const bool wide = piece_bytes >= 60 * 1024;
    auto go = [&](auto t, auto threads, auto comp) {
        constexpr int THREADS = decltype(threads)::value;
        hipLaunchKernelGGL((vocab_reduce_kernel<decltype(t), SUM, THREADS, decltype(comp)::value>), dim3((unsigned)a.units), dim3(THREADS), 0, s, a);
    };
    auto sized = [&](auto t, auto comp) {
        if (wide) go(t, std::integral_constant<int, 512>(), comp);
        else go(t, std::integral_constant<int, 256>(), comp);
    };
    auto typed = [&](auto comp) {
        if (dtype == FDD_BF16) sized(uint16_t(), comp);
        else sized(float(), comp);
    };
    if (deal_to_eligible(a, SUM ? Pass::SUMS : Pass::ARGMAX, piece_bytes)) typed(std::true_type());
    else typed(std::false_type());
}

template <typename T>
static void launch_sample(const Args& a, hipStream_t s)
{
    if (deal_to_eligible(a, Pass::SAMPLE, 0)) hipLaunchKernelGGL((vocab_sample_kernel<T, true>), dim3((unsigned)a.units), dim3(VTHREADS), 0, s, a);
    else hipLaunchKernelGGL((vocab_sample_kernel<T, false>), dim3((unsigned)a.units), dim3(VTHREADS), 0, s, a);
}

hipError_t launch_unmask(const fdd_unmask_params& p, const UnmaskPlan& plan, hipStream_t s)
{
    Args a;
    a.logits = p.logits;
    a.scaffold = p.scaffold_mask;
    a.mask = p.mask;
    a.tokens = p.tokens;
    a.conf = p.confidences;
    a.n_unmasked = p.n_unmasked;
    a.committed = p.committed;
    a.ws = static_cast<Partial*>(p.workspace);
    a.draft = nullptr;
    a.rf_tk = static_cast<const u32x4*>(p.refresh_table_k);
    a.rf_tv = static_cast<const u32x4*>(p.refresh_table_v);
    a.rf_bk = static_cast<u32x4*>(p.refresh_block_k);
    a.rf_bv = static_cast<u32x4*>(p.refresh_block_v);
    a.rf_T = p.refresh_T;
    a.rf_row_vecs = p.refresh_block_k ? (int)((size_t)p.refresh_Hkv * p.refresh_D * (p.refresh_dtype == FDD_BF16 ? 2 : 4) / 16) : 0;
    a.N = p.N; a.B = p.B; a.tau = p.tau;
    set_pieces(a, plan.vsplits, p.V, plan.vsplits);
    a.c = 0.f; a.seed_lo = 0u; a.seed_hi = 0u;
    if (unmask_in_one_launch(p.N, p.B, p.V * (p.dtype == FDD_BF16 ? 2 : 4))) {
        if (p.dtype == FDD_BF16) hipLaunchKernelGGL(block_unmask_small_kernel<uint16_t>, dim3(p.N), dim3(SMALL_THREADS), 0, s, a);
        else hipLaunchKernelGGL(block_unmask_small_kernel<float>, dim3(p.N), dim3(SMALL_THREADS), 0, s, a);
        return hipGetLastError();
    }
    launch_reduce<true>(a, p.dtype, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // (eight records' requests where there are four or fewer cost 0.2 us for every 64 positions of a block)
    if (a.vsplits <= 4) hipLaunchKernelGGL(block_select_kernel<4>, dim3(p.N), dim3(STHREADS), 0, s, a);
    else hipLaunchKernelGGL(block_select_kernel<8>, dim3(p.N), dim3(STHREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_verify(const fdd_verify_params& p, const UnmaskPlan& plan, hipStream_t s)
{
    Args a;
    a.logits = p.ar_logits;
    a.scaffold = p.scaffold_mask;
    a.mask = p.mask;
    a.tokens = p.tokens;
    a.conf = nullptr;
    a.n_unmasked = p.n_accepted;
    a.committed = p.accepted;
    a.ws = static_cast<Partial*>(p.workspace);
    a.draft = p.draft;
    a.rf_tk = nullptr; a.rf_tv = nullptr; a.rf_bk = nullptr; a.rf_bv = nullptr; a.rf_T = 0; a.rf_row_vecs = 0;
    a.N = p.N; a.B = p.B; a.tau = 0.f;
    // The sampled verifier, bound by its arithmetic, takes twice the pieces while those are 16 KB or more and 2048 at most, or, with
    // no more than two of them to a compute unit, 8 KB.  us per call, replayed, plain / twice: V = 152064 bf16, 70 % of the rows
    // live, a clear winner in 4 of 5 rows: N=1, B=32 16.8/15.6, N=4 21.5/21.3, N=8 30.4/27.3 (36.0/36.6 without winners; 512
    // threads per piece 30.9, 36.3); more pieces N=16, B=64 64.7/64.7 (99.9/115); smaller ones V = 50001, 200 rows in 5 21.5/24.3.
    // Smaller and few, half of the rows live: V = 9973, N=8, B=32 14.8/13.6, N=1 13.8/12.1; V = 16000, N=8 14.5/12.7; V = 50001, N=1
    // 14.6/13.2; too small V = 5000, N=8 11.0/11.4.
    const long long bytes = p.V * (p.dtype == FDD_BF16 ? 2 : 4), units = (long long)p.N * p.B * plan.vsplits;
    const bool twice = p.temperature > 0.f && units <= 1024 && bytes >= (units <= kNumCU ? 16ll : 32ll) * 1024 * plan.vsplits;
    set_pieces(a, plan.vsplits, p.V, twice ? 2 * plan.vsplits : plan.vsplits);
    a.c = p.temperature > 0.f ? (float)(1.4426950408889634 / (double)p.temperature) : 0.f;
    a.seed_lo = (uint32_t)p.seed;
    a.seed_hi = (uint32_t)(p.seed >> 32);
    if (p.temperature > 0.f) {
        if (p.dtype == FDD_BF16) launch_sample<uint16_t>(a, s);
        else launch_sample<float>(a, s);
    } else {
        // greedy verifier: step 3 of scaffold speculative decoding compares arg maxima only, so no exponentials
        launch_reduce<false>(a, p.dtype, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.temperature > 0.f) hipLaunchKernelGGL(verify_scan_kernel<true>, dim3(p.N), dim3(STHREADS), 0, s, a);
    else hipLaunchKernelGGL(verify_scan_kernel<false>, dim3(p.N), dim3(STHREADS), 0, s, a);
    return hipGetLastError();
}

}  // namespace fdd
