// Shared-prefix block-causal attention, fp32 storage and arithmetic, and the
// merge of its splits.
//
// The same thing as the bf16 kernel computes (paper, "Block-Causal Diffusion"
// and "Shared prefix").  Two kernels: attn_f32_kernel, with fp32 products and
// sums on the matrix cores (v_mfma_f32_16x16x4_f32), for calls of few rows and
// few keys, and attn_f32_wide_kernel further below, which takes each fp32
// product apart into bf16 products.
//
// How the work is laid out
//   * A workgroup owns 32 stacked query rows of one KV head (see AttnPlan), or 16
//     where the call leaves half of the compute units idle; its
//     8 wavefronts share the KEYS out among themselves, 16 at a time, each with
//     a streaming-softmax state (m, l, o) of its own, and merge through LDS at
//     the end.  `splits` workgroups share one row tile when the row tiles alone
//     leave the chip idle; then a second small kernel merges their partials.
//   * S^T = K Q^T: a lane owns query lane % 16 of each 16-query block and
//     keys 4 (lane / 16) .. + 3, so the probabilities are the B operand of
//     O^T += V^T P^T as they lie.  The channels are dealt to the k-steps (and to
//     the rows of O^T) such that every operand is a 16-byte piece of a K or V row:
//     the fragments come straight from global memory, no LDS, no barrier.
//   * What bounds it: the matrix pipe (64 flop per cycle and SIMD; a 16-byte
//     fragment load feeds 8 matrix instructions of 32 cycles, so the four SIMDs
//     ask for 16 bytes per cycle and CU, a quarter of what the vector cache
//     delivers).  Splitting keys instead of rows over the wavefronts costs no
//     time then, and makes the row tiles small: 32 rows fill the chip without (or
//     with few) splits, whose partials would cost a pass over memory each.
//   * A fragment register is requested again for the next tile as soon as it has
//     been used: a whole step, 4096 cycles at D = 128, of latency is covered.
//   * A short call is start, first loads, a few tiles and the LDS merge.  With 16 rows a
//     wavefront has half of the matrix work per tile and half of the merge: N = 1, B = 8,
//     L = 256, Hq = 4, Hkv = 1, D = 64 10.4 -> 7.1 us, N = 2, B = 32, L = 128, Hq = 28, Hkv = 4,
//     D = 128 16.3 -> 11.0 (replayed).
//   * Measured at N = 8, B = 32, L = 4096, Hq = 28, Hkv = 4, D = 128 (15.1 GFLOP), a call that
//     comes here with a forced cut, an unusual scale or too little scratch only and takes the
//     128-row tiles otherwise: 135 us in a loop of nothing else, 112 TFLOP/s of the 154 a large
//     fp32 matrix product reaches here; 224 of 256 CUs are used, the matrix pipe of a used CU 84 %
//     of its cycles.  Scalar fused multiply-adds from LDS tiles: 687 us in a denoise step, where
//     this kernel took 149.  Not faster, when it took 152 there: K through a private LDS ring,
//     the next tile's scores under this tile's exponentials, priorities that keep the two
//     wavefronts of a SIMD level (157 us each).
#include "fdd_internal.h"

#include <atomic>
#include <type_traits>
#include <utility>

namespace fdd {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KT = 16;                 // keys per tile
constexpr int WAVES = kF32Waves;       // wavefronts of a workgroup, sharing the keys
constexpr int THREADS = WAVES * 64;

struct Args {
    const float* q;
    const float* pk;
    const float* pv;
    const float* bk;
    const float* bv;
    float* out;
    float* ws_o;
    float* ws_ml;
    const float* ek;   // per-rollout extension [N, Ecap, Hkv, D]
    const float* ev;
    int E, Ecap;
    long long q_bs, p_bs, b_bs, e_bs, o_bs;   // element strides between the arrays of independent problems
    int N, B, L, Hq, Hkv, G, R, MT, S;
    int W, per_xcd;    // workgroups; launched workgroups / 8
    unsigned grid_x;   // workgroups per row of the launch grid
    int causal;        // in-block keys are visible up to the query's own position only
    float c;           // scale * log2(e)
    float slack;       // 8 / c: scores may pass their reference by this much
    const int32_t* qpos;   // stacked rows are the listed block positions only (ascending n*B + b), or nullptr: all of them
    int ext_per, per;      // private tiles per rollout: of its extension, in all (extension, then block)
    FastDiv dMT, dS, dHkv, dG, dB, dPer, dParts;   // divisions by launch constants
};

// block position n*B + b of entry `e` of the list of query positions (clamped into range), or e itself without a list
__device__ __forceinline__ int position_of(const int32_t* qpos, int e, int NB)
{
    return qpos ? min(max(qpos[e], 0), NB - 1) : e;
}

// the same pointer, known to be wave-uniform (kept in scalar registers)
__device__ __forceinline__ const char* uniform(const char* p)
{
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

// Tile t of the keys of a row tile whose rollouts start at n_lo: TP prefix tiles of K keys, then for every rollout the tiles
// of its extension and of its block.
struct KeyTile {
    const char* k;    // first key's row of this KV head
    const char* v;
    int valid;        // keys that exist
    int rollout;      // whose rows may see it (-1: every row)
    int key0;         // block position of the first key (block tiles under the causal mask), else hugely negative
};
template <int K, int D>
__device__ __forceinline__ KeyTile key_tile(const Args& a, int pb, int kh, int n_lo, int TP, int t)
{
    KeyTile r;
    long long row;
    long long bs;
    const float *kp, *vp;
    r.key0 = -(1 << 30);
    if (t < TP) {
        kp = a.pk; vp = a.pv; bs = a.p_bs;
        row = (long long)t * K;
        r.valid = min(K, a.L - t * K);
        r.rollout = -1;
    } else {
        const int j = t - TP, i = fast_div(j, a.dPer), w = j - i * a.per;
        r.rollout = n_lo + i;
        if (w < a.ext_per) {
            kp = a.ek; vp = a.ev; bs = a.e_bs;
            row = (long long)r.rollout * a.Ecap + w * K;
            r.valid = min(K, a.E - w * K);
        } else {
            const int k0 = (w - a.ext_per) * K;
            kp = a.bk; vp = a.bv; bs = a.b_bs;
            row = (long long)r.rollout * a.B + k0;
            r.valid = min(K, a.B - k0);
            if (a.causal) r.key0 = k0;
        }
    }
    const long long off = ((long long)pb * bs + row * a.Hkv * D + (long long)kh * D) * 4;
    r.k = uniform(reinterpret_cast<const char*>(kp) + off);
    r.v = uniform(reinterpret_cast<const char*>(vp) + off);
    r.valid = __builtin_amdgcn_readfirstlane(r.valid);
    r.rollout = __builtin_amdgcn_readfirstlane(r.rollout);
    r.key0 = __builtin_amdgcn_readfirstlane(r.key0);
    return r;
}

// Streaming softmax of a wavefront's QB blocks of 16 query rows in the layout of the 16x16x4 matrix instruction.
template <int D, int QB>
struct WaveState {
    f32x4 o[QB][D / 64][4];   // [query block][64-channel block][e]: channels 64 t + 16 g4 + 4 v + e of query c16
    float m_ref[QB];          // reference the exponentials are taken against (raw score units)
    float limit[QB];          // a score further above the reference raises it; -inf: there is none yet
    float l_run[QB];          // this lane's share of the running sum
};

// One wavefront over tiles [t_lo, t_hi) of 16 keys.  `several`: the row tile's rows belong to more than one rollout.
template <int D, int QB, typename TileAt>
__device__ __forceinline__ void f32_wave_loop(const Args& a, const TileAt& tile_at, int t_lo, int t_hi, const f32x4 (&qf)[QB][D / 16],
                                              const int (&my_rollout)[QB], const int (&my_b)[QB], bool several, WaveState<D, QB>& w)
{
    constexpr int NJ = D / 16;         // 16-byte fragment loads per tile and operand
    constexpr int NT = D / 64;         // 64-channel blocks of the output
    const int lane = thread_id_x() & 63, c16 = lane & 15, g4 = lane >> 4;
    const uint32_t stride4 = (uint32_t)(a.Hkv * D * 4);     // bytes between consecutive keys
    // Fragments of a tile.  K: row c16, channels 16 j + 4 g4 ..; V: row 4 g4 + v, channels 64 t + 4 c16 ..
    // (rows beyond `valid` repeat the last valid one: masked below, nothing read out of bounds)
    f32x4 kf[NJ], vf[NJ];
    auto k_off = [&](const KeyTile& t) { return (uint32_t)min(c16, max(t.valid, 1) - 1) * stride4 + (uint32_t)(16 * g4); };
    auto v_off = [&](const KeyTile& t, int v) { return (uint32_t)min(4 * g4 + v, max(t.valid, 1) - 1) * stride4 + (uint32_t)(16 * c16); };
    // (offsets inside a tile stay below 2^32, as the whole block K does, but may pass 2^31 with very many KV heads)
    auto load = [&](const char* base, uint32_t off) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, -1, 0x00020000);
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
    };

    auto& o = w.o;
    auto& m_ref = w.m_ref;
    auto& limit = w.limit;
    auto& l_run = w.l_run;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_ref[qb] = l_run[qb] = 0.f;
        limit[qb] = -INFINITY;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[qb][t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    if (t_lo < t_hi) {
        KeyTile now = tile_at(t_lo);
        {
            const uint32_t off = k_off(now);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                kf[j] = load(now.k, off + 64 * j);
                __builtin_amdgcn_sched_barrier(0);     // (the order of the loop's requests, which the waits in it count)
            }
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    vf[v * NT + tt] = load(now.v, v_off(now, v) + 256 * tt);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        for (int t = t_lo; t < t_hi; ++t) {
            // A fragment of the next tile is requested as soon as the matrix instructions that read its
            // predecessor are issued: every request has a whole step to arrive.  (The last tile is requested
            // once more at the end, from the caches.)
            const KeyTile next = tile_at(min(t + 1, t_hi - 1));
            const uint32_t next_k = k_off(next);
            f32x4 s[QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) s[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
                        s[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][i], qf[qb][j][i], s[qb], 0, 0, 0);
                kf[j] = load(next.k, next_k + 64 * j);
                __builtin_amdgcn_sched_barrier(0);
            }
            // register v of a query block is key 4 g4 + v
            if (now.valid < KT || now.rollout >= 0) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int key = 4 * g4 + v;
                        const bool sees = (now.rollout < 0) | (now.rollout == my_rollout[qb]);
                        const bool hidden = !sees | (key >= now.valid) | (now.key0 + key > my_b[qb]);
                        s[qb][v] = hidden ? -INFINITY : s[qb][v];
                    }
            }
            // Scores against the reference: the difference first, because rescales and merges weigh by differences of
            // references, and a rounded product m c in place of m would set each wavefront off by up to half a unit of it.
            // The reference is raised when a score outgrows it by more than 2^8 (the same softmax; fp32 keeps its
            // relative precision), for a whole row at a time: its keys lie in the four lanes c16 + 16 i.
            f32x4 p[QB];
            bool need = false;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                for (int v = 0; v < 4; ++v) p[qb][v] = s[qb][v] - m_ref[qb];
                need |= fmaxf(fmaxf(p[qb][0], p[qb][1]), fmaxf(p[qb][2], p[qb][3])) > limit[qb];
            }
            if (__any(need)) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    const bool none = limit[qb] == -INFINITY;
                    float m = fmaxf(fmaxf(s[qb][0], s[qb][1]), fmaxf(s[qb][2], s[qb][3]));
                    m = fmaxf(m, __shfl_xor(m, 16, 64));
                    m = fmaxf(m, __shfl_xor(m, 32, 64));
                    if (!none) m = fmaxf(m, m_ref[qb]);
                    const float alpha = none ? 1.f : exp2f((m_ref[qb] - m) * a.c);
                    m_ref[qb] = m == -INFINITY ? 0.f : m;
                    limit[qb] = m == -INFINITY ? m : a.slack;
                    l_run[qb] *= alpha;
#pragma unroll
                    for (int v = 0; v < 4; ++v) p[qb][v] = s[qb][v] - m_ref[qb];
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[qb][tt][e] *= alpha;
                }
            }
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                for (int v = 0; v < 4; ++v) p[qb][v] = __builtin_amdgcn_exp2f(p[qb][v] * a.c);
                l_run[qb] += (p[qb][0] + p[qb][1]) + (p[qb][2] + p[qb][3]);
            }
            // What a row does not see must not reach its sums through 0 x inf or 0 x NaN: keys that do not exist (the
            // rows loaded in their place repeat the last one) ...
            if (now.valid < KT) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) vf[v * NT + tt][e] = 4 * g4 + v < now.valid ? vf[v * NT + tt][e] : 0.f;
            }
            // ... and, in a row tile of several rollouts, values of another one that are not finite.  A lane's outputs
            // belong to one query: the tile's share is then summed by itself, added where the query sees it, and nothing
            // is left for the sums below.
            if (now.rollout >= 0 && several) {
                float x0 = 0.f;      // NaN if any value is not finite
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x0 = fmaf(vf[j][e], 0.f, x0);
                if (__builtin_expect(__any(x0 != 0.f), 0)) {
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int qb = 0; qb < QB; ++qb) {
                                f32x4 x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                                for (int v = 0; v < 4; ++v)
                                    x = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v * NT + tt][e], p[qb][v], x, 0, 0, 0);
#pragma unroll
                                for (int v = 0; v < 4; ++v) o[qb][tt][e][v] += now.rollout == my_rollout[qb] ? x[v] : 0.f;
                                __builtin_amdgcn_sched_barrier(0);
                            }
#pragma unroll
                    for (int j = 0; j < NJ; ++j) vf[j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint32_t next_v = v_off(next, v);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int qb = 0; qb < QB; ++qb)
                            o[qb][tt][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v * NT + tt][e], p[qb][v], o[qb][tt][e], 0, 0, 0);
                    vf[v * NT + tt] = load(next.v, next_v + 256 * tt);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            now = next;
        }
    }
}

template <int D, int QB>
struct F32Cfg {
    static constexpr int RT = 16 * QB;                    // rows per workgroup
    static constexpr int MERGE_FLOATS = WAVES * RT * D;   // outputs of all wavefronts, in register order
    static constexpr int LDS_BYTES = (MERGE_FLOATS + 2 * WAVES * RT + 2 * RT) * 4;   // + (m, l) per wavefront and row, and per row
};

template <int D, int QB>
__global__ __launch_bounds__(THREADS) void attn_f32_kernel(Args a)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub
    constexpr int RT = F32Cfg<D, QB>::RT;
    constexpr int NJ = D / 16;         // 16-byte fragment loads per tile and operand
    constexpr int NT = D / 64;         // 64-channel blocks of the output
    extern __shared__ __align__(16) float smem[];

    // workgroups are dealt to the 8 XCDs round-robin: those of one XCD own neighbouring row tiles of one
    // (KV head, split), which walk the same keys
    const unsigned id = wg_id_y() * a.grid_x + wg_id_x();
    const int wg = (int)(id % kNumXCD) * a.per_xcd + (int)(id / kNumXCD);
    if (wg >= a.W) return;
    const int rest = fast_div(wg, a.dMT), mt = wg - rest * a.MT;
    const int khv = fast_div(rest, a.dS), split = rest - khv * a.S;
    const int pb = fast_div(khv, a.dHkv), kh = khv - pb * a.Hkv;     // problem of the batch, KV head

    const int tid = thread_id_x(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, g4 = lane >> 4;
    const int NB = a.N * a.B;

    // ---- query rows of this lane: c16 of every 16-query block --------------------------------------
    f32x4 qf[QB][NJ];
    int my_rollout[QB], my_b[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int row = min(mt * RT + qb * 16 + c16, a.R - 1);
        const int sel = fast_div(row, a.dG), g = row - sel * a.G;
        const int nb = position_of(a.qpos, sel, NB);
        my_rollout[qb] = fast_div(nb, a.dB);
        my_b[qb] = nb - my_rollout[qb] * a.B;
        const float* qp = a.q + pb * a.q_bs + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * D + 4 * g4;
#pragma unroll
        for (int j = 0; j < NJ; ++j) qf[qb][j] = *reinterpret_cast<const f32x4*>(qp + 16 * j);
    }

    // ---- key tiles of this wavefront ---------------------------------------------------------------
    // prefix tiles, then for every rollout the rows belong to: extension tiles, block tiles
    // (rows are in ascending order of position, hence of rollout)
    const int row_hi = min(mt * RT + RT, a.R) - 1;
    const int n_lo = __builtin_amdgcn_readfirstlane(fast_div(position_of(a.qpos, fast_div(mt * RT, a.dG), NB), a.dB));
    const int n_hi = __builtin_amdgcn_readfirstlane(fast_div(position_of(a.qpos, fast_div(row_hi, a.dG), NB), a.dB));
    const int TP = (a.L + KT - 1) / KT;
    const int n_tiles = key_tiles(TP, a.per, n_lo, n_hi);
    const int part = split * WAVES + wave, parts = a.S * WAVES;
    const int t_lo = __builtin_amdgcn_readfirstlane(key_cut(n_tiles, part, parts, a.dParts));
    const int t_hi = __builtin_amdgcn_readfirstlane(key_cut(n_tiles, part + 1, parts, a.dParts));

    const auto tile_at = [&](int t) { return key_tile<KT, D>(a, pb, kh, n_lo, TP, t); };
    WaveState<D, QB> w;
    f32_wave_loop<D, QB>(a, tile_at, t_lo, t_hi, qf, my_rollout, my_b, n_lo != n_hi, w);
    auto& o = w.o;
    auto& m_ref = w.m_ref;
    auto& limit = w.limit;
    auto& l_run = w.l_run;

    // ---- merge of the wavefronts through LDS ----------------------------------------------------------
    // (lane and thread index are worked out anew: the loop has no registers to keep them in)
    const int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), c16_e = lane_e & 15;
    const int tid_e = wave * 64 + lane_e;
    float* const so = smem;                                  // [wave][qb][t][v][lane] x 4 channels
    float* const sm = smem + F32Cfg<D, QB>::MERGE_FLOATS;        // [wave][row]: m, then the wavefront's weight
    float* const sl = sm + WAVES * RT;                       // [wave][row]: l
    float* const row_l = sl + WAVES * RT;                    // [row]: l of the workgroup
    float* const row_m = row_l + RT;                         // [row]: m of the workgroup
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        float l = l_run[qb];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (lane_e < 16) {
            sm[wave * RT + qb * 16 + c16_e] = limit[qb] == -INFINITY ? -INFINITY : m_ref[qb];
            sl[wave * RT + qb * 16 + c16_e] = l;
        }
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *reinterpret_cast<f32x4*>(so + ((((wave * QB + qb) * NT + tt) * 4 + v) * 64 + lane_e) * 4) =
                    f32x4{o[qb][tt][0][v], o[qb][tt][1][v], o[qb][tt][2][v], o[qb][tt][3][v]};
    }
    __syncthreads();
    if (tid_e < RT) {
        float m = -INFINITY, l = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) m = fmaxf(m, sm[w * RT + tid_e]);
        const float m_use = m == -INFINITY ? 0.f : m;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float x = exp2f((sm[w * RT + tid_e] - m_use) * a.c);
            l = fmaf(sl[w * RT + tid_e], x, l);
            sm[w * RT + tid_e] = x;
        }
        row_l[tid_e] = l;
        row_m[tid_e] = m;
    }
    __syncthreads();
    constexpr int CHUNKS = QB * NT * 4 * 64;      // 16-byte pieces of the row tile
#pragma unroll
    for (int i0 = 0; i0 < CHUNKS; i0 += THREADS) {
        const int i = i0 + tid_e;
        if (CHUNKS % THREADS != 0 && i >= CHUNKS) break;
        const int ln = i & 63, v = (i >> 6) & 3, tt = (i >> 8) % NT, qb = (i >> 8) / NT;
        const int r = qb * 16 + (ln & 15), row = mt * RT + r;
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(so + (w * CHUNKS + i) * 4);
            const float y = sm[w * RT + r];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaf(x[e], y, acc[e]);
        }
        if (row >= a.R) continue;
        const int ch = 64 * tt + 16 * (ln >> 4) + 4 * v;
        if (a.S == 1) {
            const int sel = fast_div(row, a.dG), g = row - sel * a.G;
            const int nb = position_of(a.qpos, sel, NB);
            const float inv = 1.f / row_l[r];
            *reinterpret_cast<f32x4*>(a.out + pb * a.o_bs + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * D + ch) = acc * inv;
        } else {
            const size_t prow = (((size_t)khv * a.MT + mt) * a.S + split) * RT + r;
            *reinterpret_cast<f32x4*>(a.ws_o + prow * D + ch) = acc;
            if (ch == 0) {
                a.ws_ml[prow * 2 + 0] = row_m[r];
                a.ws_ml[prow * 2 + 1] = row_l[r];
            }
        }
    }
#endif
}

// ---------------------------------------------------------------------------
// The same attention with products on the bf16 matrix pipe, for calls with enough rows and keys (see make_attn_plan).
//
// A float of 2^-110 and more is exactly the sum of three bf16 numbers, h + m + l with h the nearest bf16 number, m that of the
// rest and l what is left (8 bits of mantissa each).  The product of two floats is then six products of bf16 numbers, exact in the
// matrix unit's fp32 sums; what is dropped (m l', l m', l l') is at most 2^-24 (1 + 2^-10) of 2^(e + e'), the powers of two below
// the factors, where |m| reaches 2^-8 and |l| 2^-17 of theirs.  Six products at sixteen times the rate: 96 cycles of matrix
// pipe per 32 keys, 32 rows and 16 channels instead of 256.  (The method is that of Henry, Tang and Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019.)
//   Of a smaller float the last parts would lie below bf16's smallest number, 2^-133, so V is split times 2^32 and Q times 2^44:
// every part of any float is then a normal bf16 number, and results carry the inverse factor.  K is split as it is: |q| stays below
// 2^84, or its parts are infinite, and so what a product with k loses below 2^-42, even if the matrix unit took subnormal parts for
// zeros; make_attn_plan sends calls with unusual scales to the 32-row tiles.  A probability of less than 2^-110 loses up to
// 2^-126 of the row's largest, no more than the exponential itself, which is flushed to zero there.
//
// How the work is laid out
//   * A workgroup has 4 wavefronts of 32 stacked rows each (one per SIMD, 512 registers) and takes tiles of 32 keys.  Each
//     wavefront keeps its queries, split, in registers.  K and V are split once per workgroup, on their way from global memory
//     through registers into LDS: 2 slots of K [part][key][channel] (16-byte pieces XOR-swizzled by the key), 2 slots of V
//     [part][16-key step][half][channel][8 keys], the order of the probabilities in the transposed score accumulator.
//   * One step: the scores of tile i+1 (48 matrix instructions at D = 128), beside them the parts of tile i's probabilities and
//     the splitting of V of tile i+1; then P V of tile i (48), beside it the exponentials of tile i+1 and the splitting of K of
//     tile i+2, whose floats were requested a step before.  Slots of one matrix instruction and a slice of vector work, fenced, as
//     in the bf16 kernel.  A wavefront alone on its SIMD takes 5 cycles per vector instruction and 8 where one waits for the one
//     before it, so a slot carries four or five that do not: pieces of ten in every other slot cost 12 % of the time.
//   * What bounds it: N = 8, B = 32, L = 4096, Hq = 28, Hkv = 4, D = 128 takes 85.5 us a call (135.1 with fp32 products, replayed): 70 us of
//     steps, 1 290 TFLOP/s of bf16 products beside the 1 420 that a loop of nothing but this mix reaches (the chip lowers its
//     clock: 2.1 us a step with 224 workgroups, 1.8 with 56), 6 us until queries and first tiles are there, the merge.
//     Measured on the way, us for that call: queries in LDS and one slot each for K and V 97.5; in registers, where the compiler
//     copied them for every use 93.6; kept in the accumulation registers 89; and no address worked out per tile 86.5.  The factors of V and Q cost 1.5 us, as much as the
//     row of a V load in the lane's offset instead of the scalar one gave (85.9 -> 84.7, one box).  One sum for
//     all products is as fast, but rounded twelve times per tile (error against 64 bits 2.5 times as large).
//   * Values that are not finite, or become so here (|q| and scores from 2^84 on, |v| from 2^96 on): a part of an
//     infinity is a NaN, and one in a tile reaches every row of a wavefront.  A wavefront whose sums are not finite at the end does
//     its keys again with fp32 products (f32_wave_loop), so such calls give what the kernel above gives, in 1.2 to 1.9 times the
//     time of its 32-row tiles (us, 32-row tiles / these, one NaN in a prefix key: N = 8, L = 4096 148 / 240; N = 1, L = 16384 72 / 125;
//     N = 1, L = 2048 23 / 27; one infinity in a value: 144 / 244, 71 / 132, 23 / 35).
constexpr int WKT = kF32WideKeyTile, WRT = kF32WideRowTile;
constexpr float V_UP = 0x1p32f, Q_UP = 0x1p44f;      // (powers of two: no rounding but a result's own below 2^-126)

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

template <int D>
struct WideCfg {
    static constexpr int CH = D / 8;                 // 16-byte pieces of a K row (bf16)
    static constexpr int RPL = 256 / (D * 2);        // K rows per 256-byte bank line
    static constexpr int PART = WKT * D * 2;         // bytes of one part of a tile
    static constexpr int SLOT = 3 * PART;
    static constexpr int V_RING = 2 * SLOT;          // K slots, then V slots
    static constexpr int LDS_BYTES = 4 * SLOT;
    static constexpr int KV = WKT * D / 8 / 256;     // groups of 8 floats per thread and operand
    static_assert(KV >= 1, "a thread has work in every tile");
};

#define FDD_PIN(x) asm volatile("" : "+v"(x))
#define FDD_FENCE() __builtin_amdgcn_sched_barrier(0)

// The nearest bf16 numbers of two floats, packed.
__device__ __forceinline__ uint32_t round_pair(float x0, float x1)
{
    const bf16x2 b = {(__bf16)x0, (__bf16)x1};
    return __builtin_bit_cast(uint32_t, b);
}
// One part of four floats, in two pieces of about as many cycles as a matrix instruction takes: the nearest bf16 numbers, packed;
// then what is left of the floats, which replaces them.
struct SplitQuad {
    uint32_t u, w;
    float y0, y2;
    __device__ __forceinline__ void first(const float* x)
    {
        u = round_pair(x[0], x[1]);
        w = round_pair(x[2], x[3]);
        // (u << 16 by another instruction: the compiler would round the float once more instead)
        y0 = __uint_as_float(__builtin_amdgcn_perm(u, 0u, 0x05040c0cu));
        y2 = __uint_as_float(__builtin_amdgcn_perm(w, 0u, 0x05040c0cu));
        FDD_PIN(y0);
        FDD_PIN(y2);
    }
    __device__ __forceinline__ void second(float* x)
    {
        const float y1 = __uint_as_float(u & 0xffff0000u), y3 = __uint_as_float(w & 0xffff0000u);
        x[0] -= y0;
        x[2] -= y2;
        x[1] -= y1;
        x[3] -= y3;
#pragma unroll
        for (int i = 0; i < 4; ++i) FDD_PIN(x[i]);
    }
};

template <typename F, int... J>
__device__ __forceinline__ void for_each_int(F& f, std::integer_sequence<int, J...>)
{
    (f(std::integral_constant<int, J>()), ...);
}

template <int D>
__global__ __launch_bounds__(256, 1) void attn_f32_wide_kernel(Args a)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub
    using C = WideCfg<D>;
    constexpr int KS = D / 16, DB = D / 32, KV = C::KV;
    extern __shared__ __align__(16) unsigned char lds[];

    // workgroups are dealt to the 8 XCDs round-robin: those of one XCD own neighbouring row tiles of one
    // (KV head, split), which walk the same keys
    const unsigned id = wg_id_y() * a.grid_x + wg_id_x();
    const int wg = (int)(id % kNumXCD) * a.per_xcd + (int)(id / kNumXCD);
    if (wg >= a.W) return;
    const int rest = fast_div(wg, a.dMT), mt = wg - rest * a.MT;
    const int khv = fast_div(rest, a.dS), split = rest - khv * a.S;
    const int pb = fast_div(khv, a.dHkv), kh = khv - pb * a.Hkv;     // problem of the batch, KV head

    const int tid = thread_id_x(), lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NB = a.N * a.B;
    const uint32_t stride4 = (uint32_t)(a.Hkv * D * 4);     // bytes between consecutive keys

    // ---- key tiles of this workgroup: prefix tiles, then the private tiles of every rollout its rows belong to ------
    const int row_hi = min(mt * WRT + WRT, a.R) - 1;
    const int n_lo = __builtin_amdgcn_readfirstlane(fast_div(position_of(a.qpos, fast_div(mt * WRT, a.dG), NB), a.dB));
    const int n_hi = __builtin_amdgcn_readfirstlane(fast_div(position_of(a.qpos, fast_div(row_hi, a.dG), NB), a.dB));
    const int TP = (a.L + WKT - 1) / WKT;
    const int n_tiles = key_tiles(TP, a.per, n_lo, n_hi);
    const int t_lo = __builtin_amdgcn_readfirstlane(key_cut(n_tiles, split, a.S, a.dParts));
    const int t_hi = __builtin_amdgcn_readfirstlane(key_cut(n_tiles, split + 1, a.S, a.dParts));
    const auto tile_at = [&](int t) { return key_tile<WKT, D>(a, pb, kh, n_lo, TP, min(t, t_hi - 1)); };

    // ---- this thread's share of a tile: KV groups of 8 channels of a key (K), of 8 keys of a channel (V) -------------
    float raw[2 * KV][8];     // K groups, then V groups
    const auto k_key = [&](int u) { return (tid + 256 * u) / C::CH; };
    const auto v_th = [&](int u) { return (wave * 64 + 256 * u) / D; };     // 2 (16-key step) + half: the same for a wavefront
    uint32_t k_lane[KV], v_lane[KV];
#pragma unroll
    for (int u = 0; u < KV; ++u) {
        k_lane[u] = (uint32_t)k_key(u) * stride4 + (uint32_t)(tid % C::CH) * 32;
        v_lane[u] = (uint32_t)((v_th(u) >> 1) * 16 + (v_th(u) & 1) * 4) * stride4 + (uint32_t)(tid % D) * 4;
    }
    // Keys that do not exist lie beyond the buffer's end and read as zeros (their scores are masked): no address depends on the
    // tile, and no branch is needed, without which the compiler can count the loads in flight.
    // (The row is part of the lane's offset, which the range check is documented to count; of the scalar offset it is documented
    // not to, so that one stays zero.  Adding it up costs nothing, N = 8, L = 4096 85.9 -> 84.7 us; kept in 8 registers a group 84.9.
    // A plan's partials, a GiB at most, keep 32 rows of keys far below 2^32 bytes, so no sum of offsets wraps.)
    const auto tile_buffer = [&](const char* base, int valid) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, (uint32_t)(valid - 1) * stride4 + (uint32_t)(D * 4), 0x00020000);
    };
    // (in quarters: a K group is two loads, a V group eight)
    const auto request_k = [&](const KeyTile& t, int u, int quarter) {
        if (quarter % 2 != 0) return;
        const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(tile_buffer(t.k, t.valid), k_lane[u] + 8 * quarter, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) raw[u][2 * quarter + e] = x[e];
    };
    const auto request_v = [&](const KeyTile& t, int u, int quarter) {
#pragma unroll
        for (int e = 2 * quarter; e < 2 * quarter + 2; ++e)
            raw[KV + u][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                tile_buffer(t.v, t.valid), v_lane[u] + (uint32_t)((e & 3) + (e >> 2) * 8) * stride4, 0, 0));
    };
    // where a group's parts go
    uint32_t dst[2 * KV];
#pragma unroll
    for (int u = 0; u < KV; ++u) {
        const int key = k_key(u);
        dst[u] = (uint32_t)(key * D * 2 + (((tid % C::CH) ^ ((key / C::RPL) & (C::CH - 1))) << 4));
        dst[KV + u] = (uint32_t)(C::V_RING + v_th(u) * (D * 16) + (tid % D) * 16);
    }
    // Splitting a group, in 14 pieces: first, second, third parts, four floats at a time; a part of the group is written to LDS
    // when it is done.  At the end the group's floats are used up: its share of tile `next` is requested.
    u32x4 part_w[3];
    SplitQuad quad;
    constexpr int NSP = 14;
    const auto split_piece = [&](int g, int piece, uint32_t slot, const KeyTile& next) {
        const int part = piece / 4, r = 4 * ((piece / 2) % 2);
        if (part < 2) {
            if (piece % 2 == 0) {
                quad.first(&raw[g][r]);
                part_w[part][r / 2] = quad.u;
                part_w[part][r / 2 + 1] = quad.w;
            } else {
                quad.second(&raw[g][r]);
            }
        }
        if (piece == 4 || piece == 8) *reinterpret_cast<u32x4*>(lds + (dst[g] + slot) + (part - 1) * C::PART) = part_w[part - 1];
        if (piece == 8 || piece == 9) {
            const int q = 4 * (piece - 8);
            part_w[2][q / 2] = round_pair(raw[g][q], raw[g][q + 1]);
            part_w[2][q / 2 + 1] = round_pair(raw[g][q + 2], raw[g][q + 3]);
        }
        if (piece == 10) *reinterpret_cast<u32x4*>(lds + (dst[g] + slot) + 2 * C::PART) = part_w[2];
        if (piece >= 10) {
            if (g < KV) request_k(next, g, piece - 10); else request_v(next, g - KV, piece - 10);
        }
    };
    // four floats of a V group get their factor, before the group is split
    const auto scale_piece = [&](int u, int quad) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            raw[KV + u][4 * quad + e] *= V_UP;
            FDD_PIN(raw[KV + u][4 * quad + e]);
        }
    };
    const auto split_groups = [&](int first, uint32_t slot, const KeyTile& next) {
#pragma unroll
        for (int g = first; g < first + KV; ++g) {
            if (g >= KV) {
                scale_piece(g - KV, 0);
                scale_piece(g - KV, 1);
            }
#pragma unroll
            for (int piece = 0; piece < NSP; ++piece) split_piece(g, piece, slot, next);
        }
    };
    const auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };     // orders LDS traffic only

    KeyTile now = {nullptr, nullptr, 0, -1, 0}, next1 = now, next2 = now;
    const int n = t_hi - t_lo;
    if (n > 0) {
        now = tile_at(t_lo);
#pragma unroll
        for (int u = 0; u < KV; ++u)
#pragma unroll
            for (int x = 0; x < 4; ++x) request_k(now, u, x);
#pragma unroll
        for (int u = 0; u < KV; ++u)
#pragma unroll
            for (int x = 0; x < 4; ++x) request_v(now, u, x);
        FDD_FENCE();
        next1 = tile_at(t_lo + 1);
        next2 = tile_at(t_lo + 2);
    }

    // ---- the query row of this lane, split: B operand of S^T = K Q^T ---------------------------------------------------
    const int row = min(mt * WRT + wave * 32 + l32, a.R - 1);
    const bool row_ok = mt * WRT + wave * 32 + l32 < a.R;
    const int sel = fast_div(row, a.dG);
    const int nb = position_of(a.qpos, sel, NB);
    const int my_rollout = fast_div(nb, a.dB), my_b = nb - my_rollout * a.B;
    bf16x8 qf[3][KS];
    {
        const float* qp = a.q + pb * a.q_bs + ((size_t)nb * a.Hq + (size_t)kh * a.G + (row - sel * a.G)) * D + 8 * half;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const f32x4 x0 = *reinterpret_cast<const f32x4*>(qp + 16 * ks), x1 = *reinterpret_cast<const f32x4*>(qp + 16 * ks + 4);
            u32x4 w[3];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const f32x4 x = k == 0 ? x0 : x1;
                float y[4] = {x[0] * Q_UP, x[1] * Q_UP, x[2] * Q_UP, x[3] * Q_UP};
                SplitQuad sq;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    sq.first(y);
                    sq.second(y);
                    w[i][2 * k] = sq.u;
                    w[i][2 * k + 1] = sq.w;
                }
                w[2][2 * k] = round_pair(y[0], y[1]);
                w[2][2 * k + 1] = round_pair(y[2], y[3]);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                qf[i][ks] = __builtin_bit_cast(bf16x8, w[i]);
                asm volatile("" : "+a"(qf[i][ks]));      // (kept where the matrix instructions read it, not copied for each)
            }
        }
    }

    // channels 32 db + 8 (v / 4) + 4 half + v % 4 of the lane's row: sums of the products of first parts, and of all others
    // (a sum of its own for the small ones: two roundings of the large sum per tile instead of twelve)
    f32x16 o[DB], o_low[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = o_low[db][v] = 0.f;
    const float c = a.c / Q_UP, slack = a.slack * Q_UP;
    float m_ref = 0.f;             // reference the exponentials are taken against (raw score units, times Q_UP)
    float limit = -INFINITY;       // a score further above the reference raises it; -inf: there is none yet
    float l_run = 0.f;             // this lane's share of the running sum

    uint32_t k_frag0[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_frag0[ks] = (uint32_t)(l32 * D * 2 + ((((l32 / C::RPL) & (C::CH - 1)) ^ half ^ (ks << 1)) << 4));
    const uint32_t v_frag0 = (uint32_t)(C::V_RING + half * (D * 16) + l32 * 16);
    // products of two numbers, smallest first: part of K or V, part of Q or P
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};

    if (n > 0) {
        f32x16 s;                  // scores of a tile, then its probabilities
        u32x4 pw[3][2];            // the probabilities' parts, B operands of P V: [part][16-key step]
        bf16x8 f[2][3];            // fragments of K or V, those of the next six products requested during the present ones
        const auto k_frag = [&](int ks, int p, uint32_t slot) {
            return *reinterpret_cast<const bf16x8*>(lds + (k_frag0[ks] + slot) + p * C::PART);
        };
        const auto v_frag = [&](int g, int p, uint32_t slot) {       // six products g: 16-key step g / DB, channel block g % DB
            return *reinterpret_cast<const bf16x8*>(lds + (v_frag0 + slot) + p * C::PART + (g / DB) * (D * 32) + (g % DB) * 512);
        };
        // Scores of the tile in a K slot, 6 KS slots; `work(j)` is the vector work beside product j.
        const auto scores = [&](f32x16& sum, uint32_t k_slot, uint32_t v_slot, auto work) {
            constexpr int NQ = 6 * KS;
#pragma unroll
            for (int p = 0; p < 3; ++p) f[0][p] = k_frag(0, p, k_slot);
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[v] = 0.f;
            FDD_FENCE();
            const auto slot = [&](auto jc) {
                constexpr int j = decltype(jc)::value, ks = j / 6, x = j % 6;
                if constexpr (x < 3) {
                    if constexpr (ks + 1 < KS) f[(ks + 1) & 1][x] = k_frag(ks + 1, x, k_slot);
                    else f[0][x] = v_frag(0, x, v_slot);
                }
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[ks & 1][PA[x]], qf[PB[x]][ks], sum, 0, 0, 0);
                work(jc);
                FDD_FENCE();
            };
            for_each_int(slot, std::make_integer_sequence<int, NQ>());
        };
        // Softmax of tile t's scores, first half, in 25 pieces: the largest score; the reference raised if need be; the
        // exponentials (of differences to the reference, see above) and their sum.  `alpha` weighs what was summed before.
        float mx = -INFINITY, alpha = 1.f;
        bool raised = false;
        const auto mask = [&](const KeyTile& t) {
            mx = -INFINITY;
            raised = false;
            if (t.valid < WKT || t.rollout >= 0) {
                const bool sees = (t.rollout < 0) | (t.rollout == my_rollout);
                const int seen = sees ? min(t.valid, my_b - t.key0 + 1) - 4 * half : -64;
                // register v is key 8 (v / 4) + 4 half + v % 4
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = 8 * (v >> 2) + (v & 3) >= seen ? -INFINITY : s[v];
            }
        };
        constexpr int NS = 25;
        const auto softmax_piece = [&](auto pc) {
            constexpr int piece = decltype(pc)::value;
            if constexpr (piece < 8) {
                // (the larger of two numbers, in one instruction)
                mx = __builtin_amdgcn_fmed3f(mx, s[2 * piece], 3.4028235e38f);
                mx = __builtin_amdgcn_fmed3f(mx, s[2 * piece + 1], 3.4028235e38f);
                FDD_PIN(mx);
            } else if constexpr (piece == 8) {
                raised = __any(mx - m_ref > limit);
                if (raised) {
                    const bool none = limit == -INFINITY;
                    float m = fmaxf(mx, __shfl_xor(mx, 32, 64));
                    if (!none) m = fmaxf(m, m_ref);
                    alpha = none ? 1.f : exp2f((m_ref - m) * c);
                    m_ref = m == -INFINITY ? 0.f : m;
                    limit = m == -INFINITY ? m : slack;
                    l_run *= alpha;
                }
            } else {
                float x = __builtin_amdgcn_exp2f((s[piece - 9] - m_ref) * c);
                FDD_PIN(x);
                s[piece - 9] = x;
                if constexpr (piece % 2 == 0) l_run += s[piece - 10] + x;
            }
        };
        // second half, in 20 pieces: the probabilities' parts, four at a time
        SplitQuad prob;
        const auto part_piece = [&](int piece) {
            const int part = piece / 8, r = 4 * (part < 2 ? (piece / 2) % 4 : piece - 16);
            float x[4] = {s[r], s[r + 1], s[r + 2], s[r + 3]};
            if (part == 2) {
                pw[2][r / 8][(r / 2) % 4] = round_pair(x[0], x[1]);
                pw[2][r / 8][(r / 2) % 4 + 1] = round_pair(x[2], x[3]);
            } else if (piece % 2 == 0) {
                prob.first(x);
                pw[part][r / 8][(r / 2) % 4] = prob.u;
                pw[part][r / 8][(r / 2) % 4 + 1] = prob.w;
            } else {
                prob.second(x);
#pragma unroll
                for (int i = 0; i < 4; ++i) s[r + i] = x[i];
            }
        };

        // ---- tile 0 into LDS, its scores, first half of its softmax; K of tile 1 into LDS ------------------------------------
        split_groups(0, 0, next1);
        split_groups(KV, 0, next1);
        barrier();
        scores(s, 0, 0, [](auto) {});
        if (n > 1) split_groups(0, C::SLOT, next2);
        mask(now);
        for_each_int(softmax_piece, std::make_integer_sequence<int, NS>());
        barrier();

        // ---- one step ------------------------------------------------------------------------------------------------------
        //   scores of tile i+1   ||  parts of tile i's probabilities, V of tile i+1 split into LDS
        //   P V of tile i        ||  first half of the softmax of tile i+1, K of tile i+2 split into LDS
        // (the last step has no tile i+1)
        const auto step = [&](auto more, int i) {
            constexpr bool MORE = decltype(more)::value;
            const uint32_t even = (i & 1) ? (uint32_t)C::SLOT : 0u, odd = (uint32_t)C::SLOT - even;    // slots of tile i, of tile i+1
            f32x16 s_next;
            KeyTile next3 = next2;
            if constexpr (MORE) next3 = tile_at(t_lo + i + 3);
            const auto beside_scores = [&](auto jc) {
                // (splitting in the odd slots, softmax in the even ones: what a slot carries must not outlast its matrix instruction)
                // (and the factors of V: of a group's two quads right before its first and third piece)
                constexpr int j = decltype(jc)::value, h = j / 2, NQ = 3 * KS, NV = NSP * KV, NX = 20 + 2 * KV, XG = NX / KV;
                if constexpr (j % 2 == 1) {
                    if constexpr (MORE) {
#pragma unroll
                        for (int w = h * NV / NQ; w < (h + 1) * NV / NQ; ++w) split_piece(KV + w / NSP, w % NSP, odd, next2);
                    }
                } else {
#pragma unroll
                    for (int w = h * NX / NQ; w < (h + 1) * NX / NQ; ++w) {
                        if (w % XG >= 2) part_piece(w - 2 * (w / XG + 1));
                        else if constexpr (MORE) scale_piece(w / XG, w % XG);
                    }
                }
            };
            if constexpr (MORE) {
                scores(s_next, odd, even, beside_scores);
                s = s_next;
                mask(next1);
            } else {
#pragma unroll
                for (int p = 0; p < 3; ++p) f[0][p] = v_frag(0, p, even);
                for_each_int(beside_scores, std::make_integer_sequence<int, 6 * KS>());
            }
            FDD_FENCE();
            constexpr int NP = 12 * DB;
            const auto slot = [&](auto jc) {
                constexpr int j = decltype(jc)::value, g = j / 6, x = j % 6;
                if constexpr (x < 3 && g + 1 < 2 * DB) f[(g + 1) & 1][x] = v_frag(g + 1, x, even);
                f32x16& sum = x == 5 ? o[g % DB] : o_low[g % DB];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[g & 1][PA[x]], __builtin_bit_cast(bf16x8, pw[PB[x]][g / DB]), sum, 0, 0, 0);
                if constexpr (MORE) {
                    constexpr int h = j / 2, NH = NP / 2, NK = NSP * KV;
                    if constexpr (j % 2 == 1) {
#pragma unroll
                        for (int w = h * NK / NH; w < (h + 1) * NK / NH; ++w) split_piece(w / NSP, w % NSP, even, next3);
                    } else {
                        const auto piece = [&](auto wc) { softmax_piece(std::integral_constant<int, h * NS / NH + decltype(wc)::value>()); };
                        for_each_int(piece, std::make_integer_sequence<int, (h + 1) * NS / NH - h * NS / NH>());
                    }
                }
                FDD_FENCE();
            };
            for_each_int(slot, std::make_integer_sequence<int, NP>());
            if constexpr (MORE) {
                barrier();
                next1 = next2;
                next2 = next3;
            }
        };
        // (a loop of its own around the steps that raise no reference: the sums stay where the matrix instructions keep them)
        for (int i = 0; i + 1 < n;) {
            do {
                step(std::true_type(), i);
                ++i;
            } while (i + 1 < n && !raised);
            if (raised) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        o[db][v] *= alpha;
                        o_low[db][v] *= alpha;
                    }
            }
        }
        step(std::false_type(), n - 1);
    }

    // ---- epilogue --------------------------------------------------------------------------------------------------------
    const size_t pseg = (((size_t)khv * a.MT + mt) * a.S + split) * WRT;      // first row of this workgroup's partial results
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    float x0 = l_tot * 0.f;      // NaN if any sum is not finite
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            o[db][v] += o_low[db][v];
            x0 = fmaf(o[db][v], 0.f, x0);
        }
    // Partial results lie in the order of the accumulator registers, [wavefront][db][v / 4][lane] x 4 floats, so that a store
    // writes 1 KB in one piece, and are written through to memory (aux 16 = device scope): the merge kernel's workgroups sit
    // on other XCDs, and lines left dirty in the L2s go out only when the launch has ended.
    const __amdgpu_buffer_rsrc_t part_rsrc = __builtin_amdgcn_make_buffer_rsrc(a.ws_o + pseg * D, 0, WRT * D * 4, 0x00020000);
    const uint32_t part0 = (uint32_t)(wave * 32 * D * 4);
    // A row that sees a key (prefix keys, or those of its own rollout up to where the causal mask ends) and has no reference: all
    // of its scores were -2^84 and less.  (Fewer such scores weigh nothing: they are 2^60 and more below the others.)
    const int own = TP + (my_rollout - n_lo) * a.per, own_end = own + (a.causal ? a.ext_per + my_b / WKT + 1 : a.per);
    if ((t_lo < t_hi && t_lo < TP || max(t_lo, own) < min(t_hi, own_end)) && limit == -INFINITY) x0 = NAN;
    if (__builtin_expect(!__any(x0 != 0.f), 1)) {
        if (!row_ok) return;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const f32x4 x = f32x4{o[db][4 * v4], o[db][4 * v4 + 1], o[db][4 * v4 + 2], o[db][4 * v4 + 3]} / V_UP;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), part_rsrc, part0 + (db * 4 + v4) * 1024 + lane * 16, 0, 16);
            }
        if (half == 0) {
            float* const ml = a.ws_ml + (pseg + wave * 32 + l32) * 2;
            ml[0] = limit == -INFINITY ? -INFINITY : m_ref / Q_UP;
            ml[1] = l_tot;
        }
        return;
    }
    // ---- the wavefront's keys again, with fp32 products --------------------------------------------------------------------
    {
        constexpr int NT = D / 64;
        const int c16 = lane & 15, g4 = lane >> 4;
        f32x4 q16[2][D / 16];
        int rollout16[2], b16[2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            const int r = min(mt * WRT + wave * 32 + qb * 16 + c16, a.R - 1);
            const int e = fast_div(r, a.dG), pos = position_of(a.qpos, e, NB);
            rollout16[qb] = fast_div(pos, a.dB);
            b16[qb] = pos - rollout16[qb] * a.B;
            const float* qp = a.q + pb * a.q_bs + ((size_t)pos * a.Hq + (size_t)kh * a.G + (r - e * a.G)) * D + 4 * g4;
#pragma unroll
            for (int j = 0; j < D / 16; ++j) q16[qb][j] = *reinterpret_cast<const f32x4*>(qp + 16 * j);
        }
        const auto half_tile = [&](int t) {       // 16 keys of a tile; none of them may exist
            KeyTile r = tile_at(t >> 1);
            if (t & 1) {
                const bool any = r.valid > 16;
                if (any) {
                    r.k += 16 * (size_t)stride4;
                    r.v += 16 * (size_t)stride4;
                }
                r.valid = any ? r.valid - 16 : 0;
                r.key0 += 16;
            }
            r.valid = min(r.valid, 16);
            return r;
        };
        WaveState<D, 2> w;
        f32_wave_loop<D, 2>(a, half_tile, 2 * t_lo, 2 * t_hi, q16, rollout16, b16, n_lo != n_hi, w);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            float l = w.l_run[qb];
            l += __shfl_xor(l, 16, 64);
            l += __shfl_xor(l, 32, 64);
            const int r = wave * 32 + qb * 16 + c16;
            if (mt * WRT + r >= a.R) continue;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const f32x4 x = f32x4{w.o[qb][t][0][v], w.o[qb][t][1][v], w.o[qb][t][2][v], w.o[qb][t][3][v]};
                    const int ch = 64 * t + 16 * g4 + 4 * v;
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), part_rsrc,
                                                           part0 + (ch / 8) * 1024 + ((ch / 4) % 2 * 32 + qb * 16 + c16) * 16, 0, 16);
                }
            if (g4 == 0) {
                a.ws_ml[(pseg + r) * 2 + 0] = w.limit[qb] == -INFINITY ? -INFINITY : w.m_ref[qb];
                a.ws_ml[(pseg + r) * 2 + 1] = l;
            }
        }
    }
#endif
}

// ---------------------------------------------------------------------------
// Merge of the splits' partials (log-sum-exp merge):
//   m* = max_s m_s,  w_s = 2^((m_s - m*) c),  out = sum_s w_s o_s / sum_s w_s l_s
// The sum runs over s in a fixed order, so results are reproducible.
struct CombineArgs {
    const float* ws_o;
    const float* ws_ml;
    float* out;
    int Hq, Hkv, G, R, MT, mrows, D;
    long long o_bs;  // elements between the outputs of the problems of a batch
    int n_seg;       // splits, at least 2
    int SG;          // segment groups: the segments of a row are shared out over SG threads per channel quad
    int RB;          // rows per block; RB * SG * D/4 = 256 threads
    float c;
    const int32_t* qpos;   // list of query positions, as in the attention kernels, or nullptr
    int NB;                // N * B
};

// grid (Hkv*MT, ceil(mrows / RB)).  Thread (r, sg, d4) sums segments sg, sg+SG, ..
// of row r for 4 channels, four loads in flight at a time; the SG partial sums
// are then added in the order sg = 0, 1, .. by the thread with sg = 0.
__global__ __launch_bounds__(256) void attn_combine_kernel(CombineArgs a)
{
    extern __shared__ __align__(16) float smem[];
    const int d4n = a.D / 4;
    const int tid = (int)thread_id_x();
    const int d4 = tid % d4n, sg = (tid / d4n) % a.SG, r = tid / (d4n * a.SG);
    const int M = (int)wg_id_x();
    const int khv = M / a.MT, mt = M - khv * a.MT;      // (problem of the batch, KV head), M-tile
    const int pb = khv / a.Hkv, kh = khv - pb * a.Hkv;
    const int rit0 = (int)wg_id_y() * a.RB;
    const int n_seg = a.n_seg;
    if (a.SG == 1 && n_seg <= 4) {
        // few segments: every thread reads the (m, l) pairs of its row itself, together with its
        // partial outputs, in one round trip to memory and without LDS (same sums, same order)
        const int rit = rit0 + r;
        const int row = mt * a.mrows + rit;
        if (rit >= a.mrows || row >= a.R) return;
        const size_t prow = ((size_t)M * a.n_seg) * a.mrows + rit;
        float2 ml[4];
        float4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ml[u] = make_float2(-INFINITY, 0.f);
            x[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (u < n_seg) {
                ml[u] = *reinterpret_cast<const float2*>(a.ws_ml + (prow + (size_t)u * a.mrows) * 2);
                x[u] = *reinterpret_cast<const float4*>(a.ws_o + (prow + (size_t)u * a.mrows) * a.D + d4 * 4);
            }
        }
        float mstar = -INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u) mstar = fmaxf(mstar, ml[u].x);
        float l = 0.f;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u < n_seg) {
                const float w = exp2f((ml[u].x - mstar) * a.c);
                l = fmaf(ml[u].y, w, l);
                acc.x = fmaf(x[u].x, w, acc.x);
                acc.y = fmaf(x[u].y, w, acc.y);
                acc.z = fmaf(x[u].z, w, acc.z);
                acc.w = fmaf(x[u].w, w, acc.w);
            }
        }
        const float inv = 1.f / l;
        const int sel = row / a.G, g = row - sel * a.G;
        const int nb = position_of(a.qpos, sel, a.NB);
        const size_t off = (size_t)(pb * a.o_bs) + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * a.D + d4 * 4;
        *reinterpret_cast<float4*>(a.out + off) =
            make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
        return;
    }
    float* const sm = smem;                           // [RB][n_seg] segment maxima
    float* const sl = smem + a.RB * n_seg;            // [RB][n_seg] segment sums
    float4* const red = reinterpret_cast<float4*>(smem + ((2 * a.RB * a.n_seg + 3) & ~3));   // [RB][SG][d4n]
    float* const redl = reinterpret_cast<float*>(red + a.RB * a.SG * d4n);        // [RB][SG]
    const size_t p0 = ((size_t)M * a.n_seg) * a.mrows + rit0;
    for (int i = tid; i < a.RB * n_seg; i += 256) {
        const int rr = i / n_seg, s = i - rr * n_seg;
        float m = -INFINITY, l = 0.f;
        if (rit0 + rr < a.mrows) {
            const float2 ml = *reinterpret_cast<const float2*>(a.ws_ml + (p0 + rr + (size_t)s * a.mrows) * 2);
            m = ml.x;
            l = ml.y;
        }
        sm[i] = m;
        sl[i] = l;
    }
    __syncthreads();
    const int rit = rit0 + r;
    const int row = mt * a.mrows + rit;
    const bool live = rit < a.mrows && row < a.R;
    float mstar = -INFINITY;
    for (int s = 0; s < n_seg; ++s) mstar = fmaxf(mstar, sm[r * n_seg + s]);
    float l = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live) {
        const float* src = a.ws_o + (p0 + r) * a.D + d4 * 4;
        const size_t seg_stride = (size_t)a.mrows * a.D;
        for (int s0 = sg; s0 < n_seg; s0 += 4 * a.SG) {
            float4 x[4];
            float w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int s = s0 + u * a.SG;
                x[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                w[u] = 0.f;
                if (s < n_seg) {
                    x[u] = *reinterpret_cast<const float4*>(src + (size_t)s * seg_stride);
                    w[u] = exp2f((sm[r * n_seg + s] - mstar) * a.c);
                    l = fmaf(sl[r * n_seg + s], w[u], l);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc.x = fmaf(x[u].x, w[u], acc.x);
                acc.y = fmaf(x[u].y, w[u], acc.y);
                acc.z = fmaf(x[u].z, w[u], acc.z);
                acc.w = fmaf(x[u].w, w[u], acc.w);
            }
        }
    }
    if (a.SG > 1) {
        red[(r * a.SG + sg) * d4n + d4] = acc;
        if (d4 == 0) redl[r * a.SG + sg] = l;
        __syncthreads();
        if (sg != 0) return;
        acc = red[(r * a.SG) * d4n + d4];
        l = redl[r * a.SG];
        for (int k = 1; k < a.SG; ++k) {
            const float4 y = red[(r * a.SG + k) * d4n + d4];
            acc.x += y.x;
            acc.y += y.y;
            acc.z += y.z;
            acc.w += y.w;
            l += redl[r * a.SG + k];
        }
    }
    if (!live) return;
    const float inv = 1.f / l;
    const int sel = row / a.G, g = row - sel * a.G;
    const int nb = position_of(a.qpos, sel, a.NB);
    const size_t off = (size_t)(pb * a.o_bs) + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * a.D + d4 * 4;
    *reinterpret_cast<float4*>(a.out + off) =
        make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
}

// The same merge for the partials of attn_f32_wide_kernel, which lie in accumulator order.  A thread takes one 16-byte chunk
// (4 channels of a row) of every SG-th segment, and the SG threads of a chunk, lanes of one wavefront, meet in lane moves.
// grid (Hkv*MT, chunks of a row tile * SG / 256)
struct WideMergeArgs {
    const float* ws_o;
    const float* ws_ml;
    float* out;
    const int32_t* qpos;
    long long o_bs;
    int Hq, G, R, NB, S;
    FastDiv dMT, dHkv, dG;
    int MT, Hkv;
    float c;
};

template <int D, int SG>
__global__ __launch_bounds__(256) void attn_wide_merge_kernel(WideMergeArgs a)
{
    constexpr int CPL = 64 / SG, UX = 4;             // chunks per wavefront, segments requested together
    const int tid = (int)thread_id_x(), lane = tid & 63, sg = lane / CPL;
    const int M = (int)wg_id_x();
    const int khv = fast_div(M, a.dMT), mt = M - khv * a.MT;      // (problem of the batch, KV head), M-tile
    const int pb = fast_div(khv, a.dHkv), kh = khv - pb * a.Hkv;
    // chunk: [wavefront of 32 rows][channel / 8][channel / 4 % 2][row]
    const int chunk = ((int)wg_id_y() * 4 + (tid >> 6)) * CPL + lane % CPL;
    const int r = chunk / (8 * D) * 32 + (chunk & 31), ch = (chunk / 32) % (D / 4) * 4;
    const int row = mt * WRT + r;
    const bool live = row < a.R;
    const f32x4* src = reinterpret_cast<const f32x4*>(a.ws_o) + (size_t)M * a.S * (WRT * D / 4) + chunk;
    const float* ml = a.ws_ml + ((size_t)M * a.S * WRT + r) * 2;
    float m = -INFINITY, l = 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    if (live)
        for (int s0 = sg; s0 < a.S; s0 += SG * UX) {
            float2 y[UX];
            f32x4 x[UX];
#pragma unroll
            for (int u = 0; u < UX; ++u) {
                const int s = s0 + u * SG;
                y[u] = make_float2(-INFINITY, 0.f);
                x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (s < a.S) {
                    y[u] = *reinterpret_cast<const float2*>(ml + (size_t)s * (2 * WRT));
                    x[u] = src[(size_t)s * (WRT * D / 4)];
                }
            }
            __builtin_amdgcn_sched_barrier(0);    // everything is requested before anything is waited for
            float mx = m;
#pragma unroll
            for (int u = 0; u < UX; ++u) mx = fmaxf(mx, y[u].x);
            // (Where no segment so far has a reference, its sums are zero, or NaN, for no score that is NaN raises a reference:
            // weights of zero keep both.)
            const float m_use = mx == -INFINITY ? 0.f : mx;
            const float old = exp2f((m - m_use) * a.c);
            m = mx;
            l *= old;
            acc *= old;
#pragma unroll
            for (int u = 0; u < UX; ++u) {
                const float w = exp2f((y[u].x - m_use) * a.c);
                l = fmaf(y[u].y, w, l);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = fmaf(x[u][e], w, acc[e]);
            }
        }
    if (SG > 1) {
        float mx = m;
#pragma unroll
        for (int d = CPL; d < 64; d *= 2) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
        const float w = m == -INFINITY ? 0.f : exp2f((m - mx) * a.c);
        l *= w;
        acc *= w;
#pragma unroll
        for (int d = CPL; d < 64; d *= 2) {
            l += __shfl_xor(l, d, 64);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], d, 64);
        }
    }
    if (!live || sg != 0) return;
    const int sel = fast_div(row, a.dG), g = row - sel * a.G;
    const int nb = position_of(a.qpos, sel, a.NB);
    *reinterpret_cast<f32x4*>(a.out + pb * a.o_bs + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * D + ch) = acc * (1.f / l);
}

}  // namespace

template <typename Kernel>
static hipError_t launch(Kernel kern, int threads, int lds_bytes, std::atomic<uint64_t>& done, const Args& a, hipStream_t s)
{
    // the LDS limit of this instantiation is raised once per device (bit d of `done`: device d)
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(done.load(std::memory_order_acquire) & bit)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, f32_grid(a.W), dim3(threads), lds_bytes, s, a);
    return hipGetLastError();
}

template <int D>
static hipError_t launch(const Args& a, int rows, hipStream_t s)
{
    static std::atomic<uint64_t> done{0}, done_few{0}, done_wide{0};
    if (rows == WRT) return launch(&attn_f32_wide_kernel<D>, 256, WideCfg<D>::LDS_BYTES, done_wide, a, s);
    if (rows == kF32FewRowTile) return launch(&attn_f32_kernel<D, 1>, THREADS, F32Cfg<D, 1>::LDS_BYTES, done_few, a, s);
    return launch(&attn_f32_kernel<D, 2>, THREADS, F32Cfg<D, 2>::LDS_BYTES, done, a, s);
}

hipError_t launch_attn_f32(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s)
{
    Args a;
    a.q = static_cast<const float*>(p.q);
    a.pk = static_cast<const float*>(p.prefix_k);
    a.pv = static_cast<const float*>(p.prefix_v);
    a.bk = static_cast<const float*>(p.block_k);
    a.bv = static_cast<const float*>(p.block_v);
    a.out = static_cast<float*>(p.out);
    a.ws_o = static_cast<float*>(p.workspace);
    a.ws_ml = reinterpret_cast<float*>(static_cast<char*>(p.workspace) + plan.ws_o_bytes);
    a.ek = static_cast<const float*>(p.ext_k);
    a.ev = static_cast<const float*>(p.ext_v);
    a.E = p.E; a.Ecap = p.ext_capacity;
    const int batch = p.batch > 1 ? p.batch : 1;
    a.q_bs = p.q_batch_stride; a.p_bs = p.prefix_batch_stride; a.b_bs = p.block_batch_stride;
    a.e_bs = p.ext_batch_stride; a.o_bs = p.out_batch_stride;
    a.N = p.N; a.B = p.B; a.L = p.L; a.Hq = p.Hq; a.Hkv = p.Hkv;
    a.G = plan.G; a.R = plan.R; a.MT = plan.MT; a.S = plan.splits;
    a.W = p.Hkv * batch * plan.MT * plan.splits;
    const dim3 grid = f32_grid(a.W);
    a.grid_x = grid.x;
    a.per_xcd = (int)(grid.x * grid.y / kNumXCD);
    a.c = scale * 1.4426950408889634f;
    a.slack = 8.f / a.c;
    a.causal = (p.flags & FDD_ATTN_CAUSAL_BLOCK) ? 1 : 0;
    a.qpos = p.n_q_positions > 0 ? p.q_positions : nullptr;
    const bool wide = plan.mtile_rows == WRT;
    if (!wide && plan.mtile_rows != kF32RowTile && plan.mtile_rows != kF32FewRowTile) return hipErrorInvalidValue;
    if (wide && plan.splits < 2) return hipErrorInvalidValue;      // (it leaves partial results)
    if (plan.key_tile != (wide ? WKT : KT)) return hipErrorInvalidValue;
    a.ext_per = (p.E + plan.key_tile - 1) / plan.key_tile;
    a.per = a.ext_per + (p.B + plan.key_tile - 1) / plan.key_tile;
    a.dMT = make_fastdiv((uint32_t)a.MT);
    a.dS = make_fastdiv((uint32_t)a.S);
    a.dHkv = make_fastdiv((uint32_t)a.Hkv);
    a.dG = make_fastdiv((uint32_t)a.G);
    a.dB = make_fastdiv((uint32_t)a.B);
    a.dPer = make_fastdiv((uint32_t)a.per);
    a.dParts = make_fastdiv((uint32_t)(a.S * (wide ? 1 : WAVES)));     // wavefronts or workgroups that share the keys
    return p.D == 128 ? launch<128>(a, plan.mtile_rows, s) : launch<64>(a, plan.mtile_rows, s);
}

hipError_t launch_attn_combine(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s)
{
    if (plan.mtile_rows == WRT) {
        WideMergeArgs a;
        a.ws_o = static_cast<const float*>(p.workspace);
        a.ws_ml = reinterpret_cast<const float*>(static_cast<const char*>(p.workspace) + plan.ws_o_bytes);
        a.out = static_cast<float*>(p.out);
        a.qpos = p.n_q_positions > 0 ? p.q_positions : nullptr;
        a.o_bs = p.out_batch_stride;
        a.Hq = p.Hq; a.G = plan.G; a.R = plan.R; a.NB = p.N * p.B; a.S = plan.splits; a.MT = plan.MT; a.Hkv = p.Hkv;
        a.dMT = make_fastdiv((uint32_t)a.MT);
        a.dHkv = make_fastdiv((uint32_t)a.Hkv);
        a.dG = make_fastdiv((uint32_t)a.G);
        a.c = scale * 1.4426950408889634f;
        const unsigned tiles = (unsigned)(p.Hkv * (p.batch > 1 ? p.batch : 1) * plan.MT);
        // (several threads per chunk where each would take more than two rounds of loads)
        const int sg = a.S > 16 ? 4 : a.S > 8 ? 2 : 1;
        auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(tiles, (unsigned)(WRT * p.D / 4 * sg / 256)), dim3(256), 0, s, a); };
        if (p.D == 128) sg == 4 ? go(&attn_wide_merge_kernel<128, 4>) : sg == 2 ? go(&attn_wide_merge_kernel<128, 2>) : go(&attn_wide_merge_kernel<128, 1>);
        else sg == 4 ? go(&attn_wide_merge_kernel<64, 4>) : sg == 2 ? go(&attn_wide_merge_kernel<64, 2>) : go(&attn_wide_merge_kernel<64, 1>);
        return hipGetLastError();
    }
    CombineArgs a;
    a.ws_o = static_cast<const float*>(p.workspace);
    a.ws_ml = reinterpret_cast<const float*>(static_cast<const char*>(p.workspace) + plan.ws_o_bytes);
    a.out = static_cast<float*>(p.out);
    const int batch = p.batch > 1 ? p.batch : 1;
    a.Hq = p.Hq; a.Hkv = p.Hkv; a.G = plan.G; a.R = plan.R; a.MT = plan.MT;
    a.o_bs = p.out_batch_stride;
    a.qpos = p.n_q_positions > 0 ? p.q_positions : nullptr;
    a.NB = p.N * p.B;
    a.mrows = plan.mtile_rows; a.D = p.D;
    a.n_seg = plan.splits;
    a.c = scale * 1.4426950408889634f;
    // more threads per row when the rows are few and the segments many
    const long long rows = (long long)p.Hkv * batch * plan.R;
    int sg = 1;
    while (sg < 8 && sg * 2 <= plan.splits && rows * sg < 16384) sg *= 2;
    a.SG = sg;
    a.RB = 256 / (sg * (p.D / 4));
    const size_t smem = (size_t)((2 * a.RB * plan.splits + 3) & ~3) * sizeof(float) + (size_t)a.RB * sg * (p.D / 4) * sizeof(float4) +
                        (size_t)a.RB * sg * sizeof(float);
    if (smem > 60 * 1024) return hipErrorInvalidValue;
    const dim3 grid(p.Hkv * batch * plan.MT, (plan.mtile_rows + a.RB - 1) / a.RB);
    hipLaunchKernelGGL(attn_combine_kernel, grid, dim3(256), smem, s, a);
    return hipGetLastError();
}

}  // namespace fdd
