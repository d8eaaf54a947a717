// Shared-prefix block-causal attention, fp32 storage and arithmetic, and the
// merge of its splits.
//
// The same thing as the bf16 kernel computes (paper, "Block-Causal Diffusion"
// and "Shared prefix"), with fp32 products and sums on the matrix cores
// (v_mfma_f32_16x16x4_f32).
//
// How the work is laid out
//   * A workgroup owns 32 stacked query rows of one KV head (see AttnPlan); its
//     8 wavefronts share the KEYS out among themselves, 16 at a time, each with
//     a streaming-softmax state (m, l, o) of its own, and merge through LDS at
//     the end.  `splits` workgroups share one row tile when the row tiles alone
//     leave the chip idle; then a second small kernel merges their partials.
//   * S^T = K Q^T: a lane owns query lane % 16 of each of two 16-query blocks and
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
//   * Measured at N = 8, B = 32, L = 4096, Hq = 28, Hkv = 4, D = 128 (15.1 GFLOP): 135 us
//     in a loop of nothing else, 112 TFLOP/s of the 154 a large fp32 matrix product
//     reaches here, and 149 us among the other kernels of a denoise step; 224 of 256
//     CUs are used, the matrix pipe of a used CU 84 % of its cycles (loop of nothing
//     else).  Scalar fused multiply-adds from LDS tiles: 687 us in a denoise step.  Not
//     faster, when the kernel took 152 us there: K through a private LDS ring, the next
//     tile's scores under this tile's exponentials, priorities that keep the two
//     wavefronts of a SIMD level (157 us each).
#include "fdd_internal.h"

#include <atomic>

namespace fdd {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KT = 16;                 // keys per tile
constexpr int RT = kF32RowTile;        // rows per workgroup: two 16-query blocks
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

template <int D>
struct F32Cfg {
    static constexpr int MERGE_FLOATS = WAVES * RT * D;   // outputs of all wavefronts, in register order
    static constexpr int LDS_BYTES = (MERGE_FLOATS + 2 * WAVES * RT + 2 * RT) * 4;   // + (m, l) per wavefront and row, and per row
};

template <int D>
__global__ __launch_bounds__(THREADS) void attn_f32_kernel(Args a)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub
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
    const uint32_t stride4 = (uint32_t)(a.Hkv * D * 4);     // bytes between consecutive keys

    // ---- query rows of this lane: c16 of both 16-query blocks --------------------------------------
    f32x4 qf[2][NJ];
    int my_rollout[2], my_b[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
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
    const int n_tiles = TP + (n_hi - n_lo + 1) * a.per;
    const int part = split * WAVES + wave, parts = a.S * WAVES;
    const int t_lo = __builtin_amdgcn_readfirstlane(key_cut(n_tiles, part, parts, a.dParts));
    const int t_hi = __builtin_amdgcn_readfirstlane(key_cut(n_tiles, part + 1, parts, a.dParts));

    struct Tile {
        const char* k;    // first key's row of this KV head
        const char* v;
        int valid;        // keys that exist
        int rollout;      // whose rows may see it (-1: every row)
        int key0;         // block position of the first key (block tiles under the causal mask), else hugely negative
    };
    auto tile_at = [&](int t) {
        Tile r;
        long long row;
        long long bs;
        const float *kp, *vp;
        r.key0 = -(1 << 30);
        if (t < TP) {
            kp = a.pk; vp = a.pv; bs = a.p_bs;
            row = (long long)t * KT;
            r.valid = min(KT, a.L - t * KT);
            r.rollout = -1;
        } else {
            const int j = t - TP, i = fast_div(j, a.dPer), w = j - i * a.per;
            r.rollout = n_lo + i;
            if (w < a.ext_per) {
                kp = a.ek; vp = a.ev; bs = a.e_bs;
                row = (long long)r.rollout * a.Ecap + w * KT;
                r.valid = min(KT, a.E - w * KT);
            } else {
                const int k0 = (w - a.ext_per) * KT;
                kp = a.bk; vp = a.bv; bs = a.b_bs;
                row = (long long)r.rollout * a.B + k0;
                r.valid = min(KT, a.B - k0);
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
    };

    // Fragments of a tile.  K: row c16, channels 16 j + 4 g4 ..; V: row 4 g4 + v, channels 64 t + 4 c16 ..
    // (rows beyond `valid` repeat the last valid one: masked below, nothing read out of bounds)
    f32x4 kf[NJ], vf[NJ];
    auto k_off = [&](const Tile& t) { return (uint32_t)min(c16, t.valid - 1) * stride4 + (uint32_t)(16 * g4); };
    auto v_off = [&](const Tile& t, int v) { return (uint32_t)min(4 * g4 + v, t.valid - 1) * stride4 + (uint32_t)(16 * c16); };
    // (offsets inside a tile stay below 2^32, as the whole block K does, but may pass 2^31 with very many KV heads)
    auto load = [&](const char* base, uint32_t off) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, -1, 0x00020000);
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
    };

    f32x4 o[2][NT][4];       // [query block][64-channel block][e]: channels 64 t + 16 g4 + 4 v + e of query c16
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[qb][t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_ref[2] = {0.f, 0.f};               // reference the exponentials are taken against (raw score units)
    float limit[2] = {-INFINITY, -INFINITY};   // a score further above the reference raises it; -inf: there is none yet
    float l_run[2] = {0.f, 0.f};               // this lane's share of the running sum

    if (t_lo < t_hi) {
        Tile now = tile_at(t_lo);
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
            const Tile next = tile_at(min(t + 1, t_hi - 1));
            const uint32_t next_k = k_off(next);
            f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb)
                        s[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][i], qf[qb][j][i], s[qb], 0, 0, 0);
                kf[j] = load(next.k, next_k + 64 * j);
                __builtin_amdgcn_sched_barrier(0);
            }
            // register v of a query block is key 4 g4 + v
            if (now.valid < KT || now.rollout >= 0) {
#pragma unroll
                for (int qb = 0; qb < 2; ++qb)
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
            f32x4 p[2];
            bool need = false;
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
                for (int v = 0; v < 4; ++v) p[qb][v] = s[qb][v] - m_ref[qb];
                need |= fmaxf(fmaxf(p[qb][0], p[qb][1]), fmaxf(p[qb][2], p[qb][3])) > limit[qb];
            }
            if (__any(need)) {
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
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
            for (int qb = 0; qb < 2; ++qb) {
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
            if (now.rollout >= 0 && n_lo != n_hi) {
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
                            for (int qb = 0; qb < 2; ++qb) {
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
                        for (int qb = 0; qb < 2; ++qb)
                            o[qb][tt][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v * NT + tt][e], p[qb][v], o[qb][tt][e], 0, 0, 0);
                    vf[v * NT + tt] = load(next.v, next_v + 256 * tt);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            now = next;
        }
    }

    // ---- merge of the wavefronts through LDS ----------------------------------------------------------
    // (lane and thread index are worked out anew: the loop has no registers to keep them in)
    const int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), c16_e = lane_e & 15;
    const int tid_e = wave * 64 + lane_e;
    float* const so = smem;                                  // [wave][qb][t][v][lane] x 4 channels
    float* const sm = smem + F32Cfg<D>::MERGE_FLOATS;        // [wave][row]: m, then the wavefront's weight
    float* const sl = sm + WAVES * RT;                       // [wave][row]: l
    float* const row_l = sl + WAVES * RT;                    // [row]: l of the workgroup
    float* const row_m = row_l + RT;                         // [row]: m of the workgroup
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
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
                *reinterpret_cast<f32x4*>(so + ((((wave * 2 + qb) * NT + tt) * 4 + v) * 64 + lane_e) * 4) =
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
    constexpr int CHUNKS = 2 * NT * 4 * 64;      // 16-byte pieces of the row tile
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

}  // namespace

template <int D>
static hipError_t launch(const Args& a, hipStream_t s)
{
    const auto kern = &attn_f32_kernel<D>;
    // the LDS limit of this instantiation is raised once per device (bit d of `done`: device d)
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(done.load(std::memory_order_acquire) & bit)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           F32Cfg<D>::LDS_BYTES);
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, f32_grid(a.W), dim3(THREADS), F32Cfg<D>::LDS_BYTES, s, a);
    return hipGetLastError();
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
    a.ext_per = (p.E + KT - 1) / KT;
    a.per = a.ext_per + (p.B + KT - 1) / KT;
    a.dMT = make_fastdiv((uint32_t)a.MT);
    a.dS = make_fastdiv((uint32_t)a.S);
    a.dHkv = make_fastdiv((uint32_t)a.Hkv);
    a.dG = make_fastdiv((uint32_t)a.G);
    a.dB = make_fastdiv((uint32_t)a.B);
    a.dPer = make_fastdiv((uint32_t)a.per);
    a.dParts = make_fastdiv((uint32_t)(a.S * WAVES));
    if (plan.mtile_rows != RT || plan.key_tile != KT) return hipErrorInvalidValue;
    return p.D == 128 ? launch<128>(a, s) : launch<64>(a, s);
}

hipError_t launch_attn_combine(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s)
{
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
