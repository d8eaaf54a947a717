// Internal declarations shared by the library's translation units (not part
// of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fdd.h"

namespace fdd {

// Thread and workgroup index, high half of a 32 x 32 bit product.  threadIdx, blockIdx, gridDim and __umulhi go through
// functions of the device library that were compiled for another floating-point mode than the files built with
// -mno-amdgpu-ieee, and the compiler does not inline across that difference: each use is a call (a cold one at the top
// of every workgroup), its result is not known to be the same in all lanes, and the sampler made 40 calls per four
// entries.  The builtins are single registers and instructions.
__device__ __forceinline__ int thread_id_x() { return (int)__builtin_amdgcn_workitem_id_x(); }
__device__ __forceinline__ unsigned wg_id_x() { return __builtin_amdgcn_workgroup_id_x(); }
__device__ __forceinline__ unsigned wg_id_y() { return __builtin_amdgcn_workgroup_id_y(); }
__device__ __forceinline__ uint32_t mul_hi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }

// MI355X has 256 compute units in 8 XCDs; grid-shape heuristics are sized
// for that chip and do not query the device, so that workspace sizes are a
// pure function of the problem shape.
constexpr int kNumCU = 256;
constexpr int kNumXCD = 8;

// Stacked-row decomposition of the attention problem.  For one KV head the
// query rows of all rollouts, positions and group heads form one list of
// R = N*B*G rows, r = (n*B + b)*G + g, cut into M-tiles of `mtile_rows`; an
// M-tile index M = kh*MT + mt runs over all KV heads.  The key range of an
// M-tile is processed in one or more segments; segment `seg` of M-tile M
// leaves a partial (m, l, o[D]) in slot M*max_seg + seg of the workspace
// unless it is the M-tile's only segment.
//   fp32 path : `splits` workgroups per M-tile, each of them kF32Waves
//               wavefronts; the key tiles (prefix and private ones) are cut
//               into splits * kF32Waves equal runs, one per wavefront.
//   bf16 path : M-tiles of 256 rows or, in short calls, 128 (mtile_rows / 32
//               wavefronts per workgroup); the unit is one key tile of one M-tile (TPU units per M-tile,
//               U in total).  Either every M-tile is cut into `uniform` equal
//               pieces, piece s covering tiles [TPU s / S, TPU (s+1) / S), or
//               (stream-K) workgroup w of W owns the contiguous unit range
//               [unit_begin(w), unit_begin(w+1)), which may cross M-tiles.
constexpr int kF32RowTile = 32;    // fp32 path: stacked rows per workgroup
constexpr int kF32FewRowTile = 16; // fp32 path: the same in calls that leave half of the compute units idle
constexpr int kF32Waves = 8;       // fp32 path: wavefronts per workgroup
constexpr int kF32WideRowTile = 128, kF32WideKeyTile = 32;   // fp32 path, products on the bf16 pipe: rows per workgroup, keys per tile

struct AttnPlan {
    int G;            // query heads per KV head
    int R;            // stacked rows per KV head
    int mtile_rows;   // rows per M-tile
    int slots;        // bf16 path: ring slots per operand in LDS
    int MT;           // M-tiles per KV head
    int key_tile;     // keys per streamed tile
    int TP;           // prefix tiles = ceil(L / key_tile)
    int splits;       // fp32 path: workgroups per M-tile
    int TPU;          // bf16 path: units per M-tile = TP + the units booked for private tiles
    int W;            // bf16 path: workgroups
    int uniform;      // bf16 path: > 0 when W = Hkv*MT*uniform, i.e. equal pieces per M-tile
    long long U;      // bf16 path: units in total
    int max_seg;      // partial slots per M-tile
    size_t ws_o_bytes;   // partial outputs  [Hkv*MT][max_seg][mtile_rows][D], fp32 (fp32 path) or bf16 (bf16 path)
    size_t ws_ml_bytes;  // partial (m, l)   [Hkv*MT][max_seg][mtile_rows][2] fp32
    size_t ws_vt_bytes;  // bf16 path: V of the full prefix tiles repacked for the P V fragments, or 0
    bool packed;         // bf16 path: the kernel reads repacked V (from the workspace or from the caller)
};

// Without `ample` the plan for calls that bring less scratch than they are asked for: fp32 calls take no 128-row tiles, bf16
// calls leave the private tiles of an M-tile to one workgroup.
bool make_attn_plan(const fdd_attn_params& p, AttnPlan* plan, bool ample = true);

// Records the message fdd_last_error() returns on this thread; returns `code`.
fdd_status set_error(fdd_status code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
// Host-side checks of an unmask call (everything but the workspace); `fn` names the entry point in messages.
fdd_status check_unmask_args(const fdd_unmask_params* p, const char* fn);

// Division by a number fixed per launch, prepared on the host: for 0 <= n < 2^31 and 1 <= d < 2^31,
// n / d = ((n + 1) * mul) >> (32 + shift), where k = 31 + max(1, ceil(log2 d)), shift = k - 32 and mul is the
// largest integer with mul * d < 2^k.  With e = 2^k - mul * d in (0, d] and n = q d + r the product is
// q + ((r + 1) - (n + 1) e / 2^k) / d, and (n + 1) e <= 2^k keeps the bracket in [r, r + 1).
struct FastDiv {
    uint32_t mul, shift;
};
inline FastDiv make_fastdiv(uint32_t d)
{
    if (d == 0) d = 1;   // never used as a divisor then; keeps the host arithmetic defined
    uint32_t s = 1;
    while ((1ull << s) < d) ++s;
    const uint64_t two_k = 1ull << (31 + s);
    FastDiv f;
    f.mul = (uint32_t)((two_k - 1) / d);
    f.shift = s - 1;
    return f;
}
__host__ __device__ __forceinline__ int fast_div(int n, const FastDiv& f)
{
    return (int)((uint32_t)(((uint64_t)((uint32_t)n + 1u) * f.mul) >> 32) >> f.shift);
}

// bf16 path: how the merge kernel takes the segments of an M-tile: `sg` threads per 16-byte chunk, each with `ux` segments at a time, in
// so many rounds of loads.  sg: more threads while the chunks of a call leave most of the chip's lanes idle and each still has
// four segments or more to request.  us per call (replayed) with 1, 2, 4, 8 of them, Hq = 28, Hkv = 4, D = 128, B = 32: N=1
// (14 k chunks), L=512 (5 segments) 10.8, 10.4, 10.5, 11.0, L=2048 (17) 13.1, 12.0, 11.0, 11.6, L=16384 (29) 24.1, 21.5, 20.1,
// 20.5; N=2 (29 k), L=8192 (15) 21.1, 19.9, 19.8, 20.4, L=32768 (31) 43.1, 40.9, 40.5, 40.8; N=4 (57 k), L=8192 (9) 27.5, 26.8, 27.4,
// 28.5; N=8 (115 k), L=4096 (4) 27.0, 27.3, 29.1, 31.9, L=6000 (9) 35.1, 36.3, 36.0, 39.1; N=16 (229 k), L=4096 (4) 41.1, 42.2, 44.9,
// 50.8; one head, N=1, B=4, L=20000 (64 chunks, 157 segments) 37.9, 26.1, 17.4, 14.9.
struct MergeCut {
    int sg, ux, rounds;
};
inline MergeCut merge_cut(long long chunks, int segments)
{
    int sg = 1;
    while (sg < 8 && sg * 8 <= segments && chunks * sg * 2 <= (1 << 17)) sg *= 2;
    const int ux = sg >= 4 ? 8 : segments > 2 || sg == 2 ? 4 : 2;
    return {sg, ux, (segments + sg * ux - 1) / (sg * ux)};
}

// Key tiles of a row tile whose first and last row belong to rollouts n_lo and n_hi: `prefix` ones, and `per` for every
// rollout from one to the other.  (A list of positions in another order than ascending gives undefined values, but may not
// lead out of the arrays: where n_hi is below n_lo these are n_lo's private tiles, not a negative number of them.)  The bf16
// path counts an M-tile's private tiles with it, whose prefix tiles are dealt separately.
__host__ __device__ inline int key_tiles(int prefix, int per, int n_lo, int n_hi)
{
    return prefix + ((n_hi > n_lo ? n_hi - n_lo : 0) + 1) * per;
}

// First key tile of part `part` of the `parts` among which n_tiles are cut, floor(n_tiles part / parts).  fp32 path: the
// wavefronts or workgroups that share a row tile; bf16 path: the units booked for an M-tile's private tiles.  n_tiles >= 0.
// (A list of two far positions makes a row tile walk the private tiles of every rollout between them, up to 2^26 in all:
// n_tiles * part may pass 2^31, the remainder's product stays below parts^2 <= 2^18.)
__host__ __device__ inline int key_cut(int n_tiles, int part, int parts, const FastDiv& by_parts)
{
    const int base = fast_div(n_tiles, by_parts), rem = n_tiles - base * parts;
    return base * part + fast_div(rem * part, by_parts);
}

// fp32 path: launch grid of `wgs` workgroups.  One dimension takes less than 2^32 work items, 2^23 workgroups of 512 (64 GiB
// of queries at D = 64); larger calls get more rows, each of whole rounds of the XCDs.
inline dim3 f32_grid(int wgs)
{
    constexpr int kMax = 1 << 22;
    const int rows = (wgs + kMax - 1) / kMax, per_row = (wgs + rows - 1) / rows;
    return dim3((unsigned)((per_row + kNumXCD - 1) / kNumXCD * kNumXCD), (unsigned)rows);
}

// Unmask calls that take one launch, a workgroup of kOneLaunchWaves wavefronts per rollout, instead of a reduction over all
// rows and the decisions behind it.  A wavefront takes its rows one after the other, a memory latency each.  us per call,
// replayed, bf16, two launches / one:
//   - short rows: N=1, B=8, V=512 7.3/4.9; B=16, V=1024 (4 KB a wavefront) 7.3/6.0, V=2048 (8 KB) 7.2/7.1; N=64, B=32, V=512
//     8.7/6.8, V=1024 9.0/7.7 (fp32, N=8, B=64, V=512, 16 KB 7.9/10.2);
//   - up to 4 rows a wavefront (B = 32), or as many rollouts as positions, whose rows would take several rounds of workgroups:
//     B=64, V=128, N=1 7.3/8.5, N=16 7.9/8.8, N=64 9.7/8.9, N=256 18.1/9.1; B=128, V=128, N=1 8.2/13.7, N=64 13.3/14.3, N=256
//     30.4/15.1;
//   - up to one round of workgroups (four per compute unit); beyond it, where the rollouts keep the wavefronts busy: B=1, V=512,
//     N=1024 8.7/6.3, N=4096 13.1/13.3, N=16384 30.8/42.3, V=2048, N=65536 118/401; B=4, N=16384, V=512 57/46, V=1024 61/73;
//     B=8, N=16384, V=1024 107/83, V=2048 118/130; B=12, N=4096, V=1000 45/38; B=16, N=16384, V=1024 225/143.
// (This also keeps the launch below 2^32 work items: N B <= 2^24.)
constexpr int kOneLaunchWaves = 8, kOneLaunchB = 128;
inline bool unmask_in_one_launch(int N, int B, long long row_bytes)
{
    const long long share = (B + kOneLaunchWaves - 1) / kOneLaunchWaves * row_bytes;      // bytes a wavefront reads
    return B <= kOneLaunchB && share <= 4096 && (B <= 32 || N >= B) && (N <= 4 * kNumCU || (B >= 4 && 3 * share <= 1024 * B));
}

// Stream-K ranges: U units over W workgroups, base = U / W, rem = U % W; the
// first `rem` workgroups own base + 1 units, the others base (>= 1).
__host__ __device__ inline int unit_begin(int w, int base, int rem) { return w * base + (w < rem ? w : rem); }

// `before_main`, if not null, is recorded on the stream right before the main kernel (after the V pre-pass).
hipError_t launch_attn_bf16(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s, hipEvent_t before_main);
hipError_t launch_prefix_pack(const void* prefix_v, int L, int Hkv, int D, void* packed, hipStream_t s);
hipError_t launch_attn_f32(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s);
hipError_t launch_attn_combine(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s);      // fp32 path
hipError_t launch_attn_merge_bf16(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s);   // bf16 path

// Vocabulary reduction: each eligible logits row is cut into `vsplits`
// pieces; a piece leaves (max, argmax, sum exp(x - max)) in the workspace.
struct UnmaskPlan {
    int vsplits;
    size_t ws_bytes;  // [N*B][vsplits] x {float max; int32 arg; float sum; int32 pad}
};
bool make_unmask_plan(const fdd_unmask_params& p, UnmaskPlan* plan);
// `argmax_only`: the plan of the greedy verifier's pass (no sums); the sampled verifier and the unmask step share the other
bool make_vocab_plan(int N, int B, long long V, int dtype, bool argmax_only, UnmaskPlan* plan);
hipError_t launch_unmask(const fdd_unmask_params& p, const UnmaskPlan& plan, hipStream_t s);
hipError_t launch_verify(const fdd_verify_params& p, const UnmaskPlan& plan, hipStream_t s);

hipError_t launch_fork_block(int N, size_t bytes, const void* src, void* dst, hipStream_t s);
hipError_t launch_kv_update(const fdd_kv_update_params& p, hipStream_t s);
hipError_t launch_block_commit(const fdd_commit_params& p, hipStream_t s);
hipError_t launch_traj_mean(int N, int P, const float* traj, float* out, hipStream_t s);

}  // namespace fdd
