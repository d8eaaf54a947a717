// Shared-prefix block-causal attention, bf16 storage, gfx950 matrix cores.
//
// What is computed (paper, "Block-Causal Diffusion" and "Shared prefix"):
// every query row of every rollout attends to the L prefix keys and to the
// B keys of its own rollout's block.  Nothing here knows about layers or
// models; the prefix K/V is read through one pointer for all rollouts.
//
// How the work is laid out
//   * For one KV head, the query rows of all rollouts, block positions and
//     group heads are stacked into one list of R = N*B*G rows and cut into
//     M-tiles of 32 rows per wavefront.  Every prefix K/V tile a workgroup
//     stages in LDS is therefore used by all its stacked rows, whichever
//     rollout they come from; the prefix is never replicated.
//   * Scores are produced transposed, S^T = K Q^T, with the 32x32x16 bf16
//     MFMA: each lane then owns ONE query row (lane % 32) and 16 keys per
//     32-key block, so the row maximum and the row sum of the streaming
//     softmax are in-lane reductions plus a single exchange between the two
//     32-lane halves.  The same registers, rounded to bf16, are the B
//     operand of O^T += V^T P^T, so P never leaves the register file and the
//     accumulator keeps one query row per lane: its rescale is a per-lane
//     scalar multiply.
//   * Every K/V tile goes from global memory straight into LDS
//     (buffer_load ... lds: no registers, no vector ALU work, no LDS writes by
//     the waves) into a ring of SLOTS slots for K and as many for V.  K tiles lie
//     [key][d] with the 16-byte pieces of a row XOR-swizzled by the row index,
//     which keeps the K fragment reads conflict-free without padding.
//   * O^T += V^T P^T needs, per lane, 8 keys of one channel, i.e. V with the
//     key index contiguous, while V lies in memory [key][d].  Where an
//     M-tile's keys are streamed by more than one workgroup (R > 256 rows per
//     KV head), or the caller did it once for the prefix, the full prefix
//     tiles of V are packed into the exact fragment order,
//     [tile][16-key step][half][d][8 keys], and read back as plain
//     conflict-free 128-bit loads.  V tiles that are moved as they lie (a
//     single M-tile per head, the ragged last prefix tile, a rollout's private
//     tiles) are read with the gfx950 LDS transpose read (ds_read_b64_tr_b16:
//     lane i of a 16-lane group receives column i of a 4 x 16 block, i.e. 4
//     consecutive keys of channel i); their 32-byte columns are XOR-swizzled
//     by the row on the global side of the load, which makes those reads
//     conflict-free too.
//   * Full prefix tiles run through a software-pipelined loop of 32 MFMAs per
//     tile (D = 64: 16).  Beside each of them stands a slice of vector
//     ALU work that does not depend on that MFMA: while the matrix pipe
//     produces the scores of tile i+1 and then the P V products of tile i,
//     the vector ALUs take the exponentials of tile i, round them to bf16 and
//     find the row maximum of tile i+1.  V of tile i+SLOTS-1 and K of tile
//     i+SLOTS are requested in step i (K is read one step before V,
//     so its slot is free one step earlier) and waits are counted (the loads
//     of a wavefront complete in issue order): with four slots four half tiles stay in
//     flight across a step boundary, with two none; LDS
//     fragments are requested three MFMAs before their use.  The loop is
//     unrolled SLOTS times so that ring slots are immediate offsets.
//   * The softmax reference value of a row is only raised when the running
//     maximum outgrows it by more than 2^8; in between probabilities may
//     exceed 1, which fp32 sums and bf16 relative precision do not mind, and
//     the accumulator rescale becomes a rare wave-uniform branch.  The result
//     is mathematically the same softmax.
//   * A workgroup has 8 wavefronts (M-tiles of 256 rows) or, where a call is
//     short, 4 (128 rows, one wavefront per SIMD), and 4 ring slots per operand
//     or, where it is very short, 2: the plan chooses (see make_attn_plan).
//     With 2 slots K of tile i+2 and V of tile i+1 are requested in step i and
//     awaited at its end.
//   * Work is dealt out in units of one 64-key prefix tile of one M-tile.
//     Either every M-tile is cut into S equal pieces (workgroups numbered so
//     that an XCD owns all M-tiles of one (KV head, piece): they walk the same
//     keys in step and the XCD's L2 serves all but the first fetch), or all
//     units, ordered by (KV head, M-tile, tile), are cut into W contiguous
//     ranges, one per workgroup (stream-K), so every compute unit gets the
//     same amount of work whatever the shape.  A range may end inside an
//     M-tile and continue in the next one: each such segment keeps its own
//     streaming-softmax state (m, l, o) per row.  An M-tile that was covered
//     by a single segment is normalised and written as bf16 output directly;
//     otherwise the segments leave their averages (bf16) and (m, l) (fp32),
//     which a second small kernel merges (log-sum-exp merge, fixed order).
//   * The ragged last prefix tile and the private tiles of every rollout the
//     M-tile's rows belong to (the rows that rollout committed since the fork,
//     then its live block: paper, "Shared prefix" and "Block-Causal
//     Diffusion") go through a simpler masked path out of the same ring: rows
//     of other rollouts are masked to -inf, and in the verify pass of scaffold
//     speculative decoding the block keys after the query's own position too.
#include <atomic>
#include <type_traits>
#include <utility>

#include "fdd_internal.h"

namespace fdd {
namespace attn_bf16 {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

constexpr int ODD_XCD_WEIGHT = 97;   // share of a piece on an odd XCD, in per cent of one on an even XCD (measured: 96..98 alike)
constexpr int KT = 64;           // keys per tile
typedef short i16x4 __attribute__((ext_vector_type(4)));

// Kernel arguments.  They are read from memory with scalar loads, a 64-byte line at a time, and every
// first touch of a line is a round trip of a few hundred nanoseconds: the fields a workgroup needs before
// it can request its first tiles come first and are pulled in together (see the top of the kernel), the
// fields of the Q load follow, the rest is only needed while the first tiles are on their way.
struct Args {
    // ---- before the first tile request -----------------------------------------------------------
    const uint16_t* pk;
    const uint16_t* pv;
    const uint16_t* vt;   // packed V^T tiles of the full prefix tiles (PACKED kernels only)
    long long p_bs, vt_bs;   // batch: element strides between the problems' prefix arrays
    int W;          // workgroups
    int per_xcd;    // ceil(W / 8)
    int S;          // > 0: every M-tile is cut into S equal pieces (W = Hkv*MT*S); 0: free ranges
    int MT, TPU;    // M-tiles per KV head; units per M-tile = max(TP, 1) + booked private units
    int base, rem;  // free ranges: U / W and U % W
    int w_even, w_odd;   // equal pieces: weight of a piece by the parity of the XCD it runs on
    int Hkv, batch;      // batch: independent problems in this launch
    int L, TP, TPF;      // prefix rows, prefix tiles, full prefix tiles = L / 64
    FastDiv dMT, dS, dTPU, dHkv, dPerXcd;   // divisions by launch constants
    // ---- the Q load ----------------------------------------------------------------------------------
    const uint16_t* q;
    const int32_t* qpos;   // stacked rows are the listed block positions only (ascending n*B + b), or nullptr: all of them
    long long q_bs;
    int G, R, Hq, NB;      // NB = N * B
    FastDiv dG;
    // ---- the rest ------------------------------------------------------------------------------------
    const uint16_t* bk;
    const uint16_t* bv;
    const uint16_t* ek;   // per-rollout extension [N, Ecap, Hkv, D]
    const uint16_t* ev;
    uint16_t* out;
    void* ws_o;      // partial averages, bf16, in accumulator order (see the epilogue)
    float* ws_ml;    // partial (m, l) per row
    long long b_bs, e_bs, o_bs;
    int E, Ecap;
    int N, B;
    int max_seg;    // partial slots per M-tile
    int causal;     // in-block keys are visible up to the query's own position only
    float c;        // scale * log2(e)
    float slack;    // 8 / c: scores may pass their reference by this much
    int ttpr;       // private tiles per rollout: extension tiles, then block tiles
    int booked;     // units booked for private tiles = TPU - TP
    FastDiv dBooked;
    FastDiv dB, dBG, dTTPR, dBase, dBase1;
};

template <int D, int WAVES, int SLOTS>
struct Cfg {
    static constexpr int THREADS = WAVES * 64;
    static constexpr int NB = SLOTS;                     // ring slots per operand in LDS (2 or 4)
    // 64 x D tiles, unpadded, moved global -> LDS in 1 KB pieces, one per wavefront instruction
    static constexpr int T_BYTES = KT * D * 2;
    static constexpr int NI = T_BYTES / 1024 / WAVES;    // pieces per wavefront and tile
    static constexpr int IPT = 2 * NI;                   // load instructions per wavefront for K and V of one tile
    static constexpr int CH = D / 8;                     // 16-byte pieces per row
    static constexpr int RPB = 1024 / (D * 2);           // rows per 1 KB piece
    static constexpr int RPL = 256 / (D * 2);            // rows per 256-byte bank line
    static constexpr int V_RING = NB * T_BYTES;          // LDS offset of the V ring (the K ring starts at 0)
    static constexpr int DUMP = 2 * NB * T_BYTES;        // where requests that have no tile go
    static constexpr int LDS_BYTES = DUMP + T_BYTES;
    static_assert(NI >= 1 && T_BYTES % (1024 * WAVES) == 0, "tile must divide over the wavefronts");
    static_assert((NB - 1) * IPT < 64, "outstanding loads must fit the counter");
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// value held by the lane 32 positions away (the other half of the wavefront)
__device__ __forceinline__ float other_half(float x)
{
    const unsigned u = __builtin_bit_cast(unsigned, x);
    // swaps lanes 32..63 of the first operand with lanes 0..31 of the second
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (thread_id_x() & 32) ? r[0] : r[1]);
}

// Wait until at most N of this wavefront's vector memory operations are
// still in flight (they complete in issue order).
template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N < 64, "counter range");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Workgroup barrier that orders LDS traffic only.  (__syncthreads() also
// fences global memory, which makes the compiler drain every tile still on
// its way into the ring.)  No memory access is moved across it.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Nothing is scheduled across this point: the source order of the pieces it
// separates is the order the hardware sees.
#define FDD_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
// Forces a value to exist at this point of the instruction stream, so that
// the vector work of a slot is not sunk towards its first use.
#define FDD_PIN(x) asm volatile("" : "+v"(x))

// f(0), f(1), .. with compile-time arguments
template <typename F, int... J>
__device__ __forceinline__ void for_slots(F& f, std::integer_sequence<int, J...>)
{
    (f(std::integral_constant<int, J>()), ...);
}

// use(j, read(j)) for j in [0, N), every fragment requested AHEAD matrix instructions before its own: left to itself the
// compiler, short of registers elsewhere, reads each one right before its use, and a wavefront that has nothing else to do
// (before the pipelined loop, in masked tiles) waits for LDS 16 times a tile.
template <int N, int AHEAD, typename Read, typename Use>
__device__ __forceinline__ void read_ahead(const Read& read, const Use& use)
{
    bf16x8 f[AHEAD + 1];
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) f[j] = read(j);
    FDD_SCHED_FENCE();
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (j + AHEAD < N) f[(j + AHEAD) % (AHEAD + 1)] = read(j + AHEAD);
        use(j, f[j % (AHEAD + 1)]);
        FDD_SCHED_FENCE();
    }
}

// Transposing LDS read.  `restrict` is for the compiler's wait insertion: before an LDS read that carries no alias
// information it waits for every tile that is still on its way into LDS (vmcnt(0)), which ordinary reads are spared by their
// type.  The plain-V loop stood still for the tiles requested in the same step, and masked tiles for the next ones.
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
__device__ __forceinline__ i16x4 read_tr(const lds_i16x4* __restrict__ p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(const_cast<lds_i16x4*>(p));
}

template <int D, int WAVES, int SLOTS, bool PACKED>
__global__ __launch_bounds__(WAVES * 64, WAVES == 8 ? 1 : 2) void attn_bf16_kernel(Args a)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub
    using C = Cfg<D, WAVES, SLOTS>;
    constexpr int NB = C::NB;
    constexpr int KS = D / 16;   // MFMA k-steps of Q K^T
    constexpr int DB = D / 32;   // 32-channel blocks of the output
    constexpr int MROWS = WAVES * 32;
    constexpr int RA = 4;        // fragments requested ahead outside the pipelined loop
    constexpr uint32_t RSRC_FLAGS = 0x00020000;

    extern __shared__ __align__(16) unsigned char lds[];
    typedef __attribute__((address_space(3))) void lds_void;
    const int tid = thread_id_x();
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);   // same value, known to be wave-uniform

    // ---- everything the first tile requests need, in one round trip to the argument block -------
    {
        long long h0 = a.p_bs, h1 = a.vt_bs;
        int h2 = a.W, h3 = a.per_xcd, h4 = a.S, h5 = a.MT, h6 = a.TPU, h7 = a.base, h8 = a.rem, h9 = a.w_even,
            h10 = a.w_odd, h11 = a.Hkv, h12 = a.batch, h13 = a.L, h14 = a.TP, h15 = a.TPF;
        uint32_t d0 = a.dMT.mul, d1 = a.dMT.shift, d2 = a.dS.mul, d3 = a.dS.shift, d4 = a.dTPU.mul, d5 = a.dTPU.shift,
                 d6 = a.dHkv.mul, d7 = a.dHkv.shift, d8 = a.dPerXcd.mul, d9 = a.dPerXcd.shift;
        const uint16_t *p0 = a.pk, *p1 = a.pv, *p2 = a.vt;
        asm volatile("" ::"s"(h0), "s"(h1), "s"(h2), "s"(h3), "s"(h4), "s"(h5), "s"(h6), "s"(h7), "s"(h8), "s"(h9), "s"(h10),
                     "s"(h11), "s"(h12), "s"(h13), "s"(h14), "s"(h15), "s"(d0), "s"(d1), "s"(d2), "s"(d3), "s"(d4), "s"(d5),
                     "s"(d6), "s"(d7), "s"(d8), "s"(d9), "s"(p0), "s"(p1), "s"(p2));
        // the fields of the Q load, and a first touch of every other 64-byte line of the block (what is read
        // from those later then comes from the scalar cache)
        const uint16_t* q0 = a.q;
        const int32_t* q1 = a.qpos;
        long long q2 = a.q_bs;
        int q3 = a.G, q4 = a.R, q5 = a.Hq, q6 = a.NB;
        uint32_t q7 = a.dG.mul, q8 = a.dG.shift;
        const uint32_t* ap = reinterpret_cast<const uint32_t*>(&a);
        static_assert(sizeof(Args) > 80 * 4 && sizeof(Args) <= 96 * 4, "one touch per 64-byte line of Args");
        uint32_t t3 = ap[48], t4 = ap[64], t5 = ap[80];
        asm volatile("" ::"s"(q0), "s"(q1), "s"(q2), "s"(q3), "s"(q4), "s"(q5), "s"(q6), "s"(q7), "s"(q8), "s"(t3), "s"(t4), "s"(t5));
    }

    // ---- this workgroup's share of the (M-tile, prefix tile) units ------------
    // Workgroups are dealt to the 8 XCDs round-robin by their launch index;
    // ranges are numbered so that the workgroups of one XCD own neighbours.
    int wg = (int)(wg_id_x() % kNumXCD) * a.per_xcd + (int)(wg_id_x() / kNumXCD);
    if (wg >= a.W) return;
    int M, t_begin, todo, piece = 0;
    if (a.S > 0) {
        // equal pieces: neighbours are the M-tiles of one (KV head, piece), which
        // walk the same keys in step, so each XCD fetches its share of K/V once
        const int rest = fast_div(wg, a.dMT), mt_ = wg - rest * a.MT;
        const int khv_ = fast_div(rest, a.dS);
        piece = rest - khv_ * a.S;
        M = khv_ * a.MT + mt_;
        if (a.w_odd == a.w_even) {
            t_begin = fast_div(a.TPU * piece, a.dS);
            todo = fast_div(a.TPU * (piece + 1), a.dS) - t_begin;
        } else {
            // The share of a piece follows the speed of the XCD it runs on (measured: the odd XCD of a
            // pair streams the same tiles a few per cent slower).  Every piece of the M-tile works out
            // the same boundaries: unit TPU * (weights before it) / (all weights).  Lane p looks at piece p (S <= 16).
            const int x = fast_div((khv_ * a.S + min(lane, a.S - 1)) * a.MT + mt_, a.dPerXcd);
            const unsigned odd = (unsigned)__builtin_amdgcn_ballot_w64(lane < a.S && (x & 1));
            auto weight = [&](int n) { return n * a.w_even - __builtin_popcount(odd & ((1u << n) - 1u)) * (a.w_even - a.w_odd); };
            const int lo = weight(piece), hi = weight(piece + 1), cum = weight(a.S);
            t_begin = (a.TPU * lo) / cum;
            todo = (a.TPU * hi) / cum - t_begin;
        }
    } else {
        const int u0 = unit_begin(wg, a.base, a.rem);
        todo = unit_begin(wg + 1, a.base, a.rem) - u0;
        M = fast_div(u0, a.dTPU);
        t_begin = u0 - M * a.TPU;
    }

    // ---- per-lane constants of the tile movement and of the fragment reads ------
    const uint32_t stride2 = (uint32_t)(a.Hkv * D * 2);       // bytes between consecutive keys
    // LDS offsets of this lane's fragments (set while the first tiles of a segment are on their way)
    uint32_t k_fragoff[KS];
    uint32_t v_fragoff_ring, vtr_off[DB];
    // Tile movement: piece jn of this wavefront covers rows (wave NI + jn) RPB .. of
    // a tile; this lane moves the 16 bytes that land at LDS piece (lane % CH) of
    // its row.  K: the pieces of a row are XOR-swizzled by the row's bank line.
    // V as it lies in memory: 32-byte columns are XOR-swizzled by the row, for
    // the transposing reads.  Packed V^T tiles are copied as they are.
    uint32_t k_voff[C::NI];
#pragma unroll
    for (int jn = 0; jn < C::NI; ++jn) {
        const int r = (wave * C::NI + jn) * C::RPB + lane / C::CH;
        // (less the instruction's offset, which moves the place in LDS and the address alike; a piece is 1 KB or more from the last)
        k_voff[jn] = (uint32_t)r * stride2 + (uint32_t)(((lane % C::CH) ^ ((r / C::RPL) & (C::CH - 1))) * 16) - jn * 1024u;
    }
    // V: one offset for all pieces of a wavefront (its column swizzle repeats every piece; the pieces' rows are in the scalar offset)
    uint32_t v_voff;
    if (PACKED) {
        v_voff = (uint32_t)(wave * C::NI * 1024 + lane * 16);
    } else {
        static_assert(C::RPB / C::RPL == 4, "the column swizzle of V repeats every piece");
        const int r = wave * C::NI * C::RPB + lane / C::CH;
        v_voff = (uint32_t)r * stride2 + (uint32_t)(((lane % C::CH) ^ ((((r / C::RPL) & 3) << 2) & (C::CH - 1))) * 16);
    }
    const uint32_t v_piece = PACKED ? 0u : C::RPB * stride2 - 1024u;      // between pieces, beyond the 1 KB of the instruction's offset
    auto k_frag = [&](uint32_t kbase, int kb, int ks) -> bf16x8 {
        return *reinterpret_cast<const bf16x8*>(lds + (kbase + k_fragoff[ks]) + kb * 32 * D * 2);
    };
    auto v_frag_tr = [&](uint32_t slot, int t4, int db) -> bf16x8 {
        const unsigned char* p0 = lds + vtr_off[db] + (slot + t4 * 16 * (D * 2));
        const i16x4 lo = read_tr((const lds_i16x4*)(p0));
        const i16x4 hi = read_tr((const lds_i16x4*)(p0 + 8 * (D * 2)));
        typedef short i16x8 __attribute__((ext_vector_type(8)));
        const i16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, both);
    };

    // (wave-uniform values are marked as such, so that addresses built from them stay in scalar registers)
    M = __builtin_amdgcn_readfirstlane(M);
    t_begin = __builtin_amdgcn_readfirstlane(t_begin);
    todo = __builtin_amdgcn_readfirstlane(todo);
    for (; todo > 0; ++M, t_begin = 0) {
        const int t_end = min(a.TPU, t_begin + todo);
        todo -= t_end - t_begin;
        // M runs over (problem of the batch, KV head, M-tile)
        const int khv = fast_div(M, a.dMT);
        const int mt = M - khv * a.MT;
        const int pb = a.batch > 1 ? fast_div(khv, a.dHkv) : 0;
        const int kh = khv - pb * a.Hkv;
        // (the arrays of problem pb are addressed where they are used: few of these pointers are live at a time)
        const uint16_t* const pk = a.pk + pb * a.p_bs;
        const uint16_t* const pv = PACKED ? a.vt + pb * a.vt_bs : a.pv + pb * a.p_bs;
        const uint32_t pk_bytes = (uint32_t)a.L * stride2;
        const uint32_t pv_bytes = PACKED ? (uint32_t)(a.Hkv * a.TPF) * C::T_BYTES : pk_bytes;
        // stores of the previous segment are out of the way of the load counting below
        wait_vm<0>();

        // ---- tile schedule ---------------------------------------------------
        // Tiles 0 .. F-1 are full 64-key prefix tiles; the rest are masked: the
        // ragged last prefix tile, then the segment's share of the private tiles
        // of every rollout the M-tile's rows belong to.
        const int t0 = min(t_begin, a.TP);
        const int n_prefix = min(t_end, a.TP) - t0;
        const int F = (n_prefix > 0 && (t0 + n_prefix) * KT > a.L) ? n_prefix - 1 : n_prefix;

        // ---- tile j: global memory -> ring slot j % NB, no registers in between ----
        int issued = 0;
        // Full prefix tile (j < F).  A request for a tile that there is not goes to the dump slot and reads nothing (a
        // buffer of no bytes): so every step issues the same loads without a branch, and its wait counts a constant.
        auto request = [&](auto is_v, int j, uint32_t slot, auto first, auto last) {
            constexpr bool V = decltype(is_v)::value;
            constexpr int P0 = decltype(first)::value, P1 = decltype(last)::value;
            const bool live = j < F;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint16_t*>(V ? pv : pk), 0, live ? (V ? pv_bytes : pk_bytes) : 0u, RSRC_FLAGS);
            unsigned char* const dst = lds + (live ? slot + (V ? C::V_RING : 0) : C::DUMP) + wave_u * (C::NI * 1024);
            const uint32_t soff = V && PACKED ? (uint32_t)(kh * a.TPF + t0 + j) * C::T_BYTES : (uint32_t)((t0 + j) * KT) * stride2 + (uint32_t)(kh * D * 2);
            auto piece = [&](auto jc) {
                constexpr int jn = decltype(jc)::value + P0;
                if constexpr (jn < P1)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)dst, 16, V ? v_voff : k_voff[jn], V ? soff + jn * v_piece : soff, jn * 1024, 0);
            };
            for_slots(piece, std::make_integer_sequence<int, P1 - P0>());
        };
        const std::integral_constant<int, 0> p_0;
        const std::integral_constant<int, C::NI> p_all;
        const std::true_type is_v;
        const std::false_type is_k;
        auto fetch_k = [&](int j, uint32_t slot) { request(is_k, j, slot, p_0, p_all); };
        auto fetch_v = [&](int j, uint32_t slot) { request(is_v, j, slot, p_0, p_all); };
        // ---- Q fragments: B operand of S^T = K Q^T ------------------------------
        const int row0_wg = mt * MROWS;
        const int row0 = row0_wg + wave * 32;
        const int row = row0 + l32;
        const bool row_ok = row < a.R;
        // a stacked row is (entry of the list of query positions, query head of the group)
        // (lanes beyond the last row compute it once more and store nothing: the loads need no branch)
        const int row_c = min(row, a.R - 1);
        const int sel = fast_div(row_c, a.dG);
        const int g = row_c - sel * a.G;
        const int nb = a.qpos ? min(max(a.qpos[sel], 0), a.NB - 1) : sel;   // n*B + b
        bf16x8 qf[KS];
        {
            const uint16_t* qp = a.q + pb * a.q_bs + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * D + half * 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                qf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qp + ks * 16));
            }
        }
        FDD_SCHED_FENCE();

        // Q is requested first and the first full tiles right after it, before anything else is worked
        // out, so that the rest of the set-up runs under their latency.  The loads of a wavefront complete
        // in issue order: with Q in front, the first step can start as soon as Q and the first tiles are
        // there, while the later ones are still on their way.
        // (K runs one tile ahead of V: K of tile j is read one step before V of tile j, so its slot is free
        // one step earlier, and one more half tile per workgroup is on its way at any time)
        // Only what the first step needs is requested here; the rest of the ring follows in the shadow of its first scores (all at
        // once, every workgroup's first tile waited behind the others' fourth: first barrier 4.5 -> 4.0 us after the start at N=8, L=4096).
        fetch_k(0, 0);
        fetch_v(0, 0);
        fetch_k(1, C::T_BYTES);
        issued = min(NB - 1, F);
        FDD_SCHED_FENCE();

        // ---- the rest of the set-up ------------------------------------------------
        {
            int lane_f = lane;
            FDD_PIN(lane_f);      // (computed here, not ahead of the requests)
            const int l32 = lane_f & 31, half = lane_f >> 5;
            // K fragment of k-step ks: row l32 of a 32-key block, 16-byte piece (2 ks + half)
            // at its swizzled place, which is the place of k-step 0 with ks XORed in
            const uint32_t k_fragoff0 = (uint32_t)(l32 * D * 2 + ((((l32 / C::RPL) & (C::CH - 1)) ^ half) << 4));
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) k_fragoff[ks] = k_fragoff0 ^ (uint32_t)(ks << 5);
            // packed V^T: [16-key step][half][d][8 keys]; the ring's offset is part of the register
            // because the offset field of an LDS read ends at 64 KB
            v_fragoff_ring = (uint32_t)(C::V_RING + half * (D * 16) + l32 * 16);
            FDD_PIN(v_fragoff_ring);
            // Unpacked V, transposing reads.  In a 16-lane group, lane 4j+q points at 4
            // channels of key row j; the read returns to lane i the 4 keys of channel i.
            // Element e of the assembled fragment is key 16 t4 + 8 (e/4) + 4 half + e%4,
            // the key order of the probabilities in the S^T accumulator.  Channel block
            // db sits at the swizzled place of block 0 with db XORed in.
            const int row_l = half * 4 + ((lane_f & 15) >> 2);
            const int x = ((lane_f >> 4) & 1) * 2 + ((lane_f & 3) >> 1);
            const int sw = (((row_l / C::RPL) & 3) << 2) & (C::CH - 1);
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                vtr_off[db] = (uint32_t)(C::V_RING + ((row_l * D * 2 + ((x ^ sw) << 4) + (lane_f & 1) * 8) ^ (db << 6)));
                FDD_PIN(vtr_off[db]);
            }
        }
        int n_seg, seg;
        if (a.S > 0) {
            n_seg = a.S;
            seg = piece;
        } else {
            // owner of a unit: the first `rem` workgroups hold base + 1 units each, the others base
            const int cut = a.rem * (a.base + 1);
            const FastDiv by1 = a.dBase1, by = a.dBase;     // (copies, here and below: 4 to 8 scalar registers fewer are put aside)
            auto owner = [&](int u) { return u < cut ? fast_div(u, by1) : a.rem + fast_div(u - cut, by); };
            const int first = owner(M * a.TPU);
            n_seg = owner((M + 1) * a.TPU - 1) - first + 1;
            seg = wg - first;
        }
        // What masked tiles need (the ragged last tile of the prefix, private tiles), in the segments that have any: rollout and
        // block position of the lane's row, the rollouts that this wavefront's rows and the whole M-tile span
        // (rows are in ascending order of position, hence of rollout; `r` is clamped to the rows that exist)
        const bool wave_has_rows = row0_wg + wave_u * 32 < a.R;
        int my_rollout = -1, my_b = 0, wave_n_lo = 0, wave_n_hi = 0, wg_n_lo = 0, tte = 0, ttpr = 1, n_tail = 0, tail0 = 0;
        if (t_end > a.TP || F < n_prefix) {
            const FastDiv by_b = a.dB, by_bg = a.dBG;
            if (row_ok) {
                my_rollout = fast_div(nb, by_b);
                my_b = nb - my_rollout * a.B;
            }
            auto rollout_of_row = [&](int r) {
                r = min(r, a.R - 1);
                if (!a.qpos) return fast_div(r, by_bg);
                const int e = __builtin_amdgcn_readfirstlane(fast_div(r, a.dG));
                return fast_div(min(max(a.qpos[e], 0), a.NB - 1), by_b);
            };
            wave_n_lo = rollout_of_row(row0);
            wave_n_hi = rollout_of_row(row0 + 31);
            wg_n_lo = __builtin_amdgcn_readfirstlane(rollout_of_row(row0_wg));
            const int wg_n_hi = __builtin_amdgcn_readfirstlane(rollout_of_row(row0_wg + MROWS - 1));
            tte = (a.E + KT - 1) >> 6;             // tiles of a rollout's extension
            ttpr = a.ttpr;                         // private tiles per rollout: extension, then block
            // The private tiles lie evenly over the booked units, each with the segment that holds the last of its own.  (All on
            // the M-tile's last segment, a rollout's extension and block and those of the rollouts after it were done one after the
            // other, 1.5 to 2 us each, when the other workgroups had ended.  us per call: N=33, B=1, L=1408, Hq=8, Hkv=8, E=1 93.7 -> 12.9;
            // N=9, B=1, L=11904, D=64, E=37 32.6 -> 10.4.  Which calls deal them out: make_attn_plan.)
            if (t_end > a.TP) {
                n_tail = key_tiles(0, ttpr, wg_n_lo, wg_n_hi);
                if (t_begin > a.TP || t_end < a.TPU) {
                    const FastDiv by = a.dBooked;
                    const int all = n_tail;
                    tail0 = key_cut(all, max(t_begin - a.TP, 0), a.booked, by);
                    n_tail = key_cut(all, t_end - a.TP, a.booked, by) - tail0;
                }
            }
        }
        const int n_tiles = n_prefix + n_tail;

        struct Tile {
            int src;        // 0: shared prefix, 1: a rollout's extension, 2: a rollout's block
            int row_base;   // first key, as a row of that K/V array
            int valid;      // keys that exist
            int rollout;    // whose rows may see it (-1: every row)
            int key0;       // block position of the first key (block tiles)
        };
        auto tile_at = [&](int j) -> Tile {
            Tile t;
            if (j < n_prefix) {
                t.src = 0;
                t.row_base = (t0 + j) * KT;
                t.valid = min(KT, a.L - t.row_base);
                t.rollout = -1;
                t.key0 = 0;
            } else {
                const int jj = j - n_prefix + tail0;
                int n = wg_n_lo + jj, w = 0;
                if (ttpr > 1) {
                    const int q_ = fast_div(jj, a.dTTPR);
                    n = wg_n_lo + q_;
                    w = jj - q_ * ttpr;
                }
                t.rollout = n;
                if (w < tte) {
                    t.src = 1;
                    t.row_base = n * a.Ecap + w * KT;
                    t.valid = min(KT, a.E - w * KT);
                    t.key0 = 0;
                } else {
                    const int k0 = (w - tte) * KT;
                    t.src = 2;
                    t.row_base = n * a.B + k0;
                    t.valid = min(KT, a.B - k0);
                    t.key0 = k0;
                }
            }
            return t;
        };

        // masked tile: rows beyond `valid` repeat the last valid row (finite values;
        // their scores are masked), so nothing is read out of bounds
        auto fetch_masked = [&](int j) {
            const Tile t = tile_at(j);
            const uint32_t rows_in_array = t.src == 0 ? (uint32_t)a.L : t.src == 1 ? (uint32_t)(a.N * a.Ecap) : (uint32_t)(a.N * a.B);
            const uint32_t bytes = rows_in_array * stride2;
            const uint16_t* const ksrc = t.src == 0 ? a.pk + pb * a.p_bs : t.src == 1 ? a.ek + pb * a.e_bs : a.bk + pb * a.b_bs;
            const uint16_t* const vsrc = t.src == 0 ? a.pv + pb * a.p_bs : t.src == 1 ? a.ev + pb * a.e_bs : a.bv + pb * a.b_bs;
            const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(ksrc), 0, bytes, RSRC_FLAGS);
            const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(vsrc), 0, bytes, RSRC_FLAGS);
            const uint32_t soff = __builtin_amdgcn_readfirstlane((uint32_t)t.row_base * stride2 + (uint32_t)(kh * D * 2));
            const uint32_t slot = (uint32_t)(j & (NB - 1)) * C::T_BYTES;
            const int last = t.valid - 1;
            int tid_f = tid;
            FDD_PIN(tid_f);
            const int wave_f = tid_f >> 6, lane_f = tid_f & 63;
#pragma unroll
            for (int jn = 0; jn < C::NI; ++jn) {
                // this lane moves the 16 bytes that land at LDS piece (lane % CH) of row r of the tile
                const int r = (wave_f * C::NI + jn) * C::RPB + lane_f / C::CH;
                const uint32_t row_off = (uint32_t)min(r, last) * stride2;
                const uint32_t k_col16 = (uint32_t)(((lane_f % C::CH) ^ ((r / C::RPL) & (C::CH - 1))) * 16);
                const uint32_t v_col16 = (uint32_t)(((lane_f % C::CH) ^ ((((r / C::RPL) & 3) << 2) & (C::CH - 1))) * 16);
                unsigned char* const kdst = lds + slot + (wave_u * C::NI + jn) * 1024;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rsrc, (lds_void*)kdst, 16, row_off + k_col16, soff, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rsrc, (lds_void*)(kdst + C::V_RING), 16, row_off + v_col16, soff, 0, 0);
            }
        };
        // tile j: global memory -> ring slot j % NB, no registers in between
        auto fetch = [&](int j_) {
            const int j = __builtin_amdgcn_readfirstlane(j_);
            fetch_masked(j);
            issued = j + 1;
        };
        // block until tile t has landed in LDS for the whole workgroup; tiles are
        // fetched in order, IPT load instructions per wavefront each
        int landed = -1;     // tiles up to this one are in LDS for every wavefront
        auto wait_landed = [&](int t) {
            landed = t;
            const int k = issued - 1 - t;
            if (NB > 2 && k >= 3) wait_vm<(NB > 2 ? 3 : 0) * C::IPT>();
            else if (NB > 2 && k == 2) wait_vm<(NB > 2 ? 2 : 0) * C::IPT>();
            else if (k == 1) wait_vm<C::IPT>();
            else wait_vm<0>();
            wg_barrier();
        };

        // masked tiles that fit the ring ahead of time
        while (issued < min(NB - 1, n_tiles)) fetch(issued);
        const int ahead = F > 0 ? issued - min(NB - 1, F) : 0;       // such tiles of a segment with full ones: fewer than NB - 1
        // all but the newest n loads and these tiles must have landed
        auto wait_but = [&](auto n) {
            constexpr int N = decltype(n)::value;
            if (NB == 2 || ahead == 0) wait_vm<N>();
            else if (ahead == 1) wait_vm<N + (NB > 2 ? 1 : 0) * C::IPT>();
            else wait_vm<N + (NB > 2 ? 2 : 0) * C::IPT>();
        };

        // ---- streaming-softmax state: one query row per lane --------------------
        float zero = 0.f;       // (a vector of constants would be built in 16 scalar registers)
        FDD_PIN(zero);
        f32x16 o[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] = zero;
        float m_ref = 0.f;         // reference value the exponentials are taken against (raw score units)
        float limit = -INFINITY;   // a score above it raises the reference: 2^8 above it, or -inf: there is none yet
        float l_run = 0.f;         // this lane's share of the running sum

        // Raise the reference when a row outgrew it by more than 2^8 (always on the first tile).  `mx` is the largest score of
        // this lane's half of the keys: whether any lane passes its limit needs no exchange, only the rare raise does.  (A
        // compare and a branch between the row maximum and the exponentials instead of a chain of ten instructions that wait for
        // one another.)
        auto update_reference = [&](float mx) {
            if (__any(mx > limit)) {
                const bool none = limit == -INFINITY;       // (nothing summed so far, or only keys the row does not see)
                float m = fmaxf(mx, other_half(mx));
                if (!none) m = fmaxf(m, m_ref);
                const float alpha = none ? 0.f : fast_exp2((m_ref - m) * a.c);
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
                m_ref = (m == -INFINITY) ? 0.f : m;
                limit = (m == -INFINITY) ? m : m + a.slack;
            }
        };

        // What step i requests: K of tile i+NB, V of tile i+NB-1 (into the slots of K of tile i, read last in step i-1, and V
        // of tile i-1).  At its end K of tile i+2 and V of tile i+1 must have landed.
        auto wait_step = [&] { wait_vm<(NB - 2) * 2 * C::NI>(); };

        bf16x8 p[4];      // probabilities of a tile as MFMA B operands, one per 16-key step

        // ---- full prefix tiles, software pipelined ---------------------------------
        // Issue order so far: Q, K0 V0 K1 (and masked tiles of a short segment).
        if (F > 0) {
            const std::integral_constant<int, 2 * C::NI> first;
            const std::integral_constant<int, (NB - 2) * 2 * C::NI> rest;
            wait_but(first);       // Q, K0
            wg_barrier();
            // what the ring still has room for: V1 K2 V2 K3
            auto request_rest = [&](auto c) {        // half tile c
                constexpr int h = decltype(c)::value;
                if constexpr (h % 2 == 0) fetch_v(1 + h / 2, (uint32_t)(1 + h / 2) * C::T_BYTES);
                else fetch_k(2 + h / 2, (uint32_t)(2 + h / 2) * C::T_BYTES);
            };
            if (!wave_has_rows) {
                // A wavefront without rows (the M-tile is not full) only moves its share of the tiles: the matrix pipe and
                // the power are left to the others (8 requests of N=1, 224 of 256 rows, L=16384: 84.0 -> 82.1 us; with 112
                // rows or fewer a SIMD has one wavefront to serve).  Same requests, waits and barriers as in the steps below.
                for_slots(request_rest, std::make_integer_sequence<int, 2 * (NB - 2)>());
                wait_but(rest);
                wg_barrier();
                for (int i = 0; i < F; ++i) {
                    fetch_k(i + NB, (uint32_t)(i & (NB - 1)) * C::T_BYTES);
                    fetch_v(i + NB - 1, (uint32_t)((i + NB - 1) & (NB - 1)) * C::T_BYTES);
                    wait_step();
                    wg_barrier();
                }
            } else {
                // prologue: scores of tile 0, the other requests of the ring spread over them
                f32x16 sa[2], sb[2];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) sa[kb][v] = 0.f;
                {
                    bf16x8 f[RA + 1];
#pragma unroll
                    for (int j = 0; j < RA; ++j) f[j] = k_frag(0, j / KS, j % KS);
                    FDD_SCHED_FENCE();
                    auto slot = [&](auto jc) {
                        constexpr int j = decltype(jc)::value, NREQ = 2 * (NB - 2) * C::NI;        // pieces to request
                        if constexpr (j + RA < 2 * KS) f[(j + RA) % (RA + 1)] = k_frag(0, (j + RA) / KS, (j + RA) % KS);
                        sa[j / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[j % (RA + 1)], qf[j % KS], sa[j / KS], 0, 0, 0);
                        auto req = [&](auto rc) {
                            constexpr int r = j * NREQ / (2 * KS) + decltype(rc)::value;
                            if constexpr (r < (j + 1) * NREQ / (2 * KS)) {
                                constexpr int h = r / C::NI, pc = r % C::NI;
                                const std::integral_constant<int, pc> p0;
                                const std::integral_constant<int, pc + 1> p1;
                                if constexpr (h % 2 == 0) request(is_v, 1 + h / 2, (uint32_t)(1 + h / 2) * C::T_BYTES, p0, p1);
                                else request(is_k, 2 + h / 2, (uint32_t)(2 + h / 2) * C::T_BYTES, p0, p1);
                            }
                        };
                        for_slots(req, std::make_integer_sequence<int, 4>());
                        FDD_SCHED_FENCE();
                    };
                    static_assert(2 * (NB - 2) * C::NI <= 4 * 2 * KS, "four requests a slot");
                    for_slots(slot, std::make_integer_sequence<int, 2 * KS>());
                }
                // largest score of the tile whose probabilities are next, over this lane's half of the keys
                float mx = -INFINITY;
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(fmaxf(mx, sa[0][v]), sa[1][v]);
                // Step 0 requests K of tile SLOTS into the slot that the scores above were read from: no wavefront may get
                // there while another one is still reading.  (They can be far apart here: the first workgroups of a
                // launch fetch these instructions from memory.)
                FDD_SCHED_FENCE();
                wait_but(rest);        // V0, K1
                wg_barrier();

                // One pipelined step: probabilities and P V of tile i from s_cur while the scores of tile i+1 go to s_nxt.
                //   slots  0-15  S(i+1), first and second 32 keys  ||  exponentials of tile i
                //   slots 16-31  P V                               ||  the last exponentials, row maximum of tile i+1
                // `par` is i % NB as a compile-time constant: ring slots become immediate offsets of the LDS reads.  The scores of
                // tile i+1 are computed whether or not it is a full tile (from whatever its slot holds); they are only used if it is.
                // On entry K up to tile i+1 and V up to tile i have landed; on exit K up to tile i+2 and V up to tile i+1.
                //
                // What a wavefront issues beside its matrix instructions (32 cycles each) has to fit into their shadow: 6 cycles a
                // vector instruction, 10 an exponential, for a wavefront alone on its SIMD (measured).  So exponentials are spread
                // evenly, one "tick" (exponential, scaling of the one after next, rounding of the last pair) every 0.85 slots, each
                // stage behind the next tick's so that nothing waits for its predecessor; requests are single instructions without
                // branches, spread over the slots as well; and the row sum is taken in one run at the end: v_dot2 shares the matrix pipe
                // and costs 16 of its cycles between two matrix instructions, 4 behind another v_dot2.
                // Cycles a step, few workgroups: D = 128, V laid out, 8 wavefronts 3036 -> 2559 (64 matrix instructions a SIMD), 4
                // wavefronts 2240 -> 1610 (32); D = 64 2240 -> 1896 and 1788 -> 1287.  With the chip full its power sets the clock:
                // N=64, B=64, L=8192 413 -> 398 us a call; N=8, B=32, L=4096, 128 rows 27.2 -> 24.3; N=1, L=16384 20.7 -> 19.6.
                auto step = [&](auto par, int i, f32x16 (&s_cur)[2], f32x16 (&s_nxt)[2]) {
                    constexpr int P = decltype(par)::value;
                    constexpr uint32_t KSLOT = (uint32_t)((P + 1) % NB) * C::T_BYTES;
                    constexpr uint32_t VSLOT = (uint32_t)P * C::T_BYTES;
                    constexpr uint32_t KNEW = (uint32_t)P * C::T_BYTES, VNEW = (uint32_t)((P + NB - 1) % NB) * C::T_BYTES;
                    constexpr int AH = 3;                                         // fragments requested ahead
                    constexpr int NS = 2 * KS, NPV = 4 * DB, NSL = NS + NPV;      // slots of the scores, of P V, of the step
                    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
                    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
                    u32x4 pw[4];     // the B operands of P V as packed words
                    auto frag = [&](int j) -> bf16x8 {
                        if (j < NS) return *reinterpret_cast<const bf16x8*>(lds + k_fragoff[j % KS] + (KSLOT + j / KS * 32 * D * 2));
                        const int t4 = (j - NS) / DB, db = (j - NS) % DB;
                        if (PACKED) return *reinterpret_cast<const bf16x8*>(lds + v_fragoff_ring + (VSLOT + t4 * (D * 32) + db * 512));
                        return v_frag_tr(VSLOT, t4, db);
                    };
                    float mc = 0.f;
                    auto scale = [&](int e) {
                        float x = fmaf(s_cur[e / 16][e % 16], a.c, -mc);
                        FDD_PIN(x);
                        s_cur[e / 16][e % 16] = x;
                    };
                    auto expo = [&](int e) {
                        float x = fast_exp2(s_cur[e / 16][e % 16]);
                        FDD_PIN(x);
                        s_cur[e / 16][e % 16] = x;
                    };
                    auto round_pair = [&](int k) {
                        const bf16x2 pr = {(__bf16)s_cur[k / 8][2 * (k % 8)], (__bf16)s_cur[k / 8][2 * (k % 8) + 1]};
                        uint32_t u = __builtin_bit_cast(uint32_t, pr);
                        FDD_PIN(u);
                        pw[k / 4][k % 4] = u;
                    };
                    bf16x8 f[AH + 1];
                    FDD_SCHED_FENCE();
#pragma unroll
                    for (int j = 0; j < AH; ++j) f[j] = frag(j);
                    FDD_SCHED_FENCE();
                    update_reference(mx);
                    mc = m_ref * a.c;
                    mx = -INFINITY;
                    FDD_SCHED_FENCE();
                    scale(0);
                    scale(1);
                    FDD_SCHED_FENCE();
                    constexpr int NT = 33, SPAN = NSL - DB;      // ticks, the slots they are spread over
                    static_assert(8 * SPAN / NT < NS && 16 * SPAN / NT < NS + DB && 24 * SPAN / NT < NS + 2 * DB && 32 * SPAN / NT < NS + 3 * DB, "probabilities before their use");
                    auto slot = [&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        if constexpr (j + AH < NSL) f[(j + AH) % (AH + 1)] = frag(j + AH);
                        if constexpr (j == 0 || j == KS) {
#pragma unroll
                            for (int v = 0; v < 16; ++v) s_nxt[j / KS][v] = 0.f;
                        }
                        if constexpr (j < NS) {
                            s_nxt[j / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[j % (AH + 1)], qf[j % KS], s_nxt[j / KS], 0, 0, 0);
                        } else {
                            constexpr int t4 = (j - NS) / DB, db = (j - NS) % DB;
                            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[j % (AH + 1)], __builtin_bit_cast(bf16x8, pw[t4]), o[db], 0, 0, 0);
                        }
                        FDD_SCHED_FENCE();
                        if constexpr (j % 2 == 1) {
                            constexpr int r = j / 2;
                            const std::integral_constant<int, r % C::NI> p0;
                            const std::integral_constant<int, r % C::NI + 1> p1;
                            if constexpr (r < C::NI) request(is_k, i + NB, KNEW, p0, p1);
                            else if constexpr (r < 2 * C::NI) request(is_v, i + NB - 1, VNEW, p0, p1);
                            FDD_SCHED_FENCE();
                        }
                        auto tick = [&](auto tc) {
                            constexpr int t = decltype(tc)::value;
                            if constexpr (t * SPAN / NT == j) {
                                if constexpr (t < 32) expo(t);
                                FDD_SCHED_FENCE();
                                if constexpr (t % 2 == 0 && t > 0) round_pair(t / 2 - 1);
                                if constexpr (t + 2 < 32) scale(t + 2);
                                FDD_SCHED_FENCE();
                            }
                        };
                        for_slots(tick, std::make_integer_sequence<int, NT>());
                        if constexpr (j >= NS + 2) {
                            constexpr int q = j - NS - 2, NQ = NPV - 2;
#pragma unroll
                            for (int v = q * 16 / NQ; v < (q + 1) * 16 / NQ; ++v) {
                                mx = fmaxf(fmaxf(mx, s_nxt[0][v]), s_nxt[1][v]);
                                FDD_PIN(mx);
                            }
                        }
                        FDD_SCHED_FENCE();
                    };
                    for_slots(slot, std::make_integer_sequence<int, NSL>());
                    // the row sum is taken over the probabilities as they enter P V (rounded to bf16): numerator and denominator then
                    // see the same values
                    float acc0 = 0.f, acc1 = 0.f;
#pragma unroll
                    for (int k = 0; k < 16; k += 2) {
                        acc0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)pw[k / 4][k % 4]), ones, acc0, false);
                        acc1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)pw[(k + 1) / 4][(k + 1) % 4]), ones, acc1, false);
                    }
                    l_run += acc0 + acc1;
                    wait_step();
                    wg_barrier();
                };
                const std::integral_constant<int, 0> r0;
                const std::integral_constant<int, 1> r1;
                const std::integral_constant<int, 2> r2;
                const std::integral_constant<int, 3> r3;
                for (int i = 0;;) {
                    step(r0, i, sa, sb);
                    if (++i == F) break;
                    step(r1, i, sb, sa);
                    if (++i == F) break;
                    if constexpr (NB == 4) {
                        step(r2, i, sa, sb);
                        if (++i == F) break;
                        step(r3, i, sb, sa);
                        if (++i == F) break;
                    }
                }
            }
            // (only requests without a tile are still on their way; masked tiles requested before the loop have landed)
            issued = max(issued, F);
        } else {
            wait_vm<0>();
            wg_barrier();
        }
        landed = issued - 1;

        // ---- masked tiles: ragged last prefix tile and the in-block tail ------------
        // On entry to iteration j tile j has landed.
        for (int j = F; j < n_tiles; ++j) {
            // the slots refilled here held tiles up to j-1, last read before the previous barrier
            while (issued < min(n_tiles, j + NB)) fetch(issued);
            if (landed < j) wait_landed(j);
            const Tile t = tile_at(j);
            const uint32_t kbase = (uint32_t)(j & (NB - 1)) * C::T_BYTES;
            const bool wave_active = wave_has_rows &&
                (t.rollout < 0 || (t.rollout >= wave_n_lo && t.rollout <= wave_n_hi));
            if (wave_active) {
                // A tile of 32 keys or fewer (a block of 32, the last rows of an extension) takes half of the products and
                // exponentials.  us per call, all of both blocks / as here: N=1, L=2048 10.98/10.75; N=8, L=2048 19.3/18.8, L=4096 with E=64
                // 28.4/27.5; N=5, B=40, L=5003, D=64, E=37 18.0/16.5 (most of it from one bound per row in place of four conditions a key).
                const int n_kb = t.valid > 32 ? 2 : 1;
                f32x16 s[2];
                // register v of block kb is key kb*32 + (v/4)*8 + half*4 + v%4; in the verify pass later keys of the block are hidden
                const int upto = a.causal && t.src == 2 ? min(t.valid, my_b + 1 - t.key0) : t.valid;
                const int seen = (t.rollout < 0 || t.rollout == my_rollout ? upto : 0) - half * 4;
                float mx = -INFINITY;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    if (kb >= n_kb) break;
#pragma unroll
                    for (int v = 0; v < 16; ++v) s[kb][v] = 0.f;
                    read_ahead<KS, RA>([&](int x) { return k_frag(kbase, kb, x); }, [&](int x, const bf16x8& f) {
                        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[x], s[kb], 0, 0, 0);
                    });
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        if (kb * 32 + (v >> 2) * 8 + (v & 3) >= seen) s[kb][v] = -INFINITY;
                        mx = fmaxf(mx, s[kb][v]);
                    }
                }
                update_reference(mx);
                const float mc = m_ref * a.c;
                float acc = 0.f;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    if (kb >= n_kb) break;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float pr = fast_exp2(fmaf(s[kb][v], a.c, -mc));
                        acc += pr;
                        p[kb * 2 + v / 8][v % 8] = (__bf16)pr;
                    }
                    read_ahead<2 * DB, RA>([&](int x) { return v_frag_tr(kbase, 2 * kb + x / DB, x % DB); },
                                           [&](int x, const bf16x8& f) {
                                               o[x % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, p[2 * kb + x / DB], o[x % DB], 0, 0, 0);
                                           });
                }
                l_run += acc;
            }
            if (j + 1 < n_tiles) wait_landed(j + 1); else wg_barrier();
        }
        const float m_run = limit == -INFINITY ? limit : m_ref;

        // ---- epilogue of the segment ------------------------------------------------
        const float l_tot = l_run + other_half(l_run);
        if (row_ok) {
            if (n_seg == 1) {
                const float inv = 1.f / l_tot;
                uint16_t* op = a.out + pb * a.o_bs + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * D;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4) {
                        const int d = db * 32 + v4 * 8 + half * 4;
                        typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
                        bf16x4 w;
#pragma unroll
                        for (int j = 0; j < 4; ++j) w[j] = (__bf16)(o[db][v4 * 4 + j] * inv);
                        *reinterpret_cast<bf16x4*>(op + d) = w;
                    }
            } else {
                // Partial of this segment: the segment's own softmax average (o / l, rounded to bf16) and its
                // (m, l) in fp32.  The averages lie in the order of the accumulator registers,
                // [M-tile][segment][wavefront][register pair][lane] x 8 bf16, so every store instruction of a
                // wavefront writes 1 KB in one piece and the merge kernel reads them the same way.
                // The stores are written through to memory (aux 16 = device scope): the merge kernel's workgroups sit on
                // other XCDs, and lines left dirty in the L2s go out only when the launch has ended (28 layers of N=1,
                // L=16384: 723 -> 696 us; N=8, L=4096: 28.9 -> 27.7; plain, non-temporal and both measured).
                const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
                const size_t pseg = (size_t)M * a.max_seg + __builtin_amdgcn_readfirstlane(seg);
                const __amdgpu_buffer_rsrc_t o_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                    static_cast<unsigned char*>(a.ws_o) + pseg * (size_t)(MROWS * D * 2), 0, MROWS * D * 2, RSRC_FLAGS);
                const uint32_t o_off = (uint32_t)(wave * (2 * DB * 64) + lane) * 16;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int v2 = 0; v2 < 2; ++v2) {
                        bf16x8 w;
#pragma unroll
                        for (int j = 0; j < 8; ++j) w[j] = (__bf16)(o[db][v2 * 8 + j] * inv);
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), o_rsrc, o_off + (db * 2 + v2) * 1024, 0, 16);
                    }
                if (half == 0) {
                    const size_t prow = pseg * MROWS + (wave * 32 + l32);
                    float* const ml = a.ws_ml + prow * 2;
                    ml[0] = m_run;
                    ml[1] = l_tot;
                }
            }
        }
    }   // next segment of this workgroup's range
#endif
}

// ---------------------------------------------------------------------------
// Pre-pass: the full 64-key prefix tiles of V, repacked once into the order
// the P V fragments are read in:  vt[kh][tile][t4][half][d][8 keys], where the
// 8 keys of (t4, half) are 16 t4 + 4 half + {0..3} and 16 t4 + 8 + 4 half + {0..3}
// (the key order of the probabilities in the S^T accumulator).  One workgroup
// per (tile, KV head): stage the tile [key][d] in LDS, then let the LDS
// transpose read do the transposition; a wavefront stores two 512-byte runs.
template <int D>
struct PackCfg {
    static constexpr int THREADS = 512;
    static constexpr int VROW = D * 2 + 64;              // padded row: conflict-free transposing reads
    static constexpr int V_BYTES = KT * VROW;
    static constexpr int K_PER_THREAD = KT * (D / 8) / THREADS;
    static constexpr int T_BYTES = KT * D * 2;
};

template <int D>
__global__ __launch_bounds__(512) void vt_pack_kernel(const uint16_t* __restrict__ pv_all, uint16_t* __restrict__ vt_all,
                                                       int Hkv, int TPF, long long p_bs, long long vt_bs)
{
    using C = PackCfg<D>;
    constexpr int DB = D / 32;
    __shared__ __align__(16) unsigned char tile[C::V_BYTES];
    // grid (tile, KV head of a problem of the batch)
    const int t = wg_id_x(), pb = wg_id_y() / Hkv, kh = wg_id_y() - pb * Hkv;
    const uint16_t* pv = pv_all + pb * p_bs;
    uint16_t* vt = vt_all + pb * vt_bs;
    const int tid = thread_id_x(), wave = tid >> 6, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const size_t kv_stride = (size_t)Hkv * D;
    const uint16_t* src = pv + (size_t)t * KT * kv_stride + (size_t)kh * D;
#pragma unroll
    for (int i = 0; i < C::K_PER_THREAD; ++i) {
        const int c = tid + i * C::THREADS;
        const int key = c / (D / 8), col = c % (D / 8);
        *reinterpret_cast<u32x4*>(tile + key * C::VROW + col * 16) =
            *reinterpret_cast<const u32x4*>(src + (size_t)key * kv_stride + col * 8);
    }
    __syncthreads();
    const int tr_lane_off = ((half * 4 + ((lane & 15) >> 2)) * C::VROW) + (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
    unsigned char* dst = reinterpret_cast<unsigned char*>(vt) + ((size_t)kh * TPF + t) * C::T_BYTES;
    for (int combo = wave; combo < 4 * DB; combo += 8) {
        const int t4 = combo / DB, db = combo % DB;
        typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
        const unsigned char* p0 = tile + tr_lane_off + (t4 * 16) * C::VROW + db * 64;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p0));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p0 + 8 * C::VROW));
        typedef short i16x8 __attribute__((ext_vector_type(8)));
        const i16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        *reinterpret_cast<i16x8*>(dst + t4 * (D * 32) + half * (D * 16) + (db * 32 + l32) * 16) = both;
    }
}

// ---------------------------------------------------------------------------
// Merge of the segments of an M-tile (log-sum-exp merge, paper-independent arithmetic of the split):
//   m* = max_s m_s,   W_s = l_s 2^((m_s - m*) c),   out = sum_s W_s avg_s / sum_s W_s
// with avg_s the segment's own softmax average as the attention kernel left it (bf16, accumulator order).
// The sums run in a fixed order, so results are reproducible.
//
// Bound by latency: a few MB through a launch of its own.  So a thread works alone as long as it can: it takes one
// chunk (8 channels of a row) of every SG-th segment, requests UX averages and the (m, l) pairs that weigh them together,
// and the SG threads of a chunk, which lie in one wavefront, meet in lane moves at the end.  No LDS, no barrier.  The
// pairs of a row are read by the threads of all its chunks; that costs less than passing weights on.
// grid (M-tiles, 2 DB SG WAVES / 4), WAVES as of the attention kernel: 4 wavefronts of 64 / SG chunks each.
struct MergeArgs {
    const u32x4* ws_o;
    const float* ws_ml;
    uint16_t* out;
    const int32_t* qpos;
    long long o_bs;
    int Hq, Hkv, G, R, MT, NB;
    int max_seg, fixed_seg, TPU, rem, cut;   // cut = rem (base + 1): units of the longer ranges
    FastDiv dMT, dHkv, dG, dBase, dBase1;
    float c;
};

// sum or maximum over the SG lanes lane % (64 / SG) + i 64 / SG, in every one of them
template <int SG, typename Op>
__device__ __forceinline__ float reduce_groups(float v, Op op)
{
    uint32_t x = __float_as_uint(v);
    if (SG >= 8) x = __float_as_uint(op(v, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true))));   // row_ror:8
    if (SG >= 4) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = __float_as_uint(op(__uint_as_float(r[0]), __uint_as_float(r[1])));
    }
    if (SG >= 2) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        x = __float_as_uint(op(__uint_as_float(r[0]), __uint_as_float(r[1])));
    }
    return __uint_as_float(x);
}

template <int D, int WAVES, int SG, int UX>
__global__ __launch_bounds__(256) void attn_merge_bf16_kernel(MergeArgs a)
{
    constexpr int DB = D / 32;
    constexpr int CPW = 2 * DB * 64;          // 16-byte chunks per wavefront of the attention kernel
    constexpr int CH = WAVES * CPW;           // chunks per M-tile and segment
    constexpr int MROWS = WAVES * 32;
    constexpr int CPL = 64 / SG;              // chunks per wavefront here
    const int tid = thread_id_x();
    const int M = (int)wg_id_x();
    int n_seg = a.fixed_seg;
    if (n_seg == 0) {    // same arithmetic as the attention kernel: workgroups whose unit range meets this M-tile
        auto owner = [&](int u) { return u < a.cut ? fast_div(u, a.dBase1) : a.rem + fast_div(u - a.cut, a.dBase); };
        n_seg = owner((M + 1) * a.TPU - 1) - owner(M * a.TPU) + 1;
    }
    if (n_seg == 1) return;     // written in final form by its only segment
    const int khv = fast_div(M, a.dMT), mt = M - khv * a.MT;      // (problem of the batch, KV head), M-tile
    const int c0 = (int)wg_id_y() * (4 * CPL);                    // the block's first chunk: [wave][register pair][lane]
    const int wave = c0 / CPW;
    const int row0 = mt * MROWS + wave * 32;  // first stacked row of the block's 32 rows
    if (row0 >= a.R) return;
    const int lane = tid & 63, sg = lane / CPL;
    const int cidx = c0 + (tid >> 6) * CPL + lane % CPL;
    const int r = cidx & 31, half = (cidx >> 5) & 1, i2 = (cidx >> 6) % (2 * DB);
    const bool live = row0 + r < a.R;
    const u32x4* src = a.ws_o + (size_t)M * a.max_seg * CH + cidx;
    const float* ml = a.ws_ml + ((size_t)M * a.max_seg * MROWS + wave * 32 + r) * 2;

    float m = -INFINITY, sum = 0.f;           // this thread's segments: largest m, sum of weights against it
    float acc[8];                             // and their weighted average
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    for (int s0 = 0; s0 < n_seg; s0 += SG * UX) {
        float2 y[UX];
        u32x4 x[UX];
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            const int s = s0 + sg + u * SG;
            y[u] = make_float2(-INFINITY, 0.f);
            x[u] = u32x4{0u, 0u, 0u, 0u};
            if (live && s < n_seg) {
                y[u] = *reinterpret_cast<const float2*>(ml + (size_t)s * (2 * MROWS));
                x[u] = src[(size_t)s * CH];
            }
        }
        __builtin_amdgcn_sched_barrier(0);    // everything is requested before anything is waited for
        float mx = m;
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            // (a segment that saw no key of this row has l = 0 and takes no part; its average is 0 as well)
            if (!(y[u].y > 0.f)) y[u].x = -INFINITY;
            mx = fmaxf(mx, y[u].x);
        }
        const float mref = mx == -INFINITY ? 0.f : mx;
        const float old = s0 > 0 ? sum * __builtin_amdgcn_exp2f((m - mref) * a.c) : 0.f;
        m = mx;
        sum = old;
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            y[u].y *= __builtin_amdgcn_exp2f((y[u].x - mref) * a.c);
            sum += y[u].y;
        }
        // weights are divided before they meet the values: the sum of a few thousand keys' worth of large values would overflow
        const float inv = sum > 0.f ? 1.f / sum : 0.f;
        if (s0 > 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] *= old * inv;
        }
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            const float w = y[u].y * inv;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[2 * j] = fmaf(__uint_as_float(x[u][j] << 16), w, acc[2 * j]);
                acc[2 * j + 1] = fmaf(__uint_as_float(x[u][j] & 0xffff0000u), w, acc[2 * j + 1]);
            }
        }
    }
    if (SG > 1) {
        const float mx = reduce_groups<SG>(m, [](float p, float q) { return fmaxf(p, q); });
        const float f = __builtin_amdgcn_exp2f((m - (mx == -INFINITY ? 0.f : mx)) * a.c);
        auto add = [](float p, float q) { return p + q; };
        sum *= f;
        const float total = reduce_groups<SG>(sum, add), share = total > 0.f ? sum / total : 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = reduce_groups<SG>(acc[j] * share, add);
    }
    if (!live || sg != 0) return;
    const int pb = fast_div(khv, a.dHkv), kh = khv - pb * a.Hkv;
    const int row = row0 + r;
    const int sel = fast_div(row, a.dG), g = row - sel * a.G;
    const int nb = a.qpos ? min(max(a.qpos[sel], 0), a.NB - 1) : sel;
    uint16_t* op = a.out + pb * a.o_bs + ((size_t)nb * a.Hq + (size_t)kh * a.G + g) * D + (i2 >> 1) * 32 + (i2 & 1) * 16 + half * 4;
    typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
    bf16x4 lo, hi;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        lo[j] = (__bf16)acc[j];
        hi[j] = (__bf16)acc[4 + j];
    }
    *reinterpret_cast<bf16x4*>(op) = lo;
    *reinterpret_cast<bf16x4*>(op + 8) = hi;
}

template <int D, int WAVES, int SLOTS, bool PACKED>
hipError_t launch(const Args& a, bool pack_now, hipStream_t stream, hipEvent_t before_main)
{
    using C = Cfg<D, WAVES, SLOTS>;
    const size_t lds_bytes = C::LDS_BYTES;
    const auto kern = &attn_bf16_kernel<D, WAVES, SLOTS, PACKED>;
    // the LDS limit of this instantiation is raised once per device (bit d of `done`: device d)
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(done.load(std::memory_order_acquire) & bit)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_release);
    }
    if (PACKED && pack_now) {
        hipLaunchKernelGGL(vt_pack_kernel<D>, dim3(a.TPF, a.Hkv * a.batch), dim3(512), 0, stream, a.pv,
                           const_cast<uint16_t*>(a.vt), a.Hkv, a.TPF, a.p_bs, a.vt_bs);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (before_main) {
        hipError_t e = hipEventRecord(before_main, stream);
        if (e != hipSuccess) return e;
    }
    const int grid = a.per_xcd * kNumXCD;   // padded so that every XCD gets the same count
    hipLaunchKernelGGL(kern, dim3(grid), dim3(C::THREADS), lds_bytes, stream, a);
    return hipGetLastError();
}

}  // namespace attn_bf16

using namespace attn_bf16;

hipError_t launch_attn_bf16(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s, hipEvent_t before_main)
{
    Args a;
    a.q = static_cast<const uint16_t*>(p.q);
    a.pk = static_cast<const uint16_t*>(p.prefix_k);
    a.pv = static_cast<const uint16_t*>(p.prefix_v);
    a.bk = static_cast<const uint16_t*>(p.block_k);
    a.bv = static_cast<const uint16_t*>(p.block_v);
    a.out = static_cast<uint16_t*>(p.out);
    char* ws = static_cast<char*>(p.workspace);
    a.ws_o = ws;
    a.ws_ml = reinterpret_cast<float*>(ws + plan.ws_o_bytes);
    const bool pack_now = plan.packed && !p.prefix_v_packed;
    a.vt = pack_now ? reinterpret_cast<const uint16_t*>(ws + plan.ws_o_bytes + plan.ws_ml_bytes)
                    : static_cast<const uint16_t*>(p.prefix_v_packed);
    a.ek = static_cast<const uint16_t*>(p.ext_k);
    a.ev = static_cast<const uint16_t*>(p.ext_v);
    a.E = p.E; a.Ecap = p.ext_capacity;
    a.batch = p.batch > 1 ? p.batch : 1;
    a.q_bs = p.q_batch_stride; a.p_bs = p.prefix_batch_stride; a.b_bs = p.block_batch_stride;
    a.e_bs = p.ext_batch_stride; a.o_bs = p.out_batch_stride;
    // packed V: the caller's stride, or the in-call copies lying back to back in the workspace
    a.vt_bs = pack_now ? (long long)p.Hkv * (p.L / 64) * 64 * p.D : (long long)(p.packed_batch_stride / 2);
    a.N = p.N; a.B = p.B; a.L = p.L; a.Hq = p.Hq; a.Hkv = p.Hkv;
    a.G = plan.G; a.R = plan.R; a.MT = plan.MT; a.TP = plan.TP; a.TPF = p.L / 64;
    a.TPU = plan.TPU; a.W = plan.W; a.max_seg = plan.max_seg; a.S = plan.uniform;
    a.per_xcd = (plan.W + kNumXCD - 1) / kNumXCD;
    a.base = (int)(plan.U / plan.W); a.rem = (int)(plan.U % plan.W);
    a.causal = (p.flags & FDD_ATTN_CAUSAL_BLOCK) ? 1 : 0;
    a.c = scale * 1.4426950408889634f;
    a.slack = 8.f / a.c;
    a.ttpr = (p.E + 63) / 64 + (p.B + 63) / 64;
    a.booked = plan.TPU - plan.TP;
    a.dBooked = make_fastdiv((uint32_t)a.booked);
    a.qpos = p.n_q_positions > 0 ? p.q_positions : nullptr;
    a.NB = p.N * p.B;
    a.dMT = make_fastdiv((uint32_t)a.MT);
    a.dS = make_fastdiv((uint32_t)(a.S > 0 ? a.S : 1));
    a.dTPU = make_fastdiv((uint32_t)a.TPU);
    a.dHkv = make_fastdiv((uint32_t)a.Hkv);
    a.dG = make_fastdiv((uint32_t)a.G);
    a.dB = make_fastdiv((uint32_t)a.B);
    a.dBG = make_fastdiv((uint32_t)(a.B * a.G));
    a.dTTPR = make_fastdiv((uint32_t)a.ttpr);
    a.dBase = make_fastdiv((uint32_t)(a.base > 0 ? a.base : 1));
    a.dBase1 = make_fastdiv((uint32_t)(a.base + 1));
    a.dPerXcd = make_fastdiv((uint32_t)a.per_xcd);
    // (with 2..16 pieces of 32 units or more a shift of 3 % is at least one unit)
    a.w_even = 100;
    a.w_odd = (a.S >= 2 && a.S <= 16 && a.TPU >= 32 * a.S) ? ODD_XCD_WEIGHT : 100;
    auto go = [&](auto waves, auto slots) {
        constexpr int WAVES = decltype(waves)::value, SLOTS = decltype(slots)::value;
        if (plan.packed)
            return p.D == 128 ? launch<128, WAVES, SLOTS, true>(a, pack_now, s, before_main) : launch<64, WAVES, SLOTS, true>(a, pack_now, s, before_main);
        return p.D == 128 ? launch<128, WAVES, SLOTS, false>(a, false, s, before_main) : launch<64, WAVES, SLOTS, false>(a, false, s, before_main);
    };
    const std::integral_constant<int, 8> w8;
    const std::integral_constant<int, 4> w4, s4;
    const std::integral_constant<int, 2> s2;
    if (plan.mtile_rows == 256) return go(w8, s4);
    if (plan.mtile_rows == 128) return plan.slots == 2 ? go(w4, s2) : go(w4, s4);
    return hipErrorInvalidValue;
}

hipError_t launch_attn_merge_bf16(const fdd_attn_params& p, const AttnPlan& plan, float scale, hipStream_t s)
{
    MergeArgs a;
    a.ws_o = static_cast<const u32x4*>(p.workspace);
    a.ws_ml = reinterpret_cast<const float*>(static_cast<const char*>(p.workspace) + plan.ws_o_bytes);
    a.out = static_cast<uint16_t*>(p.out);
    a.qpos = p.n_q_positions > 0 ? p.q_positions : nullptr;
    a.o_bs = p.out_batch_stride;
    const int batch = p.batch > 1 ? p.batch : 1;
    a.Hq = p.Hq; a.Hkv = p.Hkv; a.G = plan.G; a.R = plan.R; a.MT = plan.MT; a.NB = p.N * p.B;
    a.max_seg = plan.max_seg; a.fixed_seg = plan.uniform; a.TPU = plan.TPU;
    const int base = (int)(plan.U / plan.W);
    a.rem = (int)(plan.U % plan.W);
    a.cut = a.rem * (base + 1);
    a.dMT = make_fastdiv((uint32_t)a.MT);
    a.dHkv = make_fastdiv((uint32_t)a.Hkv);
    a.dG = make_fastdiv((uint32_t)a.G);
    a.dBase = make_fastdiv((uint32_t)(base > 0 ? base : 1));
    a.dBase1 = make_fastdiv((uint32_t)(base + 1));
    a.c = scale * 1.4426950408889634f;
    const MergeCut cut = merge_cut((long long)p.Hkv * batch * plan.R * (p.D / 8), plan.uniform > 0 ? plan.uniform : plan.max_seg);
    auto go = [&](auto d, auto sgc, auto ux) {
        constexpr int D = decltype(d)::value, SG = decltype(sgc)::value, UX = decltype(ux)::value;
        const dim3 grid((unsigned)(p.Hkv * batch * plan.MT), (unsigned)(plan.mtile_rows / 32 * 2 * (D / 32) * SG / 4));
        if (plan.mtile_rows == 256) hipLaunchKernelGGL((attn_merge_bf16_kernel<D, 8, SG, UX>), grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((attn_merge_bf16_kernel<D, 4, SG, UX>), grid, dim3(256), 0, s, a);
    };
    auto sized = [&](auto d) {
        const std::integral_constant<int, 1> i1;
        const std::integral_constant<int, 2> i2;
        const std::integral_constant<int, 4> i4;
        const std::integral_constant<int, 8> i8;
        if (cut.sg == 8) go(d, i8, i8);
        else if (cut.sg == 4) go(d, i4, i8);
        else if (cut.sg == 2) go(d, i2, i4);
        else if (cut.ux == 4) go(d, i1, i4);
        else go(d, i1, i2);
    };
    if (p.D == 128) sized(std::integral_constant<int, 128>());
    else sized(std::integral_constant<int, 64>());
    return hipGetLastError();
}

hipError_t launch_prefix_pack(const void* prefix_v, int L, int Hkv, int D, void* packed, hipStream_t s)
{
    const int TPF = L / KT;
    if (TPF == 0) return hipSuccess;
    const uint16_t* src = static_cast<const uint16_t*>(prefix_v);
    uint16_t* dst = static_cast<uint16_t*>(packed);
    if (D == 128) hipLaunchKernelGGL(vt_pack_kernel<128>, dim3(TPF, Hkv), dim3(512), 0, s, src, dst, Hkv, TPF, 0ll, 0ll);
    else hipLaunchKernelGGL(vt_pack_kernel<64>, dim3(TPF, Hkv), dim3(512), 0, s, src, dst, Hkv, TPF, 0ll, 0ll);
    return hipGetLastError();
}

}  // namespace fdd
