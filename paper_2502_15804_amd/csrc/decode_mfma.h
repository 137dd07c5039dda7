// Decode kernel for bf16 K/V/q on the matrix cores.
//
// Why matrix cores on a bandwidth-bound path: with G = 8 query heads per KV head the
// scores and the weighted sum cost 4*G*D = 4096 flop per retained token, i.e. 8 flop per
// byte streamed.  At the 5.6 TB/s this kernel aims for that is 45 TFLOP/s of plain fp32
// FMAs plus the bf16 unpacking, more than half of what the vector ALUs can issue, and it
// left the vector kernel compute bound at about 1.7 TB/s.  As 16x16 MFMA tiles the same
// contraction keeps the matrix pipes under 5 % busy and leaves the vector ALU only the
// softmax of 4 scores per lane per tile.
//
// Shapes.  A wave works on tiles of 16 tokens.  The G query heads sit in the N dimension,
// padded to 16 with copies of the last head (their columns are computed and never stored):
//     S^T[token][head] = K[token][:] . q[head][:]       4 x mfma_16x16x32 (contract over d)
//     O^T[d][head]    += V^T[d][token] P[token][head]   8 x mfma_16x16x32 (contract over tokens, twice: see below)
// A weight goes into the product as two bf16 numbers, its upper half and what that leaves: the contraction has room for
// 32 numbers where a tile has 16 tokens, and the matrix cores are idle anyway.  Against weights rounded to one bf16 number
// the error of an fp32 output falls from 1.5e-3 to 2.3e-6 of its norm (Llama-70B shape) and that of lse from 1.3e-5 to 4e-8, for
// 0 to 0.6 % of the time; pieces of a pair may then be as large as is fast, where fewer and longer ones cost precision before.
// A lane owns head (lane % 16) in the scores, in P and in O^T alike, so the reference
// maximum, the rescaling and the bf16 weights never leave the lane.
//
// One wave per SIMD means nothing hides a wave's own latencies, so the work on a tile is
// laid out as one LDS round trip, the score MFMAs, a
// handful of vector instructions and the PV MFMAs.  To that end the softmax keeps a stale
// reference maximum m per head: weights are 2^(s - m) with m raised (and O, l rescaled,
// which needs the only cross-lane exchange) only when some score exceeds m by more than
// kBump, so the weights stay below 2^kBump and the result is the same softmax.
//
// Data path.  K and V rows, the query rows of each item and the slot's item list go from
// HBM straight into LDS (global_load_lds_dwordx4, no registers), each wave filling its own
// ring of kStages tiles.  Inside the item loop there is no load the compiler knows about: it
// would answer each with an s_waitcnt vmcnt(0) that also waits for every tile in flight,
// i.e. one exposed memory latency per item.  The workgroup is persistent: it walks the
// items the planner gave its slot, and a wave's ring runs on into the next item while the
// current one is being finished, so only the first tile of a slot waits for HBM.  16-byte
// pieces are stored XOR-swizzled (the swizzle is applied to the global address a lane
// fetches, since the LDS slot of a lane is fixed) so that the row-per-lane reads of K and
// the transposing reads of V (ds_read_b64_tr_b16) spread over all banks.
#pragma once
#include "common.h"

namespace fairkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short i16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(2))) int i32x2_t;
typedef __attribute__((ext_vector_type(2))) uint16_t u16x2_t;

constexpr int kTok = 16;      // tokens per tile (the M of the score MFMA, the K of the PV MFMA)
// Tiles per wave resident in LDS: one being consumed, the other in flight; 64 KB per compute unit are on their way
// at any time.  Three stages (96 KB) fit the LDS for up to 8 columns and were measured side by side on one GPU:
// 0.3-0.4 us slower per launch on the workloads that keep HBM saturated (deeper queues, no more bandwidth) and
// no faster on the one that does not.
constexpr int ring_stages(int) { return 2; }
constexpr float kBump = 8.f;  // log2 units a score may exceed the reference maximum before it is raised

#define FAIRKV_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// One wave-wide direct load HBM -> LDS: lane j's 16 bytes at base + off land at LDS byte
// address lds_base + 16 j (base and lds_base are wave-uniform; lds_base travels in M0).
// Written as inline assembly so that the compiler does not track it: it would otherwise
// drain ALL outstanding loads (s_waitcnt vmcnt(0)) before any LDS read, which defeats the
// multi-stage ring.  The waits are placed by hand with wait_vmcnt below.
// The load is non-temporal (nt): K and V rows are read once per launch, and a stream marked that way does not
// displace or wait on the L2's other contents.  Measured against the same kernel without the hint: 8 % less time per launch on the 188 MB and 174 MB layers, 4 % on the 68 MB layer,
// 14 % on a layer of whole pairs of equal length; the sc0 / sc1 bits on top of it change nothing.
// The base goes through a scalar move for the same reason as the stores of common.h (publish_f32x4); the move is also the
// wait state the hardware wants between a scalar write of M0 and an LDS load that uses it.
__device__ __forceinline__ void load16_to_lds(const void *base, uint32_t off, uint32_t lds_base)
{
    uint64_t from;
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0 nt"
                 : "=&s"(from) : "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}
// N such loads, 1 KB apart in LDS: the instruction's immediate offset moves the LDS address and the global one alike, so
// M0 is written once.  off[i] + 1024 i is the byte offset of load i from base.
template <int N>
__device__ __forceinline__ void load_tile_to_lds(const void *base, const uint32_t (&off)[N], uint32_t lds_base)
{
    static_assert(N == 2 || N == 4, "loads per tile");
    uint64_t from;
    if constexpr (N == 2)
        asm volatile("s_mov_b32 m0, %4\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %1, %0 nt\n\t"
                     "global_load_lds_dwordx4 %2, %0 offset:1024 nt"
                     : "=&s"(from) : "v"(off[0]), "v"(off[1]), "s"(base), "s"(lds_base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %6\n\ts_mov_b64 %0, %5\n\tglobal_load_lds_dwordx4 %1, %0 nt\n\t"
                     "global_load_lds_dwordx4 %2, %0 offset:1024 nt\n\t"
                     "global_load_lds_dwordx4 %3, %0 offset:2048 nt\n\t"
                     "global_load_lds_dwordx4 %4, %0 offset:3072 nt"
                     : "=&s"(from) : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base), "s"(lds_base) : "memory", "m0");
}
// The same without the hint, for what several workgroups read (the query rows of a pair whose pieces sit in
// different slots) or what comes back on every decode step (a layer's item list): 0.3 us per launch less on the
// workloads with many cut pairs or many items, 0.2 us more on a layer of whole pairs.
__device__ __forceinline__ void load16_to_lds_keep(const void *base, uint32_t off, uint32_t lds_base)
{
    uint64_t from;
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                 : "=&s"(from) : "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}

// What lies at an LDS address.
template <class T>
__device__ __forceinline__ __attribute__((address_space(3))) T *lds_at(uint32_t address)
{
    return reinterpret_cast<__attribute__((address_space(3))) T *>(address);
}

// s_waitcnt that waits for the vector-memory counter only (gfx9 encoding: vmcnt is split
// over bits [3:0] and [15:14]; expcnt [6:4] and lgkmcnt [11:8] are left at "no wait").
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Eight E4M3 bytes widened to eight bf16 (exact; v_cvt_scalef32_pk_bf16_fp8 with scale 1 takes two bytes
// at a time: the low or the high half of a dword).
__device__ __forceinline__ bf16x8_t widen8(i32x2_t w)
{
    const bf16x2_t a0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[0], 1.0f, false);
    const bf16x2_t a1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[0], 1.0f, true);
    const bf16x2_t a2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[1], 1.0f, false);
    const bf16x2_t a3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[1], 1.0f, true);
    return bf16x8_t{a0[0], a0[1], a1[0], a1[1], a2[0], a2[1], a3[0], a3[1]};
}

// The maximum / sum over the four lanes of a wave that hold the same column (16 lanes apart).
__device__ __forceinline__ float quarters_max(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);      // rows 0 0 2 2 and 1 1 3 3
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const uint32_t w = __float_as_uint(y);
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quarters_sum(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const uint32_t w = __float_as_uint(y);
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// A whole pair of at most this many tokens is run by one wave alone: it streams all the pair's tiles through its
// own ring and writes the output straight from its registers, with no fold across waves and no barrier.  Short
// pairs shared by four waves leave most of the rings empty (a 32-token pair is two tiles: two waves have nothing
// to fetch and the other two one tile each), so a slot of many short pairs had about one pair in flight at a time
// and each cost a memory round trip; alone, four pairs stream side by side.
constexpr int kSoloTokens = FAIRKV_SHORT_PAIR_TOKENS;

// Items per fill of a wave's list in registers (ItemList): one per lane.  Between two fills the ring drains, and the list and the next tile
// are waited for one after the other; with the 128 items of a table in LDS that came half as often.  us per layer with such a table and
// now, 8 KV heads, 24 to 56 tokens a pair: slots of 63 items 82.2 and 81.6, 67 86.5 and 87.3, 75 96.4 and 94.9, 100 127.3 and 125.4, 133 186.6
// and 182.5; on 8-bit caches 61.0 and 58.4, 63.6 and 62.4, 71.6 and 69.9, 89.8 and 89.0, 121.9 and 121.4.
constexpr int kList = 64;

// A wave's own copy of (part of) its slot's item list: lane j holds item j.  A field of an item is one v_readlane away,
// where a table in LDS costs a wait of 130 cycles for each of the handful of fields that start an item, and a barrier
// after the lanes that check the items have written it: with the arguments held (arrive_together), from a workgroup's first
// instruction to its first tile 6100 -> 4500 cycles on an idle memory system, us per layer for one sequence 9.9 -> 9.4, for the
// Llama-70B shape 16.5 -> 16.2, with an 8-bit cache 12.2 -> 11.6.  An item that does not belong to this problem gets n_chunks 0
// and no tokens.
struct ItemList {
    uint32_t row_lo, row_hi;
    int32_t n, b, h, chunk, n_chunks, part;
    __device__ __forceinline__ int64_t row(int i) const
    {
        return static_cast<int64_t>((static_cast<uint64_t>(__builtin_amdgcn_readlane(row_hi, i)) << 32) | static_cast<uint32_t>(__builtin_amdgcn_readlane(row_lo, i)));
    }
    __device__ __forceinline__ int tokens(int i) const { return __builtin_amdgcn_readlane(n, i); }
    __device__ __forceinline__ int head(int i) const { return __builtin_amdgcn_readlane(h, i); }
    __device__ __forceinline__ bool valid(int i) const { return __builtin_amdgcn_readlane(n_chunks, i) != 0; }
    __device__ __forceinline__ int query_group(int qg_stride, int i) const
    {
        return __builtin_amdgcn_readlane(b, i) * qg_stride + __builtin_amdgcn_readlane(h, i);
    }
    __device__ __forceinline__ bool last_chunk(int i) const
    {
        return __builtin_amdgcn_readlane(chunk, i) == __builtin_amdgcn_readlane(n_chunks, i) - 1;
    }
    __device__ __forceinline__ Piece piece(const CallArgs &a, int i, float v_mul) const
    {
        return Piece{__builtin_amdgcn_readlane(b, i) * a.Hkv + head(i), query_group(a.q_len * a.Hkv, i), __builtin_amdgcn_readlane(part, i),
                     __builtin_amdgcn_readlane(chunk, i), __builtin_amdgcn_readlane(n_chunks, i), v_mul};
    }
};
// Lane j's item out of the fetched records in LDS, checked without a branch (lanes past the list hold whatever is there).
__device__ __forceinline__ ItemList item_list(const CallArgs &a, const fairkv_item *raw, int lane)
{
    const uint4 x = reinterpret_cast<const uint4 *>(raw + lane)[0], y = reinterpret_cast<const uint4 *>(raw + lane)[1];
    ItemList e{x.x, x.y, max(static_cast<int>(x.z), 0), static_cast<int>(x.w), static_cast<int>(y.x), static_cast<int>(y.y),
               static_cast<int>(y.z), static_cast<int>(y.w)};
    // Unsigned compares, so that negative numbers fail; n_rows and n_parts are not negative.  With row's upper half no more than
    // n_rows', row + n does not wrap around.
    auto u = [](int32_t v) __attribute__((always_inline)) { return static_cast<uint32_t>(v); };
    const uint64_t end = ((static_cast<uint64_t>(e.row_hi) << 32) | e.row_lo) + u(e.n), n_rows = static_cast<uint64_t>(a.n_rows);
    bool ok = u(e.b) < u(a.B);       // combined without a branch
    ok &= u(e.h) < u(a.Hkv);
    ok &= e.row_hi <= static_cast<uint32_t>(n_rows >> 32);
    ok &= end <= n_rows;
    ok &= u(e.chunk) < u(e.n_chunks);
    ok &= u(e.n_chunks) <= u(a.n_parts);
    ok &= u(e.part - e.chunk) <= u(a.n_parts - e.n_chunks);
    e.n = ok ? e.n : 0;
    e.n_chunks = ok ? e.n_chunks : 0;
    return e;
}

// KV8: K and V are stored as 8-bit floats (E4M3), one byte per element, and widened to bf16 in registers
// (exactly: every E4M3 value is a bf16 value), so the arithmetic is that of the bf16 path.  A row is half as
// long, so a stage holds 32 tokens instead of 16 in the same 8 KB, and a step works on two 16-token score
// tiles and one 32-token P.V product:
//     S^T = K . q^T    2 x 4 x mfma_16x16x32 on K widened 8 bytes at a time
//     O^T += V^T . P   8 x mfma_16x16x32; the contraction index k = 8 lq + r of a lane stands for token
//                      4 lq + r of the first score tile (r < 4) or of the second (r >= 4), which is how the
//                      lane's own eight weights are laid out already; V^T comes out of the LDS through the
//                      8-bit transposing read: lane i of a 16-lane group addresses the 8 bytes (token
//                      t_(i/2), columns 8 (i%2) .. +7) and lane j receives byte j%8 of the fragments
//                      j/8, j/8 + 2, ..., i.e. column j of tokens t_0 .. t_7 (layout checked on the GPU).
// TRACE: the measurement instantiation behind fairkv_decode_attn_trace; it writes wall-clock stamps of its phases
// (see trace_stamp) and is otherwise the same code.
// SOLO: the plan has short whole pairs (at most kSoloTokens tokens) and they are run by single waves.  Plans
// without any run an instantiation without that code: its presence alone cost 0.3-0.4 us per launch on every
// workload (measured side by side on one GPU), on a kernel of under 20 us.
template <int D, int G, bool DEEP, bool KV8, bool SOLO, bool TRACE = false>
__global__ __launch_bounds__(kThreads, 1) void fairkv_decode_mfma_kernel(DecodeArgs args)
{
    static_assert(D == 64 || D == 128, "head_dim");
    static_assert(G >= 1 && G <= 16, "query heads of a group fit the N dimension");
    constexpr int TOK = KV8 ? 2 * kTok : kTok;          // tokens per stage and per step
    constexpr int kStages = ring_stages(G);
    // Tiles per wave the early start requests: one.  With the whole ring requested at once (two tiles per wave,
    // 16 MB over the chip before anything has come back) the memory system serves the 1024 waves in no fair
    // order, some workgroups see their first tile a microsecond after the others and, each having a fixed share of
    // the work, finish that much later; the second stage is requested when the item list has landed instead.
    // Side by side on one GPU: 0.4-0.5 us per launch less on all four workloads.
    constexpr int kEarly = 1;
    static_assert(kStages == 2 && kEarlyTok >= kEarly * kWaves * TOK && kEarlyTok < 512, "ring, early start");
    static_assert(sizeof(fairkv_item) == 32, "two 16-byte pieces per item");
    constexpr int QROWB = D * 2;             // bytes per q row (bf16)
    constexpr int ROWB = KV8 ? D : D * 2;    // bytes per K or V row
    constexpr int PPR = ROWB / 16;           // 16-byte pieces per row: 16 or 8
    constexpr int RPI = 64 / PPR;            // rows one wave-wide 16-byte load covers
    constexpr int LPT = TOK / RPI;           // wave-wide loads per K (or V) tile
    constexpr int TILEB = TOK * ROWB;        // bytes of one K (or V) tile
    constexpr int STAGEB = 2 * TILEB;        // K tile then V tile
    constexpr int LOADS = 2 * LPT;           // vector-memory instructions per stage
    constexpr int NSL = D / 32;              // d slices of the score contraction
    constexpr int NDB = D / 16;              // 16-wide d blocks of the output
    constexpr int QBYTES = G * QROWB;        // the G query rows of a group are contiguous in q
    constexpr int QL = (QBYTES + 1023) / 1024;   // wave-wide loads per query block
    constexpr int QBUF = QL * 1024;

    __shared__ __attribute__((aligned(1024))) char lds[kWaves * kStages * STAGEB];
    __shared__ __attribute__((aligned(1024))) char qlds[kWaves * kStages * QBUF];   // a query block per ring stage: the tiles in
                                                                                    // the ring may belong to kStages different items
    __shared__ __attribute__((aligned(1024))) fairkv_item raw[kList];         // items as fetched
    // Two sets, used in turn, so that one barrier per item is enough; one set and a second barrier with 16 columns, where
    // at D = 128 two sets do not fit beside the rings (at D = 64 they would).
    constexpr int kSets = G <= 8 ? 2 : 1;
    __shared__ __attribute__((aligned(16))) float st_o[kSets][kWaves * G * kStRow<D>];
    __shared__ __attribute__((aligned(16))) float st_ml[kSets][kWaves * G * 2];
    __shared__ int32_t roles[kPend];
    Piece pend[kPend] = {};
    int set = 0;
    int n_pend = 0;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: loop control is scalar
    const int l16 = lane & 15;      // head in B/C operands, token row in the K operand, d in the V operand
    const int lq = lane >> 4;       // which quarter of the contraction index this lane feeds

    if constexpr (TRACE) trace_stamp(args, kTraceStart, threadIdx.x == 0);
    // The kernel arguments are asked for here and waited for below (arrive_together): what depends on the lane alone is worked out in between.  Without
    // the barrier the compiler asks for them behind those 95 instructions.  With the rows of the first tile requested before its queries and
    // the end of an item read ahead of its tiles (both below), us per layer: Llama-70B shape 16.03 -> 15.72, the same with an 8-bit cache
    // 10.98 -> 10.78, one sequence 8.52 -> 8.40, Pareto budgets at batch 128 20.78 -> 20.44; the 24B shape (32.9) within the noise.
    const SlotStart slot = slot_start(args);
    const CallArgs held = args;
    HeadFactors factors{};
    if constexpr (KV8) factors = args.factors;
    __builtin_amdgcn_sched_barrier(0);
    // Lane j of load i of a tile fills LDS slot (row i*RPI + j/PPR, column j%PPR); the piece it
    // fetches is column ^ swizzle(row).  Byte offsets of that piece inside a full K and V tile:
    const int ld_row = lane / PPR, ld_col = lane % PPR;
    uint32_t k_off[LPT], v_off[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int r = i * RPI + ld_row;
        k_off[i] = ld_row * ROWB + (ld_col ^ (r % PPR)) * 16;             // plus i * 1024, which the load adds
        v_off[i] = ld_row * ROWB + (ld_col ^ ((2 * r) % PPR)) * 16;
        asm volatile("" : "+v"(k_off[i]), "+v"(v_off[i]));
    }
    const uint32_t ring_lds =
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FAIRKV_LDS_PTR(lds))) + wave * (kStages * STAGEB);
    const uint32_t q_lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FAIRKV_LDS_PTR(qlds))) + wave * (kStages * QBUF);
    const char *q_ring = qlds + wave * (kStages * QBUF);
    const uint32_t raw_lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FAIRKV_LDS_PTR(raw))) + (wave & 1) * 1024;
    const int list_item = 32 * (wave & 1) + (lane >> 1);
    // Where a lane reads its operands in a tile: the K row l16 (pieces 4 s + lq) and, through the
    // transposing read, 4 d's of V row 4 lq + l16/4 (lane j of a 16-lane group receives element
    // j%4 of the rows its lanes 4i + j/4 address).
    // (8-bit caches: 8 bytes of K row l16 or 16 + l16 at byte 32 s + 8 lq; for V the fragment this
    // lane addresses in the transposing read, see above.)
    // LDS addresses in the stage of the tile that is next to be consumed.
    constexpr int NKR = KV8 ? 2 * NSL : NSL;
    uint32_t k_rd[NKR], v_rd[NDB];
    if constexpr (!KV8) {
#pragma unroll
        for (int s = 0; s < NSL; ++s) k_rd[s] = ring_lds + l16 * ROWB + ((4 * s + lq) ^ (l16 % PPR)) * 16;
        const int vrow = 4 * lq + (l16 >> 2), vsub = l16 & 3;
#pragma unroll
        for (int nb_ = 0; nb_ < NDB; ++nb_)
            v_rd[nb_] = ring_lds + TILEB + vrow * ROWB + (((2 * nb_ + (vsub >> 1)) ^ ((2 * vrow) % PPR)) * 16) + (vsub & 1) * 8;
    } else {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int s = 0; s < NSL; ++s) {
                const int row = 16 * u + l16;
                k_rd[u * NSL + s] = ring_lds + row * ROWB + (((2 * s + (lq >> 1)) ^ (row % PPR)) * 16) + (lq & 1) * 8;
            }
        const int r = l16 >> 1;                                            // which of the lane group's 8 tokens
        const int vrow = r < 4 ? 4 * lq + r : 16 + 4 * lq + (r - 4);
#pragma unroll
        for (int nb_ = 0; nb_ < NDB; ++nb_)
            v_rd[nb_] = ring_lds + TILEB + vrow * ROWB + ((nb_ ^ ((2 * vrow) % PPR)) * 16) + (l16 & 1) * 8;
    }
#pragma unroll
    for (int s = 0; s < NKR; ++s) asm volatile("" : "+v"(k_rd[s]));
#pragma unroll
    for (int nb_ = 0; nb_ < NDB; ++nb_) asm volatile("" : "+v"(v_rd[nb_]));

    arrive_together(held, slot);
    const char *const q_base = static_cast<const char *>(held.q), *const k_base = static_cast<const char *>(held.k);
    const int64_t v_minus_k = static_cast<const char *>(held.v) - k_base;
    const int g_shift = held.g_shift;
    const int i_begin = slot.i_begin, i_end = slot.i_end;
    if (i_end <= i_begin) return;   // an idle slot
    // Fetch of the kList items that start at `first`: one load by each wave, 32 items by waves 0 and 2, the next 32 by waves 1 and 3
    // (a condition on the wave costs more than the second load).  Past the end of the slot's list the last item is read again.
    auto fetch_items = [&](const fairkv_item *items, int first) __attribute__((always_inline)) {
        load16_to_lds_keep(items + first, min(list_item, i_end - first - 1) * 32 + (lane & 1) * 16, raw_lds);
    };
    fetch_items(held.items, i_begin);

    // The fetch cursor (f_*) stands on this wave's next tile of item f_item and runs ahead of the compute cursor, possibly into
    // later items: f_left tokens of the item from that tile on (none or less: the wave is through with the item), f_k the address
    // of its first K row, f_step tokens from one of the wave's tiles to the next.  An item's tiles go to the waves in turn (wave,
    // wave + kWaves, ...), or all to one wave that runs the item alone.  `ahead` tiles are fetched and not yet consumed, the
    // oldest in stage c_stage.  The query block of an item is requested together with the wave's first tile of it (f_new), into
    // the q buffer of that tile's stage, so it has landed when the tile has; next_q says that the newest tile came with one.
    constexpr int kShared = kWaves * TOK;
    int f_item = 0, f_left = 0, f_step = kShared, f_qg = 0, f_stage = 0, c_stage = 0, ahead = 0;
    uint64_t f_k = 0;
    bool f_new = true, next_q = false;

    // The cursor's tile into the next stage: LOADS loads, QL more for the queries of another item.  Rows past the end of the item
    // re-read its last row (finite data with weight 0).
    auto fetch_rows = [&]() __attribute__((always_inline)) {
        const char *k = reinterpret_cast<const char *>(f_k), *v = k + v_minus_k;
        const uint32_t k_lds = ring_lds + f_stage * STAGEB, v_lds = k_lds + TILEB;
        if (f_left >= TOK) {
            load_tile_to_lds<LPT>(k, k_off, k_lds);
            load_tile_to_lds<LPT>(v, v_off, v_lds);
        } else {
#pragma unroll
            for (int i = 0; i < LPT; ++i) {
                const int r = i * RPI + ld_row, row = min(r, f_left - 1);
                load16_to_lds(k, row * ROWB + (ld_col ^ (r % PPR)) * 16, k_lds + i * 1024);
                load16_to_lds(v, row * ROWB + (ld_col ^ ((2 * r) % PPR)) * 16, v_lds + i * 1024);
            }
        }
    };
    auto fetch_queries = [&](const uint32_t (&q_off)[QL]) __attribute__((always_inline)) {
        const char *src = q_base + (static_cast<size_t>(f_qg) << g_shift) * QROWB;
#pragma unroll
        for (int i = 0; i < QL; ++i) load16_to_lds_keep(src, q_off[i], q_lds + f_stage * QBUF + i * 1024);
    };
    auto step_on = [&]() __attribute__((always_inline)) {
        next_q = f_new;
        f_new = false;
        f_left -= f_step;
        f_k += static_cast<uint32_t>(f_step) * ROWB;
        f_stage ^= 1;
        ++ahead;
    };
    auto row_address = [&](int64_t row) __attribute__((always_inline)) { return reinterpret_cast<uint64_t>(k_base) + row * ROWB; };

    // Early start: the kernel arguments carry query group, first row and the first kEarlyTok tokens' worth of the length of the
    // slot's first item, so the item list, the first query
    // block and the first tile are all requested at once, before anything has come back from memory; the rows of the tile first, which need the
    // least to be worked out.
    const int n0 = static_cast<int>(slot.np & 0x1ffu);
    if (n0 > 0) {
        f_qg = static_cast<int>(slot.np >> 9);
        f_k = row_address(static_cast<int64_t>(slot.row) + wave * TOK);      // the early start always shares the first item among the waves
        f_left = n0 - wave * TOK;
        if (f_left > 0) fetch_rows();
    }
    // Lane offsets of the G query rows of a query group: column c = (new token c >> g_shift, head c & mask) of
    // q [B][q_len][Hq][D]: the heads of one new token are contiguous, the new tokens are Hq rows apart.
    uint32_t q_off[QL];
#pragma unroll
    for (int i = 0; i < QL; ++i) {
        const int o = min(i * 1024 + lane * 16, QBYTES - 16);      // byte o of the [G][QROWB] image in LDS
        q_off[i] = col_row(g_shift, held.Hq, o / QROWB) * QROWB + o % QROWB;
    }
    if (n0 > 0 && f_left > 0) {
        fetch_queries(q_off);
        step_on();
    }
    auto fetch_next = [&]() __attribute__((always_inline)) {
        if (f_new) fetch_queries(q_off);
        fetch_rows();
        step_on();
    };
    const ArgLanes arg_lanes(held);
    auto call_args = [&]() __attribute__((always_inline)) {
        CallArgs a = arg_lanes.get();
        if constexpr (TRACE) a.trace = args.trace;
        return a;
    };
    const float scale_log2 = held.scale_log2;
    const int q_len = held.q_len, qg_stride = q_len * held.Hkv;      // query groups of a sequence
    // 8-bit caches: lane h holds scale_log2 times the K factor of KV head h (modulo kScaleHeads), lane kScaleHeads + h v_scale
    // times its V factor
    float head_mul = 0.f;
    if constexpr (KV8) {
        head_mul = lane_values(factors.k, factors.v) * (lane < kScaleHeads ? scale_log2 : held.v_scale);
    }

    const char *q_rd = q_ring + min(l16, G - 1) * QROWB + lq * 16;
    const int col_hidden = q_len - 1 - (min(l16, G - 1) >> g_shift);      // rows at a pair's end that the lane's column does not see

    // A wave's share of an item: outputs, reference maximum of the lane's head, this lane's share of the weights.  Made ready while the
    // first tile is on its way, and after an item for the next.
    f32x4_t o[NDB];
    float m_run, l_run;
    auto begin_item = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int nb_ = 0; nb_ < NDB; ++nb_) o[nb_] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        m_run = -INFINITY;
        l_run = 0.f;
    };
    begin_item();
    ItemList list{};
    for (int batch = i_begin; batch < i_end; batch += kList) {
        const int nb = min(kList, i_end - batch);
        const bool early = n0 > 0 && batch == i_begin;
        // short whole pairs go to single waves in turn (not the item the early start has already shared out)
        auto owner_of = [&](int i, int n) __attribute__((always_inline)) {
            return SOLO && __builtin_amdgcn_readlane(list.n_chunks, i) == 1 && n <= kSoloTokens && !(early && i == 0) ? i % kWaves : -1;
        };
        // first token of this wave's first tile of an item, as far from the end as `n` says: none left if another wave runs it
        auto left_of = [&](int n, int owner) __attribute__((always_inline)) {
            return SOLO && owner >= 0 ? (owner == wave ? n : 0) : n - wave * TOK;
        };
        auto seek = [&](int item) __attribute__((always_inline)) {           // point the fetch cursor at an item of the list
            f_item = item;
            f_left = 0;
            f_new = true;
            if (item < nb) {
                const int n = list.tokens(item), owner = owner_of(item, n);
                f_left = left_of(n, owner);
                f_step = SOLO && owner >= 0 ? TOK : kShared;
                f_k = row_address(list.row(item) + (SOLO && owner >= 0 ? 0 : wave * TOK));
                f_qg = list.query_group(qg_stride, item);
            }
        };
        auto top_up = [&]() __attribute__((always_inline)) {
            while (ahead < kStages && f_item < nb) {
                if (f_left > 0)
                    fetch_next();
                else
                    seek(f_item + 1);
            }
        };
        if (batch != i_begin) {
            __syncthreads();                  // nobody still reads the previous list
            fetch_items(arg_lanes.get().items, batch);
        }
        // the items have landed once only what was requested after them, the early start's tile and queries, is outstanding
        if (ahead > 0)
            wait_vmcnt<LOADS + QL>();
        else
            wait_vmcnt<0>();
        __syncthreads();
        list = item_list(arg_lanes.get(), raw, lane);
        if (early) {                          // the first tile of item 0 is on its way, as far as n0 said: on to its full length
            const int n = n0 < kEarlyTok ? n0 : max(list.tokens(0), kEarlyTok);
            if (lane == 0) list.n = n;
            f_left += n - n0;
        } else {
            seek(0);
        }
        if constexpr (TRACE)
            if (batch == i_begin) trace_stamp(args, kTraceTable, threadIdx.x == 0);

        for (int ci = 0; ci < nb; ++ci) {
            const int n = list.tokens(ci), owner = owner_of(ci, n);
            if (SOLO && owner >= 0 && owner != wave) continue;      // another wave runs this pair alone
            const bool last_chunk = list.last_chunk(ci);
            const int scale_h = list.head(ci) % kScaleHeads;
            top_up();
            // tokens of the item from the wave's next tile on
            int left = left_of(n, owner);
            const int step = SOLO && owner >= 0 ? TOK : kShared;
            // scores to log2 units: the same factor for every pair unless an 8-bit cache has a scale per KV head
            const float s_mul = KV8 ? lane_value(head_mul, scale_h) : scale_log2;
            // Several new tokens per sequence: their K/V rows are the last q_len rows of the pair, and
            // new token j does not see the rows of the new tokens after it.  Only the pair's last
            // chunk holds such rows.
            const int hidden_max = last_chunk ? q_len - 1 : 0;
            const int hidden = last_chunk ? col_hidden : 0;
            bf16x8_t qb[NSL];
            // What the end of the item needs, read out of the lanes here, where the wave waits for a tile anyway, and not behind the last tile, where
            // these 35 instructions stand between it and the output.  With the fold's reads of both its columns in one go, us per layer:
            // Llama-70B shape 15.74 -> 15.67, the same with an 8-bit cache 10.93 -> 10.84, 24B shape with 16 columns 37.27 -> 37.12.
            // Not with short pairs on 8-bit caches of D = 64: what is held takes up to 20 scalar registers more than there are (34 spilled instead of 9).
            // us per layer ahead, behind, 8 KV heads, 110 sequences of 60 tokens a pair: 8 columns 9.93, 9.80, 16 columns 10.25, 10.17; Pareto
            // budgets at batch 100: 10.92, 10.78 and 11.35, 11.19.  At D = 128 and on bf16 caches ahead is the faster by 0 to 1 %.
            constexpr bool kEndAhead = !(KV8 && SOLO && D == 64);
            auto piece = [&](const CallArgs &call) __attribute__((always_inline)) {
                return list.piece(call, ci, KV8 ? lane_value(head_mul, kScaleHeads + scale_h) : call.v_scale);
            };
            const CallArgs a_ahead = kEndAhead ? call_args() : CallArgs{};
            const Piece pc_ahead = kEndAhead ? piece(a_ahead) : Piece{};

            for (bool fresh = true; left > 0; fresh = false) {
                // The tile has landed once no more is outstanding than was requested after it: the other tile of the ring
                // and its query block.
                if (ahead == 1)
                    wait_vmcnt<0>();
                else if (!next_q)
                    wait_vmcnt<LOADS>();
                else
                    wait_vmcnt<LOADS + QL>();
                if constexpr (TRACE)
                    if (batch == i_begin && ci == 0 && fresh) trace_stamp(args, kTraceFirstTile, threadIdx.x == 0);
                if (fresh) {
                    // q as the B operand of the score MFMA: lane holds q[head l16][32 s + 8 lq .. +8].  Heads
                    // >= G repeat head G-1: their columns of the products are computed and never stored.
#pragma unroll
                    for (int s = 0; s < NSL; ++s)
                        qb[s] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(q_rd + c_stage * QBUF + s * 64));
                }

                constexpr int NS = TOK / 4;                          // scores per lane
                float sv[NS];
                const bool masked = left - hidden_max < TOK;         // some column does not see the whole tile
                // ---- every LDS read of the tile, issued together; scores: S^T[token][head l16], in log2 units
                i32x2_t vt8[NDB];
                i16x4_t vt[NDB];
                if constexpr (KV8) {
                    i32x2_t kw[NKR];
#pragma unroll
                    for (int s = 0; s < NKR; ++s) kw[s] = *lds_at<i32x2_t>(k_rd[s]);
#pragma unroll
                    for (int nb_ = 0; nb_ < NDB; ++nb_) vt8[nb_] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(lds_at<i32x2_t>(v_rd[nb_]));
                    // two 16-token tiles: token 16 u + 4 lq + i
                    f32x4_t sacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int s = 0; s < NSL; ++s)
                            sacc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(widen8(kw[u * NSL + s]), qb[s], sacc[u], 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < NS; ++r) sv[r] = sacc[r >> 2][r & 3] * s_mul;
                } else {
                    bf16x8_t kw[NSL];
#pragma unroll
                    for (int s = 0; s < NSL; ++s) kw[s] = *lds_at<bf16x8_t>(k_rd[s]);
#pragma unroll
                    for (int nb_ = 0; nb_ < NDB; ++nb_) vt[nb_] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_at<i16x4_t>(v_rd[nb_]));
                    f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};             // token 4 lq + i
#pragma unroll
                    for (int s = 0; s < NSL; ++s) sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kw[s], qb[s], sacc, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < NS; ++r) sv[r] = sacc[r] * s_mul;
                }
                if (masked) {
                    const int seen = left - hidden - 4 * lq;
#pragma unroll
                    for (int r = 0; r < NS; ++r)
                        if (16 * (r >> 2) + (r & 3) >= seen) sv[r] = -INFINITY;
                }

                // ---- raise the reference maximum if some score is far above it (always on the first tile, where there is
                //      nothing to rescale yet)
                float mx = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
                if constexpr (KV8) mx = fmaxf(mx, fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
                if (__builtin_amdgcn_ballot_w64(mx > m_run + kBump) != 0) {
                    const float m_new = fmaxf(m_run, quarters_max(mx));
                    if (!fresh) {
                        const float alpha = m_new == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
                        l_run *= alpha;
#pragma unroll
                        for (int nb_ = 0; nb_ < NDB; ++nb_)
#pragma unroll
                            for (int i = 0; i < 4; ++i) o[nb_][i] *= alpha;
                    }
                    m_run = m_new;
                }

                // ---- weights ----------------------------------------------------------------------
                float p[NS];
#pragma unroll
                for (int r = 0; r < NS; ++r) p[r] = __builtin_amdgcn_exp2f(sv[r] - m_run);
                if (masked) {     // a column that has seen nothing yet has m = -inf: its weights are 0, not exp2(nan)
#pragma unroll
                    for (int r = 0; r < NS; ++r)
                        if (sv[r] == -INFINITY) p[r] = 0.f;
                }

                // ---- O^T[d][head] += V^T P ---------------------------------------------------------
                if constexpr (KV8) {      // the sum of the weights is that of the rounded ones, so out is an exact convex combination of V rows
                    uint32_t pw[NS / 2];
#pragma unroll
                    for (int r = 0; r < NS; r += 2) {
                        pw[r / 2] = pack_bf16(p[r], p[r + 1]);
                        l_run = l_run + bf16_lo(pw[r / 2]) + bf16_hi(pw[r / 2]);
                    }
                    const bf16x8_t pb = __builtin_bit_cast(bf16x8_t, uint4{pw[0], pw[1], pw[2], pw[3]});
#pragma unroll
                    for (int nb_ = 0; nb_ < NDB; ++nb_) o[nb_] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(widen8(vt8[nb_]), pb, o[nb_], 0, 0, 0);
                } else {
                    // A weight is the sum of two bf16 numbers: its upper half, and what that leaves, rounded, in the other half of the contraction.
                    // Both are positive if the weight is, so an infinite V stays one: where nothing is left, or less than bf16 has, the
                    // rest is the smallest number of bf16, 2^-133 (0 for a weight of 0).  The smallest weight is 2^-126 and the largest at least 1.
                    // (The last row of a tile that is not full is read again with weight 0, which makes a NaN of an infinite V there.)  0 to 0.2 % of a launch.
                    uint32_t upper[NS / 2], rest[NS / 2], ones = 0x00010001u;
                    asm("" : "+s"(ones));      // a minimum with a known 1 becomes two compares and two selects
#pragma unroll
                    for (int r = 0; r < NS; r += 2) {
                        l_run = l_run + p[r] + p[r + 1];
                        upper[r / 2] = __builtin_amdgcn_perm(__float_as_uint(p[r + 1]), __float_as_uint(p[r]), 0x07060302u);
                        const float left0 = p[r] - bf16_hi(__float_as_uint(p[r])), left1 = p[r + 1] - bf16_hi(__float_as_uint(p[r + 1]));      // exact
                        const u16x2_t floor = __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, upper[r / 2]), __builtin_bit_cast(u16x2_t, ones));
                        rest[r / 2] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, pack_bf16(left0, left1)), floor));
                    }
                    const bf16x8_t pb = __builtin_bit_cast(bf16x8_t, uint4{upper[0], upper[1], rest[0], rest[1]});
#pragma unroll
                    for (int nb_ = 0; nb_ < NDB; ++nb_) {
                        const uint2 x = __builtin_bit_cast(uint2, vt[nb_]);
                        o[nb_] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, uint4{x.x, x.y, x.x, x.y}), pb, o[nb_], 0, 0, 0);
                    }
                }
                const uint32_t to_other = c_stage == 0 ? STAGEB : -STAGEB;
#pragma unroll
                for (int s = 0; s < NKR; ++s) k_rd[s] += to_other;
#pragma unroll
                for (int nb_ = 0; nb_ < NDB; ++nb_) v_rd[nb_] += to_other;
                c_stage ^= 1;
                --ahead;
                left -= step;
                if (left > 0) top_up();
            }

            if constexpr (TRACE) {
                if (batch == i_begin && ci == 0) trace_stamp(args, kTraceItem0Streamed, threadIdx.x == 0);
                if (batch + ci == i_end - 1) trace_stamp(args, kTraceLastStreamed, threadIdx.x == 0);
            }
            // ---- fold the four token quarters of l, stage this wave's result, finish the item ------
            l_run = quarters_sum(l_run);
            const CallArgs a = kEndAhead ? a_ahead : call_args();
            const Piece pc = kEndAhead ? pc_ahead : piece(a);
            if (SOLO && owner >= 0) {
                // This wave has seen the whole pair: out = O / l and lse straight from its registers.  A lane holds
                // coordinates 16 nb + 4 lq .. + 3 of head l16.
                if (l16 < G && pc.n_chunks != 0) {
#pragma unroll
                    for (int nb_ = 0; nb_ < NDB; ++nb_)
                        write_out4<D>(a, pc.qg, l16, 16 * nb_ + 4 * lq, make_float4(o[nb_][0], o[nb_][1], o[nb_][2], o[nb_][3]), m_run,
                                      l_run, pc.v_mul);
                }
                begin_item();
                continue;
            }
            if (l16 < G) {
#pragma unroll
                for (int nb_ = 0; nb_ < NDB; ++nb_)
                    *reinterpret_cast<float4 *>(st_o[set] + (wave * G + l16) * kStRow<D> + 16 * nb_ + 4 * lq) =
                        make_float4(o[nb_][0], o[nb_][1], o[nb_][2], o[nb_][3]);
                if (lq == 0) {
                    *reinterpret_cast<float2 *>(st_ml[set] + (wave * G + l16) * 2) = make_float2(m_run, l_run);
                }
            }
            if (pc.n_chunks != 0) {
                item_epilogue<D, G, DEEP, TRACE>(a, pc, st_o[set], st_ml[set], pend, n_pend, roles);
                if constexpr (kSets == 2)
                    set ^= 1;
                else
                    __syncthreads();
            }
            // Plans without short pairs have few items per slot: what the last one would make ready for a next is left out.  With short pairs the
            // condition costs more than it saves, 30 vector registers among it.  us per layer with it everywhere, and now, 8 KV heads: 110
            // sequences of 60 tokens a pair, one query head per KV head 10.84 and 10.60, two 11.09 and 10.81, eight 11.64 and 11.58, on 8-bit caches
            // two 11.13 and 10.93, eight 12.07 and 11.89; Pareto budgets at batch 100 13.84 and 13.60, 14.35 and 14.03, 15.04 and 14.93, 12.17 and
            // 12.04, 13.13 and 13.00.
            if (SOLO || batch + ci + 1 < i_end) begin_item();
            if constexpr (TRACE)
                if (batch == i_begin && ci == 0) trace_stamp(args, kTraceItem0Done, threadIdx.x == 0);
        }
        wait_vmcnt<0>();   // nothing of this batch may still be landing in the rings
    }
    if (n_pend > 0) flush_pending<D, G, DEEP, TRACE>(call_args(), pend, n_pend, roles);
    if constexpr (TRACE) trace_stamp(args, kTraceEnd, threadIdx.x == 0);
}

}  // namespace fairkv
