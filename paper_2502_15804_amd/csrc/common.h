// Shared pieces of the decode kernels: argument block, layout facts, small device helpers,
// and the workgroup epilogue that folds the waves of a workgroup and writes either the
// final output (an item that is a whole pair) or the item's partial result.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdint>

#include "fairkv.h"
#include "rows.h"

namespace fairkv {

constexpr int kWaves = 4;                 // waves per workgroup
constexpr int kThreads = kWaves * 64;
constexpr int kTile = 64;                 // tokens a wave handles per step: one per lane
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;

__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
    return x;
}

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Two fp32 numbers rounded to bf16 (to nearest even), the first in the lower half.
typedef __attribute__((ext_vector_type(2))) float f2_t;
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2_t{lo, hi}, bf16x2_t));
}

// Four consecutive outputs: element base + off of out, both multiples of 4 (out is 16-byte aligned), base the same for
// the whole wave.  Results are written once and not read again by this launch: non-temporal stores keep them from
// waiting in the L2 for the write-back at the end of the kernel (0.45 us per launch on a layer of whole pairs, 0.25 us
// on the many-small-pairs workload).
__device__ __forceinline__ void store_out4(void *out, int out_dtype, size_t base, uint32_t off, float4 x)
{
    if (out_dtype == FAIRKV_F32) {
        typedef __attribute__((ext_vector_type(4))) float f4;
        __builtin_nontemporal_store(f4{x.x, x.y, x.z, x.w}, reinterpret_cast<f4 *>(static_cast<float *>(out) + base + off));
    } else {
        typedef __attribute__((ext_vector_type(2))) uint32_t u2;
        const u2 w = {pack_bf16(x.x, x.y), pack_bf16(x.z, x.w)};
        __builtin_nontemporal_store(w, reinterpret_cast<u2 *>(static_cast<uint16_t *>(out) + base + off));
    }
}

__device__ __forceinline__ int64_t uniform64(int64_t x)   // a wave-uniform value, moved to scalar registers
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<int>(x));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<int>(x >> 32));
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}
// ... and a pointer
template <class T>
__device__ __forceinline__ T *uniform_ptr(T *p)
{
    return reinterpret_cast<T *>(uniform64(static_cast<int64_t>(reinterpret_cast<uintptr_t>(p))));
}

// Partial results travel between workgroups that may sit on different XCDs, whose L2 caches
// are not coherent with each other.  Stores and loads at agent scope (the sc1 bit) go through to the
// level all XCDs share, without the cache-wide write-back and invalidate that a device fence costs
// (measured: tens of microseconds per launch).
// Stores of four (two) floats at byte off of a base that is the same for the wave; 16-byte (8-byte) aligned.
// The compiler does not see these stores: drain_vmem() waits for them, and the wait states it would keep around them are
// kept here.  Behind them: the s_nop stands for the two between a store of more than 8 bytes and an instruction that
// overwrites the store's data registers (without it a build in which the very next vector instruction did so stored that
// instruction's result).  In front: a memory instruction may read a scalar register no sooner than five wait states after
// a vector instruction wrote it, which is what the base may be (uniform_ptr ends in a readfirstlane, a spilled register
// comes back with a readlane); a scalar instruction waits for it by itself, so the base goes through a scalar move.
typedef __attribute__((ext_vector_type(4))) float f4_t;
__device__ __forceinline__ void publish_f32x4(float *base, uint32_t off, float4 x)
{
    const f4_t v = {x.x, x.y, x.z, x.w};
    uint64_t at;
    asm volatile("s_mov_b64 %0, %3\n\tglobal_store_dwordx4 %1, %2, %0 sc1\n\ts_nop 1"
                 : "=&s"(at) : "v"(off), "v"(v), "s"(uniform_ptr(base)) : "memory");
}
__device__ __forceinline__ void publish_f32x2(float *base, uint32_t off, float x, float y)
{
    const f2_t v = {x, y};
    uint64_t at;
    asm volatile("s_mov_b64 %0, %3\n\tglobal_store_dwordx2 %1, %2, %0 sc1"
                 : "=&s"(at) : "v"(off), "v"(v), "s"(uniform_ptr(base)) : "memory");
}
// Loads go through a buffer resource at the first of the partials: one instruction each, lane offset in a vector
// register, partial in a scalar one.  kAgent is the sc1 bit in the cache-policy operand.
constexpr int kAgent = 16;
constexpr uint32_t kRsrcFlags = 0x00027000;      // untyped 32-bit elements
__device__ __forceinline__ __amdgpu_buffer_rsrc_t parts_rsrc(float *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(base), 0, bytes, kRsrcFlags);
}

constexpr int kScaleHeads = 8;            // KV heads that may carry scales of their own (8-bit caches)

// What a kernel asks of its arguments at one time or another, 128 bytes: read whole, in one round trip (arrive_together).
struct CallArgs {
    const void *q, *k, *v;
    const fairkv_item *items;   // grouped by slot
    int32_t q_len, g_shift;     // new tokens per sequence; log2 of the query heads per KV head.  A kernel's
                                // template parameter G counts columns: q_len * (1 << g_shift), column
                                // c = new token (c >> g_shift), head (c & mask) of the group
    int32_t Hq, Hkv;
    int32_t B, out_dtype, n_parts, n_group_counters;
    int64_t n_rows;             // rows of k and of v
    float *part_o;              // [n_parts][G][D]   unnormalised outputs relative to the item's maximum
    float *part_ml;             // [n_parts][G][2]   (maximum in log2 units, sum of weights)
    int32_t *arrivals;          // [B*Hkv] items (or groups of items) of a cut pair that have delivered; 0 between calls.
                                // Behind them [n_group_counters] the same per group of kGroup items, index spread16(first part + group)
    void *out;
    float *lse;
    float scale_log2;           // scale * log2(e) (times the K scale of an 8-bit cache): scores are kept in log2
                                // units so exp is one v_exp_f32
    float v_scale;              // 1, or the V scale of an 8-bit cache: multiplies out
    unsigned long long *trace;  // fairkv_decode_attn_trace only: [workgroups][kTraceStamps], else null
};
static_assert(sizeof(CallArgs) == 128, "two cache lines");

// 8-bit caches with a scale per KV head: further factors on scale_log2 and v_scale, indexed h % kScaleHeads (all 1 otherwise; read by the
// 8-bit kernels only).
struct HeadFactors {
    float k[kScaleHeads], v[kScaleHeads];
};
struct DecodeArgs : CallArgs {
    HeadFactors factors;
    // What a workgroup needs before it has read anything from memory, riding in the kernel arguments.  Slot j has words
    // 3 j ...: the index of its first item (its last is the one before slot j + 1's first), the first K/V row of that
    // item, and in one word its query group (b * q_len * Hkv + h, bits 9..31) and min(tok_count, kEarlyTok) (bits
    // 0..8; 0 = no early start for this slot).
    uint32_t slot[3 * FAIRKV_MAX_SLOTS + 1];
};

// Phases a traced launch stamps with the 100 MHz wall clock, per workgroup (thread 0 of wave 0).  A stamp
// keeps its latest value: the hand-over stamps are those of the workgroup's last hand-over.
enum {
    kTraceStart = 0,         // first instruction
    kTraceTable,             // item list landed and checked
    kTraceFirstTile,         // first K/V tile landed
    kTraceItem0Streamed,     // wave 0 has consumed its tiles of the first item
    kTraceItem0Done,         // first item folded and written (or kept pending)
    kTraceLastStreamed,      // wave 0 has consumed its tiles of the last item
    kTraceFlushBegin,        // hand-over: all waves are there
    kTraceFlushPublished,    // partials' stores issued
    kTraceFlushCounted,      // count-in returned, roles known
    kTraceFlushMerged,       // merges (if any) computed and written
    kTraceFlushEnd,
    kTraceEnd,               // last instruction
    kTraceMergeLoaded,       // the first batch of partials of the merges has landed (this stamp makes the merge wait for it)
    kTraceStamps = 16
};
__device__ __forceinline__ void trace_stamp(const CallArgs &a, int what, bool who)
{
    if (a.trace && who) a.trace[static_cast<size_t>(blockIdx.x) * kTraceStamps + what] = wall_clock64();
}
constexpr int kEarlyTok = 384;            // tokens of a slot's first item that the early start may request
static_assert(sizeof(DecodeArgs) <= 4096, "kernel arguments are limited to 4 KiB");

// The query rows of pair (b, h) start at row qg << g_shift of q, and its outputs at the same row of out and lse, where
// qg = b * q_len * Hkv + h is its query group; column c of the pair is this many rows further.
__device__ __forceinline__ uint32_t col_row(int g_shift, int Hq, int c)
{
    return static_cast<uint32_t>((c >> g_shift) * Hq + (c & ((1 << g_shift) - 1)));
}
__device__ __forceinline__ size_t group_row(const CallArgs &a, int qg) { return static_cast<size_t>(qg) << a.g_shift; }

// out = o / l (times the output's factor) and lse for coordinates d .. d + 3 of column c of a pair, from its
// unnormalised output, maximum and weight sum.
template <int D>
__device__ __forceinline__ void write_out4(const CallArgs &a, int qg, int c, int d, float4 o, float m, float l, float v_mul)
{
    const size_t row = group_row(a, qg);
    const uint32_t col = col_row(a.g_shift, a.Hq, c);
    // 1 / l: the hardware's estimate and a Newton step, 4 instructions for the 10 of a division, as good to half a unit in the last place
    float inv = __builtin_amdgcn_rcpf(l);
    inv = l > 0.f ? fmaf(fmaf(-l, inv, 1.f), inv, inv) * v_mul : 0.f;
    store_out4(a.out, a.out_dtype, row * D, col * D + d, make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv));
    if (d == 0 && a.lse) a.lse[row + col] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
}

// A slot's words of the kernel arguments.
struct SlotStart {
    int i_begin, i_end;     // its items
    uint32_t row, np;       // of the first item: first row; query group and capped length
};
__device__ __forceinline__ SlotStart slot_start(const DecodeArgs &a)
{
    const uint32_t *w = a.slot + 3 * blockIdx.x;
    return SlotStart{static_cast<int>(w[0]), static_cast<int>(w[3]), w[1], w[2]};
}
// The arguments, asked for in one round trip: left to itself the compiler asks for each where it is first used, and with one
// wave per SIMD every such trip of 500-600 cycles is waited out.  The asm makes it need all of them here.
__device__ __forceinline__ void arrive_together(const CallArgs &a, const SlotStart &s)
{
    asm volatile("" ::"s"(s.i_begin), "s"(s.i_end), "s"(s.row), "s"(s.np), "s"(a.q), "s"(a.k), "s"(a.v), "s"(a.items), "s"(a.q_len),
                 "s"(a.g_shift), "s"(a.Hq), "s"(a.Hkv), "s"(a.B), "s"(a.out_dtype), "s"(a.n_parts), "s"(a.n_group_counters), "s"(a.n_rows),
                 "s"(a.part_o), "s"(a.part_ml), "s"(a.arrivals), "s"(a.out), "s"(a.lse), "s"(a.scale_log2), "s"(a.v_scale));
}
// A pointer put together from words: it points to global memory.  (The compiler knows that of a kernel argument; without it,
// stores become flat ones, which it follows by waits for everything that is outstanding: 0.5 to 1.3 % of a launch.)
template <class T>
__device__ __forceinline__ void to_global(T *&p)
{
    p = (T *)(__attribute__((address_space(1))) T *)reinterpret_cast<uintptr_t>(p);
}
// ... and kept in the lanes of one vector register (word i in lane i), so that neither another trip nor some twenty scalar
// registers are spent on what is needed once per item or once per launch: reading a word back is one instruction.
struct ArgLanes {
    uint32_t lanes;
    static constexpr int kWords = sizeof(CallArgs) / 4, kFirst = 6, kLast = 29;      // q, k and v stay in scalar registers; trace is read where it is used
    __device__ __forceinline__ explicit ArgLanes(const CallArgs &a) : lanes(0)
    {
        uint32_t w[kWords];
        __builtin_memcpy(w, &a, sizeof a);
        // The wait states in front: a vector instruction may have written a word (a spilled one comes back with a v_readlane).  Behind: a
        // v_readlane of the result may be next.
#pragma unroll
        for (int i = kFirst; i <= kLast; i += 4)
            asm("s_nop 1\n\tv_writelane_b32 %0, %1, %5\n\tv_writelane_b32 %0, %2, %5+1\n\tv_writelane_b32 %0, %3, %5+2\n\tv_writelane_b32 %0, %4, %5+3\n\ts_nop 0"
                : "+v"(lanes) : "s"(w[i]), "s"(w[i + 1]), "s"(w[i + 2]), "s"(w[i + 3]), "n"(i));
    }
    __device__ __forceinline__ CallArgs get() const
    {
        uint32_t w[kWords] = {};
#pragma unroll
        for (int i = kFirst; i <= kLast; ++i) w[i] = __builtin_amdgcn_readlane(lanes, i);
        CallArgs a;
        __builtin_memcpy(&a, w, sizeof a);
        to_global(a.items), to_global(a.part_o), to_global(a.part_ml), to_global(a.arrivals), to_global(a.out), to_global(a.lse);
        return a;
    }
};
static_assert((ArgLanes::kLast + 1 - ArgLanes::kFirst) % 4 == 0, "four at a time");
static_assert(offsetof(CallArgs, items) == 4 * ArgLanes::kFirst && offsetof(CallArgs, v_scale) == 4 * ArgLanes::kLast, "what the lanes hold");

// The factors of the KV heads of an 8-bit cache, those of K in lanes 0 .. kScaleHeads - 1, those of V in the next lanes.
__device__ __forceinline__ float lane_values(const float (&k)[kScaleHeads], const float (&v)[kScaleHeads])
{
    static_assert(kScaleHeads == 8, "sixteen lanes");
    float lanes = 0.f;
#pragma unroll
    for (int i = 0; i < 2 * kScaleHeads; i += 4) {
        const float *w = i < kScaleHeads ? k + i : v + (i - kScaleHeads);
        asm("s_nop 1\n\tv_writelane_b32 %0, %1, %5\n\tv_writelane_b32 %0, %2, %5+1\n\tv_writelane_b32 %0, %3, %5+2\n\tv_writelane_b32 %0, %4, %5+3\n\ts_nop 0"
            : "+v"(lanes) : "s"(w[0]), "s"(w[1]), "s"(w[2]), "s"(w[3]), "n"(i));
    }
    return lanes;
}
__device__ __forceinline__ float lane_value(float lanes, int i)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lanes), i));
}

// Layout facts of the vector-ALU kernel.  A bf16 row of K or V is LPR 16-byte pieces; one wave-wide
// 16-byte-per-lane access covers RPI whole rows, so every global access is a run of
// contiguous, fully used cache lines.
template <int D>
struct Geo {
    static constexpr int ES = 2;
    static constexpr int ROW_BYTES = D * ES;
    static constexpr int LPR = ROW_BYTES / 16;   // lanes (16-byte pieces) per row
    static constexpr int RPI = 64 / LPR;         // rows per wave-wide access
    static constexpr int NI = kTile / RPI;       // wave-wide accesses per 64-token tile
    static constexpr int EPC = 16 / ES;          // elements per 16-byte piece
    static constexpr int DW = ROW_BYTES / 4;     // dwords per row
};


// A cut piece that a workgroup has finished: its partial is stored (see item_epilogue) but not yet counted in.  The
// hand-over, which costs several memory round trips, happens once per workgroup, when the slot's list is done or kPend
// pieces are waiting, and not in the middle of the stream.  Every field is the same for all threads.
// Two: a line cut leaves a slot at most two pieces of cut pairs (its first and its last item).
constexpr int kPend = 2;
struct Piece {
    int32_t pair, qg, part, chunk, n_chunks;
    float v_mul;      // what multiplies the pair's output (1, or the V scale of an 8-bit cache)
};

// s_waitcnt vmcnt(0), once as an instruction the compiler accounts for (simm16 of gfx9: vmcnt 0,
// expcnt 7 and lgkmcnt 15 = no wait) and once as a fence for its own reordering of memory operations.
__device__ __forceinline__ void drain_vmem()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Hand over the pending pieces.  Called by all threads of the workgroup.
//
// A pair cut into fewer than kDeepFrom pieces: the partials are stored, wait until the stores are
// acknowledged, count in on the pair's counter; the workgroup that finds itself last merges the
// pair's partials (all of them were stored before their workgroups counted in):
//   m* = max_c m_c,  l* = sum_c l_c 2^(m_c - m*),  out = sum_c o_c 2^(m_c - m*) / l*
// (exact in real arithmetic, so a cut pair gives what the whole pair would) and sets the counter
// back to zero.
//
// A pair cut into more pieces would make one workgroup fetch all of them, batch after batch, at the rate of a single
// compute unit.  Its pieces form groups of kGroup consecutive ones, each group with a counter of its own: the last piece of
// a group to arrive merges the group into one partial (m*, l*, sum_c o_c 2^(m_c - m*), not divided), stores it in the slot
// of the group's first piece, waits for the acknowledgement and only then counts in on the pair's counter, on which the
// last GROUP to arrive merges the group partials.  Two short merges by different workgroups instead of one long one.
// Measured (us per layer, one sequence of 8 pairs / 8 pairs of 4096 tokens / batch 4 / Fair-Copying share / Llama-70B
// shape): from 64 pieces on 10.8 / 13.6 / 11.7 / - / 16.4, from 32 9.9 / 12.0 / 11.0 / 32.8 / 16.4, from 16 9.4 / 10.5 /
// 10.2 / 32.8 / 16.4, from 12 9.4 / 10.4 / 10.1 / 33.3 / 16.4, from 9 9.6 / 10.4 / 10.2 / 33.4 / 16.9 (more plans then
// need the instantiation with this code).  Groups of 4 or 6 instead of 8: one pair of 8192 tokens 11.0 -> 11.9, 11.3.
constexpr int kGroup = 8;
constexpr int kDeepFrom = 16;
enum { kRoleNone = 0, kRoleFinal = 1, kRoleGroup = 2 };

// Where counter i of n lies: neighbours n / 16 counters apart, each on a cache line of its own, for the count-ins of one line
// wait for one another (a permutation of 0 .. n - 1).  One pair in 128 pieces 10.8 -> 9.9 us, one sequence of eight pairs 8.66 -> 8.58; the
// counters of whole pairs, of which one sees two or three count-ins, gain nothing from it.
__device__ __forceinline__ int spread16(int i, int n)
{
    const int apart = n >> 4;
    return i < 16 * apart ? (i & 15) * apart + (i >> 4) : i;
}

constexpr int kMergeBatch = 8;   // partials of a cut pair fetched at once by the merging workgroup

// A partial goes to the workspace: four consecutive coordinates (the idx-th four of [G][D]) and, with the first of a
// column, its maximum and weight sum.  Nothing waits for the stores here.
template <int D, int G>
__device__ __forceinline__ void publish_part(const CallArgs &a, int part, int idx, float4 o, float m, float l)
{
    publish_f32x4(a.part_o + static_cast<size_t>(part) * (G * D), idx * 16, o);
    if (idx % (D / 4) == 0) publish_f32x2(a.part_ml + static_cast<size_t>(part) * (G * 2), idx / (D / 4) * 8, m, l);
}

// Partials first, first + step, ... (count of them; 0: nothing to do) of a pair into one: the pair's output or, if
// to_group, the partial of a group of pieces.  The same for all threads.
struct Merge {
    Piece pc;
    int first, step, count;
    bool to_group;
};
// The merges of a workgroup: a thread owns four consecutive coordinates of one column (of two columns, when there are 16
// of them).  What bounds it: memory round trips, and the instructions of a wave that is alone on its SIMD (4 cycles each).
// So the first batch of partials is requested for two things at once before any is used, the two merges or, with two
// columns per thread, the columns of a merge; what is the same for the wave stays in scalar registers, and a partial that
// is not there costs one branch.  The last workgroup of a launch is usually the last of both its pairs: one merge after the
// other cost it a round trip more (Llama-70B shape 0.1 us per launch, one sequence 0.2, 8-bit cache 0.2).
template <int D, int G, bool DEEP, bool TRACE = false>
__device__ __forceinline__ void merge_parts(const CallArgs &a, const Merge (&mg)[kPend])
{
    constexpr int D4 = D / 4, NC4 = G * D4, OB = G * D * 4, MB = G * 2 * 4;      // bytes of a partial's outputs, of its statistics
    constexpr int IT = (NC4 + kThreads - 1) / kThreads;                           // fours of coordinates per thread
    static_assert(IT <= 2 && kPend == 2, "two things at once");
    f4_t o[2][kMergeBatch];
    f2_t ml[2][kMergeBatch];
    auto fetch = [&](int u, int it, const Merge &m, int c0) __attribute__((always_inline)) {
        const int idx = threadIdx.x + it * kThreads;      // past the last coordinate: loaded and not used
        const size_t part = static_cast<size_t>(m.first) + static_cast<size_t>(m.step) * c0;
        const uint32_t span = static_cast<uint32_t>(m.step * (min(kMergeBatch, m.count - c0) - 1) + 1);
        const __amdgpu_buffer_rsrc_t ro = parts_rsrc(a.part_o + part * (G * D), span * OB);
        const __amdgpu_buffer_rsrc_t rm = parts_rsrc(a.part_ml + part * (G * 2), span * MB);
#pragma unroll
        for (int j = 0; j < kMergeBatch; ++j) {
            if (c0 + j >= m.count) break;
            ml[u][j] = __builtin_bit_cast(f2_t, __builtin_amdgcn_raw_buffer_load_b64(rm, idx / D4 * 8, m.step * j * MB, kAgent));
            o[u][j] = __builtin_bit_cast(f4_t, __builtin_amdgcn_raw_buffer_load_b128(ro, idx * 16, m.step * j * OB, kAgent));
        }
    };
#pragma unroll
    for (int turn = 0; turn < IT; ++turn) {       // IT == 1: both merges at once; else merge `turn`, both columns at once
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const Merge &m = mg[IT == 1 ? u : turn];
            if (m.count > 0) fetch(u, IT == 1 ? 0 : u, m, 0);
        }
        if constexpr (TRACE)
            if (turn == 0) {
                drain_vmem();
                trace_stamp(a, kTraceMergeLoaded, threadIdx.x == 0);
            }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const Merge &m = mg[IT == 1 ? u : turn];
            const int it = IT == 1 ? 0 : u, idx = threadIdx.x + it * kThreads;
            if (m.count == 0) continue;
            float m_star = -INFINITY, l_star = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
            for (int c0 = 0;;) {
                float m_new = m_star;
#pragma unroll
                for (int j = 0; j < kMergeBatch; ++j) {
                    if (c0 + j >= m.count) break;
                    m_new = fmaxf(m_new, ml[u][j][0]);
                }
                const float keep = m_star == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_star - m_new);
                l_star *= keep;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] *= keep;
#pragma unroll
                for (int j = 0; j < kMergeBatch; ++j) {
                    if (c0 + j >= m.count) break;
                    const float f = ml[u][j][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[u][j][0] - m_new);
                    l_star = fmaf(ml[u][j][1], f, l_star);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] = fmaf(o[u][j][e], f, acc[e]);
                }
                m_star = m_new;
                c0 += kMergeBatch;
                if (c0 >= m.count) break;
                fetch(u, it, m, c0);
            }
            if (idx >= NC4) continue;
            const float4 sum = make_float4(acc[0], acc[1], acc[2], acc[3]);
            if (DEEP && m.to_group)      // the group's partial, in the slot of its first piece
                publish_part<D, G>(a, m.first, idx, sum, m_star, l_star);
            else
                write_out4<D>(a, m.pc.qg, idx / D4, idx % D4 * 4, sum, m_star, l_star, m.pc.v_mul);
        }
    }
}

// DEEP: the plan has a pair in kDeepFrom pieces or more.  Without it the group code is not even compiled in.
template <int D, int G, bool DEEP, bool TRACE = false>
__device__ __forceinline__ void flush_pending(const CallArgs &a, const Piece (&pend)[kPend], int &n_pend, int32_t *roles /* LDS [kPend] */)
{
    if constexpr (TRACE) trace_stamp(a, kTraceFlushBegin, threadIdx.x == 0);
    drain_vmem();                                      // this thread's stores have reached the shared level ...
    __syncthreads();                                   // ... and every other thread's, before the workgroup counts itself in
    if constexpr (TRACE) trace_stamp(a, kTraceFlushPublished, threadIdx.x == 0);
    // Round 0: every pending piece counts in (a piece of a deeply cut pair on its group's counter) and
    // the last arrivals merge.  Round 1, only if this workgroup merged a group: that group counts in on
    // the pair's counter.  Whoever finds itself last sets the counter back for the next call on this workspace.
    int role[kPend] = {kRoleNone, kRoleNone};
    for (int round = 0; round < (DEEP ? 2 : 1); ++round) {
        if (threadIdx.x < static_cast<unsigned>(n_pend)) {
            const Piece &pc0 = pend[0], &pc1 = pend[1];
            const bool second = threadIdx.x != 0;
            const int pair = second ? pc1.pair : pc0.pair, nc = second ? pc1.n_chunks : pc0.n_chunks;
            int32_t *counter = a.arrivals + pair;
            int last = nc - 1, role_if_last = kRoleFinal;
            bool counts = round == 0;
            if constexpr (DEEP) {
                const int chunk = second ? pc1.chunk : pc0.chunk, first = (second ? pc1.part : pc0.part) - chunk;
                // two levels only if every group of the pair has a counter
                const bool deep = nc >= kDeepFrom && static_cast<int64_t>(first) + (nc - 1) / kGroup < a.n_group_counters;
                if (round == 0 && deep) {
                    counter = a.arrivals + static_cast<size_t>(a.B) * a.Hkv + spread16(first + chunk / kGroup, a.n_group_counters);
                    last = min(kGroup, nc - chunk / kGroup * kGroup) - 1;
                    role_if_last = kRoleGroup;
                } else if (round == 1) {
                    counts = (second ? role[1] : role[0]) == kRoleGroup;
                    last = (nc + kGroup - 1) / kGroup - 1;
                }
            }
            int mine = kRoleNone;
            if (counts && __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == last) {
                mine = role_if_last;
                __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            roles[threadIdx.x] = mine;
        }
        __syncthreads();
        if constexpr (TRACE) trace_stamp(a, kTraceFlushCounted, threadIdx.x == 0);
        bool any_group = false;
        role[0] = __builtin_amdgcn_readfirstlane(roles[0]);
        role[1] = n_pend > 1 ? __builtin_amdgcn_readfirstlane(roles[1]) : kRoleNone;
        Merge mg[kPend];
#pragma unroll
        for (int p = 0; p < kPend; ++p) {
            mg[p] = Merge{pend[p], pend[p].part - pend[p].chunk, 1, role[p] == kRoleNone ? 0 : pend[p].n_chunks, false};
            if constexpr (DEEP) {
                const int k = pend[p].chunk / kGroup, ng = (pend[p].n_chunks + kGroup - 1) / kGroup;
                if (role[p] == kRoleGroup) {
                    any_group = true;
                    mg[p].first += k * kGroup;
                    mg[p].count = min(kGroup, pend[p].n_chunks - k * kGroup);
                    if (mg[p].count == 1) mg[p].count = 0;     // its partial is the group's already
                    mg[p].to_group = true;
                } else if (round == 1 && role[p] != kRoleNone) {
                    mg[p].step = kGroup;
                    mg[p].count = ng;
                }
            }
        }
        if (mg[0].count + mg[1].count > 0) merge_parts<D, G, DEEP, TRACE>(a, mg);
        if constexpr (TRACE) trace_stamp(a, kTraceFlushMerged, threadIdx.x == 0);
        if (!DEEP || !any_group) break;                    // the same for all threads
        drain_vmem();                                      // the group partials are acknowledged ...
        __syncthreads();                                   // ... all of them, before the groups count in
    }
    n_pend = 0;
    drain_vmem();     // the compiler stops tracking the loads above: no guard waits on their registers later on
    if constexpr (TRACE) trace_stamp(a, kTraceFlushEnd, threadIdx.x == 0);
}

// The waves' results of an item in LDS: unnormalised outputs [kWaves][G][kStRow<D>], and per column the running
// maximum (log2 units) and the weight sum [kWaves][G][2].  A row is 16 bytes longer than its D floats: the lanes of a
// wave write the same coordinates of all its columns at once, which would all fall on the same banks.
template <int D>
constexpr int kStRow = D + 4;

// End of one item, called by all threads of the workgroup after every wave has put its result into st_o and st_ml.
// Folds the waves:
//   m* = max_w m_w,  l* = sum_w l_w 2^(m_w - m*),  o* = sum_w o_w 2^(m_w - m*).
// An item that is a whole pair writes out = o*/l* and lse.  An item of a cut pair stores its partial (m*, l*, o*) in
// the workspace, without waiting for it, and joins `pend`.  One barrier, before the fold: st_o and st_ml may be
// written again after the next barrier only.
template <int D, int G, bool DEEP, bool TRACE = false>
__device__ __forceinline__ void item_epilogue(const CallArgs &a, const Piece &pc, const float *st_o, const float *st_ml,
                                              Piece (&pend)[kPend], int &n_pend, int32_t *roles)
{
    const bool whole_pair = pc.n_chunks == 1;
    constexpr int D4 = D / 4;
    __syncthreads();
    // a thread owns four consecutive coordinates of one column (of two columns, with 16 of them at D = 128); all its LDS reads are issued
    // together, both columns' (one column after the other in a loop: two waits, and a condition per lane on the second)
    constexpr int NC4 = G * D4, IT = (NC4 + kThreads - 1) / kThreads;
    static_assert(NC4 <= kThreads || NC4 % kThreads == 0, "all threads or the first of them");
    if (NC4 >= kThreads || threadIdx.x < static_cast<unsigned>(NC4)) {
        float2 ml[IT][kWaves];
        float4 ow[IT][kWaves];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int idx = threadIdx.x + it * kThreads, g = idx / D4, d = (idx % D4) * 4;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                ml[it][w] = *reinterpret_cast<const float2 *>(st_ml + (w * G + g) * 2);
                ow[it][w] = *reinterpret_cast<const float4 *>(st_o + (w * G + g) * kStRow<D> + d);
            }
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int idx = threadIdx.x + it * kThreads, g = idx / D4, d = (idx % D4) * 4;
            float m_star = -INFINITY;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) m_star = fmaxf(m_star, ml[it][w].x);
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            float l_star = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const float f = ml[it][w].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[it][w].x - m_star);
                acc.x += ow[it][w].x * f;
                acc.y += ow[it][w].y * f;
                acc.z += ow[it][w].z * f;
                acc.w += ow[it][w].w * f;
                l_star += ml[it][w].y * f;
            }
            if (whole_pair) {
                write_out4<D>(a, pc.qg, g, d, acc, m_star, l_star, pc.v_mul);
            } else {
                publish_part<D, G>(a, pc.part, idx, acc, m_star, l_star);
            }
        }
    }
    if (!whole_pair) {
        if (n_pend == 0)
            pend[0] = pc;
        else
            pend[1] = pc;
        if (++n_pend == kPend) flush_pending<D, G, DEEP, TRACE>(a, pend, n_pend, roles);
    }
}

}  // namespace fairkv
