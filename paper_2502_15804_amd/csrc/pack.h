// Building and growing the packed ragged cache on the GPU: gather of the kept rows of a dense
// K/V cache (what a per-head compressor leaves behind, Section 2) and the append of a decode
// step's new row per pair.  Pure data movement: rows travel as 16-byte pieces, a wave-wide
// access covers whole rows, so every read and write is a run of fully used cache lines.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "fairkv.h"
#include "rows.h"

namespace fairkv {

struct PackArgs {
    const char *k_dense, *v_dense;    // [B][Hkv][T][row bytes]
    char *k_out, *v_out;              // [n_rows][row bytes]
    const int64_t *keep_ptr;          // [B*Hkv+1]
    const int32_t *keep_t;            // [keep_ptr[B*Hkv]]
    const int64_t *off;               // [B*Hkv]
    const fairkv_item *items;         // work list: (row, tok_count, b, h) name runs of packed rows
    const int32_t *slot_ptr;          // [gridDim.x + 1]
    int32_t *bad;                     // rows and items skipped because they point outside; may be null
    int64_t n_rows;
    int32_t B, Hkv, T;
    int32_t parts;                    // workgroups per slot, which is gridDim.y (read from there it costs the host 0.2 us a launch)
};

// `parts` workgroups per slot of the work list (pack_parts); of an item, which is a run of rows of one pair, workgroup
// y moves passes y, y + parts, ... of kRowsPerPass rows.
// What bounds it: the memory's rate for reads and writes mixed (a plain copy reaches 4.8 TB/s).  One workgroup per slot,
// i.e. one per compute unit, has 8 KB of rows on the way and waits for each pass: 39.9 us for the 136 MB of a layer of
// the Llama-70B shape, 3.4 TB/s.  Two, four, eight: 29.5, 28.3 (4.8 TB/s), 29.8 us; more passes in flight per workgroup
// instead: 28.5 us for two workgroups with four, slower on small caches (5.5 -> 6.3 us for one sequence).
constexpr int kPackParts = 4;

// Workgroups per slot.  A workgroup costs the fetches in front of its first pass (slot, item, pair, index), so a slot gets
// no more of them than it has passes on the average, up to kPackParts; n_rows is what the host knows of the passes.  Up to
// FAIRKV_MAX_SLOTS slots always get kPackParts: with about one workgroup per compute unit the chip is idle otherwise.
// us for one, two and four workgroups per slot, L the Llama-70B shape, S 128 pairs of 100 tokens with D = 64:
//   256 slots          L 40.6 30.1 29.3   S 6.9 6.2 6.2
//   3072 (L: 2.7 passes a slot, S: 0.1)   L 28.9 28.4 31.0   S 6.3 6.5 6.8
//   4096 slots of 64 tokens (L: 2)        L 31.4 29.5 30.3   S 6.7 6.9 7.5
//   2048 slots of 64 tokens (L: 4)        L 30.3 28.8 29.3   S 6.2 6.2 6.5
// Over 32 to 4096 slots of six caches, planned with the defaults and in pieces of at least 64 tokens, no plan takes more
// than 2.5 % longer than with one workgroup per slot; four everywhere took up to 13 % longer.
__host__ __device__ constexpr int pack_parts(int64_t n_rows, int n_slots, int row_bytes)
{
    const int64_t passes = n_rows / (4096 / row_bytes) / n_slots;      // of 4 KB of K and of V, per slot
    return n_slots <= FAIRKV_MAX_SLOTS || passes >= kPackParts ? kPackParts : passes >= 1 || n_slots <= 2048 ? 2 : 1;
}
static_assert(kPackParts == 4, "pack_parts gives 4, 2 or 1");

template <int ROWB>
__global__ __launch_bounds__(256) void fairkv_pack_kernel(PackArgs a)
{
    typedef __attribute__((ext_vector_type(4))) uint32_t u4;   // rows are read once and written once: non-temporal both ways
    constexpr int PPR = ROWB / 16;            // 16-byte pieces per row
    constexpr int kRowsPerPass = 256 / PPR;
    const int first_row = blockIdx.y * kRowsPerPass, step = a.parts * kRowsPerPass;
    const int piece = threadIdx.x % PPR, sub = threadIdx.x / PPR;
    for (int i = a.slot_ptr[blockIdx.x]; i < a.slot_ptr[blockIdx.x + 1]; ++i) {
        const fairkv_item it = a.items[i];
        const int n = it.tok_count;
        if (n <= 0) continue;
        bool ok = it.b >= 0 && it.b < a.B && it.h >= 0 && it.h < a.Hkv && rows_within(it.row, n, a.n_rows);
        int64_t pair = 0, begin = 0, first = 0;
        if (ok) {
            pair = static_cast<int64_t>(it.b) * a.Hkv + it.h;
            // All three are requested before one is looked at: 128 pairs of 100 tokens, D = 64, 5.92 -> 5.62 us, one sequence 3.80 -> 3.62.
            const int64_t at = a.off[pair], end = a.keep_ptr[pair + 1];
            first = a.keep_ptr[pair];
            begin = it.row - at;
            ok = (begin >= 0) & (first >= 0) & (begin <= end - first - n);
        }
        if (!ok) {
            if (threadIdx.x == 0 && blockIdx.y == 0 && a.bad) atomicAdd(a.bad, 1);
            continue;
        }
        const int32_t *kt = a.keep_t + first + begin;
        const char *ksrc = a.k_dense + pair * a.T * ROWB + piece * 16;
        const char *vsrc = a.v_dense + pair * a.T * ROWB + piece * 16;
        char *kdst = a.k_out + it.row * ROWB + piece * 16;
        char *vdst = a.v_out + it.row * ROWB + piece * 16;
        // The index of the next pass is requested before the row of this one, so a pass costs one memory latency (the
        // row), not two (index, then row).  Rows past the end and rows with a bad index are loaded from a clamped
        // (valid) address and not stored.
        int32_t t_next = kt[min(first_row + sub, n - 1)];
        for (int r0 = first_row; r0 < n; r0 += step) {
            const int32_t t = t_next;
            t_next = kt[min(r0 + step + sub, n - 1)];
            const int64_t tc = min(max(t, 0), a.T - 1);
            const u4 kk = __builtin_nontemporal_load(reinterpret_cast<const u4 *>(ksrc + tc * ROWB));
            const u4 vv = __builtin_nontemporal_load(reinterpret_cast<const u4 *>(vsrc + tc * ROWB));
            const int r = r0 + sub;
            if (r >= n) continue;
            if (t < 0 || t >= a.T) {
                if (piece == 0 && a.bad) atomicAdd(a.bad, 1);
                continue;
            }
            __builtin_nontemporal_store(kk, reinterpret_cast<u4 *>(kdst + static_cast<int64_t>(r) * ROWB));
            __builtin_nontemporal_store(vv, reinterpret_cast<u4 *>(vdst + static_cast<int64_t>(r) * ROWB));
        }
    }
}

struct AppendArgs {
    const char *k_new, *v_new;   // [B*Hkv][row bytes]
    char *k, *v;                 // packed
    const int64_t *off;
    int32_t *len;                // in/out
    const int32_t *cap;
    int32_t *full;               // pairs found at capacity; may be null
    int64_t n_rows;
    int32_t n_pairs;
};

// A pair is served by PPR consecutive lanes of one wave (PPR divides 64): all of them read the
// pair's length with the same instruction, before the lane of piece 0 stores the new length.
// What bounds it: round trips to memory.  The kernel's arguments come in one (left to itself the compiler asks for them in four
// groups), the new rows and what says where they go in another, and the checks have no branch: 13 sequences of 8 KV heads,
// D = 64, bf16, 2.66 -> 2.00 us (2.30 with the rows asked for behind the checks).
template <int ROWB>
__global__ __launch_bounds__(256) void fairkv_append_kernel(AppendArgs a)
{
    constexpr int PPR = ROWB / 16;
    asm volatile("" ::"s"(a.k_new), "s"(a.v_new), "s"(a.k), "s"(a.v), "s"(a.off), "s"(a.len), "s"(a.cap), "s"(a.n_rows), "s"(a.n_pairs));
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t pair = idx / PPR;
    const int piece = static_cast<int>(idx % PPR);
    if (pair >= a.n_pairs) return;
    typedef __attribute__((ext_vector_type(4))) uint32_t u4;
    u4 kk = *reinterpret_cast<const u4 *>(a.k_new + pair * ROWB + piece * 16), vv = *reinterpret_cast<const u4 *>(a.v_new + pair * ROWB + piece * 16);
    const int32_t l = a.len[pair], cap = a.cap[pair];
    const int64_t off = a.off[pair];
    const uint64_t row = static_cast<uint64_t>(off) + static_cast<uint32_t>(l);      // of numbers that are not negative: does not wrap around
    __builtin_amdgcn_sched_barrier(0);          // all five on their way before one is looked at
    asm volatile("" : "+v"(kk), "+v"(vv));      // needed here: the compiler would ask for them behind the branch
    if ((l < 0) | (l >= cap) | (off < 0) | (row >= static_cast<uint64_t>(a.n_rows))) {
        if (piece == 0 && a.full) atomicAdd(a.full, 1);
        return;
    }
    *reinterpret_cast<u4 *>(a.k + row * ROWB + piece * 16) = kk;
    *reinterpret_cast<u4 *>(a.v + row * ROWB + piece * 16) = vv;
    if (piece == 0) a.len[pair] = l + 1;
}

}  // namespace fairkv
