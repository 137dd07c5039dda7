// Decode kernel for fp32 K/V/q on the matrix cores.
//
// What bounds it: HBM.  With G = 8 query heads per KV head a retained token is 1 KB and 4096 flop; as 16x16x4 fp32
// MFMA tiles (the G heads padded to 16 columns) that is 8192 flop per KB streamed, i.e. a third of the
// fp32 matrix rate at 6 TB/s.  On the vector ALU the same token cost the softmax of its 64-token tile, one scalar
// load of q per multiply and the reduction over lanes, and a wave waited for each tile before it asked for the next.
//
// Measured against the vector-ALU kernel that served fp32 before: the Llama-70B shape
// (B 16, 64 / 8 heads, D 128, lognormal budgets, 135 MB; the planner's defaults) 537 -> 31.7 us per layer, 128 x 8 pairs of 1024 tokens (1.07 GB)
// 6.7 TB/s; 30.1 -> 28.9 us, one sequence 12.3 -> 11.6, since the kernel's arguments come in one trip and the items sit in
// registers.  Four waves (one per SIMD) against eight: 0.3-1.5 % faster at every size tried, 3 % at 1 GB.
//
// Everything stays in 32 bits: an fp32 MFMA multiplies and adds like a chain of fused multiply-adds.
//
// Shapes.  A wave works on tiles of 16 tokens, lane = (l16, lq) with l16 = lane % 16, lq = lane / 16:
//     S^T[token][head] = K[token][:] . q[head][:]    D/4 x mfma_16x16x4: A row = token l16, contraction index lq
//     O^T[d][head]    += V^T[d][token] P[token][head]  D/4 x mfma_16x16x4: A row stands for a d, contraction index lq
// The order of a contraction and the meaning of an output row are free, so they are chosen such that every operand is
// a 16-byte load straight from memory into the registers that the matrix instruction reads, with no trip through LDS:
//     step (c, j) of the scores contracts d = 16 c + 4 lq + j: lane loads K[token l16][16 c + 4 lq .. + 3] (and q alike);
//     step r of the sum contracts token 4 lq + r, which is the token whose score the lane holds in register r;
//     row i of output block (u, j) is d = 64 u + 4 i + j: lane loads V[token 4 lq + r][64 u + 4 l16 .. + 3].
//
// Pipelining.  The registers of K are requested again (the wave's next tile, of the next item when this one is done)
// as soon as the scores have been issued, those of V after the weighted sum, so a tile is in flight while the other
// half of the arithmetic runs.
#pragma once
#include "decode_mfma.h"

namespace fairkv {

template <int D, int G, bool DEEP>
__global__ __launch_bounds__(kThreads, 1) void fairkv_decode_f32_kernel(DecodeArgs args)
{
    static_assert(D == 64 || D == 128, "head_dim");
    static_assert(G >= 1 && G <= 8, "query heads of a group");
    constexpr int ROWB = D * 4;
    constexpr int NC = D / 16;      // 16-byte pieces of a K row (or q row) per lane
    constexpr int NU = D / 64;      // 16-byte pieces of a V row per lane

    __shared__ __attribute__((aligned(1024))) fairkv_item raw[kList];                   // items as fetched
    __shared__ __attribute__((aligned(16))) float st_o[2][kWaves * G * kStRow<D>];      // two sets, used in turn
    __shared__ __attribute__((aligned(16))) float st_ml[2][kWaves * G * 2];
    __shared__ int32_t roles[kPend];
    Piece pend[kPend] = {};
    int n_pend = 0, set = 0;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;

    const SlotStart slot = slot_start(args);
    arrive_together(args, slot);
    const char *const q_base = static_cast<const char *>(args.q), *const k_base = static_cast<const char *>(args.k),
               *const v_base = static_cast<const char *>(args.v);
    const int g_shift = args.g_shift;
    const int i_begin = slot.i_begin, i_end = slot.i_end;
    if (i_end <= i_begin) return;   // an idle slot

    // The kList items that start at `first`, 32 by each of the first two waves; past the end of the list its last item again.
    const uint32_t raw_lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FAIRKV_LDS_PTR(raw))) + wave * 1024;
    auto fetch_items = [&](const fairkv_item *items, int first) __attribute__((always_inline)) {
        const int last = min(kList, i_end - first) - 32 * wave - 1;
        if (last >= 0) load16_to_lds_keep(items + first + 32 * wave, min(lane >> 1, last) * 32 + (lane & 1) * 16, raw_lds);
    };
    fetch_items(args.items, i_begin);

    // tiles of an n-token item that fall to this wave: wave, wave + kWaves, ...
    auto tiles_of = [&](int n) __attribute__((always_inline)) {
        const int n_tiles = (n + kTok - 1) / kTok;
        return n_tiles > wave ? (n_tiles - wave + kWaves - 1) / kWaves : 0;
    };

    // The fetch cursor: the wave's next tile, f_t of f_tiles of item f_item (n tokens from row on).
    int f_item = 0, f_t = 0, f_tiles = 0, f_n = 0, f_qg = 0;
    int64_t f_row = 0;
    f32x4_t kr[NC], vr[4][NU], qr[NC];
    // One tile: 16 rows from `row` on, of which those up to `last` are the item's.  Rows past it re-read that row;
    // their scores are masked and their V is replaced by zeros.
    auto load_k = [&](int64_t row, int last) __attribute__((always_inline)) {
        const char *base = k_base + row * ROWB;
        const uint32_t off = min(l16, last) * ROWB + lq * 16;
#pragma unroll
        for (int c = 0; c < NC; ++c) kr[c] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(base + off + c * 64));
    };
    auto load_v = [&](int64_t row, int last) __attribute__((always_inline)) {
        const char *base = v_base + row * ROWB;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t off = min(4 * lq + r, last) * ROWB + l16 * 16;
#pragma unroll
            for (int u = 0; u < NU; ++u) vr[r][u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(base + off + u * 256));
        }
    };
    auto f_tok0 = [&]() __attribute__((always_inline)) { return (wave + f_t * kWaves) * kTok; };
    auto load_q = [&]() __attribute__((always_inline)) {      // columns past the group repeat its last head; they are never stored
        const char *base = q_base + (static_cast<size_t>(f_qg) << g_shift) * ROWB;
        const uint32_t off = min(l16, G - 1) * ROWB + lq * 16;
#pragma unroll
        for (int c = 0; c < NC; ++c) qr[c] = *reinterpret_cast<const f32x4_t *>(base + off + c * 64);
    };

    // The first tile of a list, V last: in the order of the loop below, so that its waits for K need not be waits for everything.
    auto load_first = [&]() __attribute__((always_inline)) {
        load_q();
        __builtin_amdgcn_sched_barrier(0);
        load_k(f_row + f_tok0(), f_n - 1 - f_tok0());
        __builtin_amdgcn_sched_barrier(0);
        load_v(f_row + f_tok0(), f_n - 1 - f_tok0());
        __builtin_amdgcn_sched_barrier(0);
    };

    // Early start: the first item's rows are requested from what the kernel arguments say of it, before the item list is here.
    const int n0 = static_cast<int>(slot.np & 0x1ffu);
    const bool seeded = n0 > 0;
    if (seeded) {
        f_qg = static_cast<int>(slot.np >> 9);
        f_row = slot.row;
        f_n = n0;
        f_tiles = tiles_of(n0);
        if (f_tiles > 0) {
            load_first();
        }
    }

    const ArgLanes arg_lanes(args);
    const float scale_log2 = args.scale_log2;
    const int qg_stride = args.q_len * args.Hkv;

    ItemList list{};
    for (int batch = i_begin; batch < i_end; batch += kList) {
        const int nb = min(kList, i_end - batch);
        const bool early = seeded && batch == i_begin;
        const bool loaded = early && f_tiles > 0;               // the first tile is on its way already
        if (batch != i_begin) {
            __syncthreads();                                    // nobody still reads the previous list
            fetch_items(arg_lanes.get().items, batch);
        }
        // the items were requested before the first tile and its queries: they have landed once only those are outstanding
        if (loaded)
            wait_vmcnt<2 * NC + 4 * NU>();
        else
            wait_vmcnt<0>();
        __syncthreads();
        list = item_list(arg_lanes.get(), raw, lane);
        if (early && lane == 0) list.n = n0 < kEarlyTok ? n0 : max(list.n, kEarlyTok);   // its first tile is on its way, as many as n0 said

        auto seek = [&](int item) __attribute__((always_inline)) {
            f_item = item;
            f_t = 0;
            f_tiles = 0;
            if (item < nb) {
                f_row = list.row(item);
                f_n = list.tokens(item);
                f_qg = list.query_group(qg_stride, item);
                f_tiles = tiles_of(f_n);
            }
        };
        auto skip_done = [&]() __attribute__((always_inline)) {   // on to the next item that has a tile for this wave
            while (f_t >= f_tiles && f_item < nb) seek(f_item + 1);
            return f_item < nb;
        };
        if (early) {
            f_item = 0;
            f_n = list.tokens(0);                               // its full length
            f_tiles = tiles_of(f_n);
        } else {
            seek(0);
        }
        if (!loaded && skip_done()) {
            load_first();
        }

        for (int ci = 0; ci < nb; ++ci) {
            const int n = list.tokens(ci);
            const int my_tiles = tiles_of(n);

            f32x4_t o[NU][4];
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) o[u][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            float m_run = -INFINITY, l_run = 0.f;   // reference maximum of the lane's head, this lane's share of the weights

            for (int t = 0; t < my_tiles; ++t) {
                // ---- scores: S^T[token 4 lq + r][head l16]; two chains of sums --------------------------
                f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[c][0], qr[c][0], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[c][1], qr[c][1], s1, 0, 0, 0);
                    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[c][2], qr[c][2], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[c][3], qr[c][3], s1, 0, 0, 0);
                }
                const int tok0 = (wave + t * kWaves) * kTok;
                const bool masked = n - tok0 < kTok;

                // ---- the K registers are free: the next tile's rows, and its query rows if it is another item's.
                // Without a next tile one row of this one is read again: with the same number of loads on every path
                // the compiler can wait for V below while the rows of K stay in flight.
                __builtin_amdgcn_sched_barrier(0);
                int64_t next = f_row + tok0;
                int next_last = 0;
                ++f_t;
                if (skip_done()) {
                    next = f_row + f_tok0();
                    next_last = f_n - 1 - f_tok0();
                    if (f_t == 0) load_q();
                }
                load_k(next, next_last);
                __builtin_amdgcn_sched_barrier(0);

                float sv[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) sv[r] = (s0[r] + s1[r]) * scale_log2;
                if (masked) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (4 * lq + r >= n - tok0) {
                            sv[r] = -INFINITY;
#pragma unroll
                            for (int u = 0; u < NU; ++u) vr[r][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                        }
                }

                // ---- raise the reference maximum to the largest score (at once, unlike the bf16 kernel: weights stay at
                //      or below 1, so the sums reach no further than the largest V; a tile is long enough to hide it)
                float mx = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
                if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) {
                    const float m_new = fmaxf(m_run, quarters_max(mx));
                    const float alpha = m_new == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first tile
                    l_run *= alpha;
#pragma unroll
                    for (int u = 0; u < NU; ++u)
#pragma unroll
                        for (int j = 0; j < 4; ++j) o[u][j] *= alpha;
                    m_run = m_new;
                }
                float p[4];
                const float m_ref = m_run == -INFINITY ? 0.f : m_run;     // nothing but -inf so far: weights 0, not exp2(nan)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p[r] = __builtin_amdgcn_exp2f(sv[r] - m_ref);
                    l_run += p[r];
                }

                // ---- O^T[64 u + 4 i + j][head] += V^T P -----------------------------------------------
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int u = 0; u < NU; ++u)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            o[u][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[r][u][j], p[r], o[u][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                load_v(next, next_last);
                __builtin_amdgcn_sched_barrier(0);
            }

            // ---- fold the four token quarters of l, stage this wave's result, finish the item ------
            l_run = quarters_sum(l_run);
            if (l16 < G) {
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r)      // rows 4 lq + r of the four blocks j: four consecutive coordinates
                        *reinterpret_cast<float4 *>(st_o[set] + (wave * G + l16) * kStRow<D> + 64 * u + 16 * lq + 4 * r) =
                            make_float4(o[u][0][r], o[u][1][r], o[u][2][r], o[u][3][r]);
                if (lq == 0) {
                    *reinterpret_cast<float2 *>(st_ml[set] + (wave * G + l16) * 2) = make_float2(m_run, l_run);
                }
            }
            if (list.valid(ci)) {
                const CallArgs a = arg_lanes.get();
                item_epilogue<D, G, DEEP>(a, list.piece(a, ci, a.v_scale), st_o[set], st_ml[set], pend, n_pend, roles);
                set ^= 1;
            }
        }
    }
    if (n_pend > 0) flush_pending<D, G, DEEP>(arg_lanes.get(), pend, n_pend, roles);
}

}  // namespace fairkv
