// The check of a plan's items that every decode call makes before it launches.  Host code alone, so that it can be built and tested
// without a GPU's compiler.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "fairkv.h"
#include "rows.h"

namespace fairkv {

// The host's copy of a plan's items and the call that they are for; none of the numbers is negative.
struct PlanItems {
    const fairkv_item *items;
    int32_t n_items, n_parts, B, Hkv, q_len;
    int64_t n_rows;
};

// What the items of a plan are found to be.
struct PlanCheck {
    bool ok;
    int32_t deepest = 0;             // pieces of the pair that is cut into the most
    int32_t shortest = INT32_MAX;    // tokens of the shortest whole pair
    int32_t looks = 0;               // at items, for what the check costs
};

// Every cut pair must come with all its pieces, each exactly once: a piece that is missing would leave the
// pair's arrival counter short for ever (no output, and a counter that is not zero for the next call); one
// that comes twice would have two workgroups write one partial slot.
// count_scratch: n_parts numbers, for callers that must not allocate; else null.
inline PlanCheck check_plan(const PlanItems &c, int32_t *count_scratch)
{
    const int32_t B = c.B, Hkv = c.Hkv, q_len = c.q_len, n_items = c.n_items, n_parts = c.n_parts;
    PlanCheck r{true};
    // A plan that lists its pieces in the order of their partial slots, as a line cut does, needs no counting: item i has slot i, and each
    // piece follows its predecessor.  No branch and no store per item.  us per call with counting
    // and without: 16 items 0.51 and 0.23, 256 1.55 and 0.87, 1073 7.5 and 3.6, 2048 13.5 and 6.7.
    // Behind each kBlock items, the pass ends if one of them broke the order (or is to be refused); the pairs that were whole
    // before that block, the first `whole` items and slots, are done.  us for all checks of a call, with every item counted, with the
    // pass always run to its end, and now: a plan of LPT_SPLIT, 743 items, 10.6, 11.9 and 9.4, 1104 items 13.3, 16.1 and 11.1; LPT and NAIVE,
    // 1024 pairs, 12.3, 14.1 and 10.6; in order, 1114 items, 13.3, 9.3 and 9.3.  With blocks of 128 LPT_SPLIT takes 9.8 and 11.6, of 256 10.2 and 11.7.
    constexpr int32_t kBlock = 64;
    auto u = [](int32_t v) { return static_cast<uint32_t>(v); };      // differences may wrap; those of two numbers that are not negative do not
    int32_t whole = 0;
    int32_t follows = 0, n_chunks = 0;      // `follows`: chunk that the next item has to be
    for (int32_t begin = 0, end; begin < n_items; begin = end) {
        end = begin + std::min(kBlock, n_items - begin);
        uint32_t bad = 0;                 // any bit: not in order, or refused
        int32_t sign = 0;                 // negative: refused
        int64_t rows = 0;                 // the same
        for (int32_t i = begin; i < end; ++i) {
            const fairkv_item it = c.items[i];
            const int32_t next = static_cast<int32_t>(u(it.chunk) + 1u);
            bad |= static_cast<uint32_t>((it.part ^ i) | (it.chunk ^ follows) | (follows == 0 ? 0 : it.n_chunks ^ n_chunks));
            sign |= it.b | static_cast<int32_t>(u(B) - 1u - u(it.b)) | it.h | static_cast<int32_t>(u(Hkv) - 1u - u(it.h)) | it.tok_count;
            const uint64_t last_row = static_cast<uint64_t>(c.n_rows) - u(it.tok_count);      // that the item may begin at: negative if it is too long
            rows |= it.row | static_cast<int64_t>(last_row) | static_cast<int64_t>(last_row - static_cast<uint64_t>(it.row));
            r.deepest = std::max(r.deepest, it.n_chunks);
            r.shortest = std::min(r.shortest, it.n_chunks == 1 ? it.tok_count : INT32_MAX);
            follows = next == it.n_chunks ? 0 : next;
            n_chunks = it.n_chunks;
        }
        if (q_len > 1)      // see below
            for (int32_t i = begin; i < end; ++i) {
                const fairkv_item &it = c.items[i];
                bad |= static_cast<uint32_t>((it.n_chunks > 1) & (u(it.chunk) + 1u == u(it.n_chunks)) & (it.tok_count < q_len - 1));
            }
        r.looks += end - begin;
        if (bad != 0 || sign < 0 || rows < 0) break;
        whole = end - follows;      // less the pieces of a pair that goes on
    }
    if (whole == n_items) return r;
    // Any order: count[first slot of a pair] counts that pair's pieces; a piece's own slot must be used once.  Slots from `whole` on: a pair
    // that reaches into those before would use one of them again.
    r.ok = false;
    r.looks += n_items - whole;
    const int32_t n_slots = n_parts - whole;
    std::vector<int32_t> count_own;
    int32_t *count = count_scratch;
    if (!count) {
        count_own.assign(static_cast<size_t>(n_slots), 0);
        count = count_own.data();
    } else {
        for (int32_t i = 0; i < n_slots; ++i) count[i] = 0;
    }
    for (int32_t i = whole; i < n_items; ++i) {
        const fairkv_item &it = c.items[i];
        r.deepest = std::max(r.deepest, it.n_chunks);
        if (it.n_chunks == 1) r.shortest = std::min(r.shortest, it.tok_count);
        if (it.b < 0 || it.b >= B || it.h < 0 || it.h >= Hkv || it.tok_count < 0) return r;
        if (!rows_within(it.row, it.tok_count, c.n_rows)) return r;      // the kernel reads exactly these rows of K and V
        if (it.n_chunks < 1 || it.chunk < 0 || it.chunk >= it.n_chunks) return r;
        const int64_t first = static_cast<int64_t>(it.part) - it.chunk - whole, own = first + it.chunk;      // up to 2^31 - 1 each
        if (first < 0 || first + it.n_chunks > n_slots) return r;
        // the rows new tokens hide from one another (the last q_len - 1 of a pair) must not reach
        // back beyond the pair's last chunk: the kernel masks inside that chunk only
        if (q_len > 1 && it.n_chunks > 1 && it.chunk == it.n_chunks - 1 && it.tok_count < q_len - 1) return r;
        count[first] += 1 << 8;                 // pieces of the pair that starts at this slot
        count[own] += 1;                        // uses of this slot
        if ((count[own] & 0xff) > 1 || (count[first] >> 8) > it.n_chunks) return r;
    }
    for (int32_t i = whole; i < n_items; ++i) {
        const fairkv_item &it = c.items[i];
        if ((count[it.part - it.chunk - whole] >> 8) != it.n_chunks) return r;
    }
    r.ok = true;
    return r;
}

}  // namespace fairkv
