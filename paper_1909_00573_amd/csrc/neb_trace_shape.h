// Launch shapes of the traversal (neb_render.hip): a block is one wave, whose
// lanes each walk a ray.
#pragma once
#include <algorithm>
#include <cstdint>

namespace neb {

constexpr int kTraceBlock = 64;  // threads per traversal block (one wave)

// LDS of a block: the lanes' stacks, and what lanes that share rays exchange
// (per lane a nearest hit of 8 bytes, a count of 4, a donation of 8)
constexpr int kTraceShareBytes = kTraceBlock * (8 + 4 + 8);
constexpr int trace_lds_bytes(int stack) { return stack * kTraceBlock * 4 + kTraceShareBytes; }
constexpr int kLdsBytes = 160 * 1024;  // of a CU
// blocks that a CU's LDS holds: 17, 12 and 9 for stacks of 32, 48 and 64
// entries (what hipOccupancyMaxActiveBlocksPerMultiprocessor says, too)
constexpr int trace_blocks_resident(int stack) { return kLdsBytes / trace_lds_bytes(stack); }
// blocks per CU that a launch configuration may name (20, 13 and 10: what the
// stacks alone leave room for); launches have at most the resident ones
constexpr int trace_blocks_accepted(int stack) { return kLdsBytes / (stack * kTraceBlock * 4); }

// A queue of at most this many rays per wave of its launch is dealt out at once.
constexpr int kDealRays = 16;

// 32-bit byte offsets hold for node and triangle pools of at most 4 GB
inline bool trace_small_pools(int64_t node_bytes, int64_t tri_bytes) {
    return std::max(node_bytes, tri_bytes) <= (int64_t)UINT32_MAX;
}

// Whether closest-hit launches of a context deal short queues out: frames of
// at most 65 536 pixels, whose queues leave most of the chip without a wave.
// City of 120 x 120 lots at 160 x 120, two iterations: 7.2 -> 2.6 ms; of 12 x 12
// lots at 60 x 50 1.50 -> 0.66; 64 x 64 preview 1.29 -> 1.11.  The line is a cautious
// one, not where dealing stops to pay.  Per iteration, ms, undealt, dealt up
// to 16 rays a wave and up to 64: city of 250 x 250 lots at 240 x 200 1.73 (always
// dealt), 1.74, 1.55; at 300 x 250 2.9, 2.3, 1.9; room at 401 x 227 1.33, 1.35,
// 1.29; city at 640 x 500 4.7, 4.65, 4.35; room at 512 x 512 3.64, 3.63, 3.64;
// city of 288 x 288 lots at 1024 x 1024 5.82, 5.86, 5.85.
inline bool trace_deals(int64_t npix, int64_t node_bytes, int64_t tri_bytes) {
    return npix <= 65536 && trace_small_pools(node_bytes, tri_bytes);
}

// blocks of a launch over a queue of at most cap rays, on `cus` compute units
// with at most `most` blocks resident each: bpc blocks per CU (0: one block per
// 64 queue slots, -1: `most`), never more than the queue has lanes' worth of
// rays, or than leave a wave eight rays of it where the queue is dealt out
// (two: 60 x 50 city 0.82 instead of 0.66 ms)
inline int trace_blocks(int cus, int64_t cap, int bpc, int most, bool deals) {
    if (bpc < 0 || bpc > most) bpc = most;
    const int64_t least = bpc > 0 && deals ? 8 : kTraceBlock;
    const int64_t blocks = bpc > 0 ? (int64_t)cus * bpc : 1 << 20;
    return (int)std::max<int64_t>(1, std::min(blocks, (cap + least - 1) / least));
}

}  // namespace neb
