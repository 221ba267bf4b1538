// Layers over a rank-space bitmap (rankbits.hip): host-side declarations.
#pragma once

#include "internal.h"

namespace cg {

constexpr int kRbMaxN = 12;              // 32-bit ranks
constexpr uint32_t kRbLgDigits = 9;      // segments of the bitmap in a large step: 512
constexpr int kRbLargeMinN = 10;         // large steps from n = 10
constexpr uint32_t kRbWindow = 64;       // layers whose counters are on the device at once
constexpr uint32_t kRbStride = 16;       // words between two counters: a line each
constexpr uint32_t kRbChain = 16;        // layers launched between two read-backs at most
// error bits of RbArgs::flags
constexpr uint32_t kRbFlagRoom = 1;      // more states than the layer array holds
constexpr uint32_t kRbFlagPart = 2;      // a part of the partition overran

// The states of all layers lie one layer after another in `all`; layer d is
// all[off(d) .. off(d) + cnt(d)). Counters of layer d are at word
// (d % kRbWindow) * kRbStride of cnt and off.
struct RbArgs {
    uint64_t *all;
    uint64_t cap;            // states that fit `all`
    uint32_t *seen;          // visited: one bit per state (rb_bitmap_words(n) words)
    const GenSel *sel;
    uint32_t k;
    uint64_t max_frontier;   // 0 = none
    uint64_t *cnt, *off;
    uint32_t *flags;
};

// Starts the counters at layer d (off, F known to the host) and marks the
// states all[0 .. off + F) as visited.
void launch_rb_begin(int n, const RbArgs &a, uint32_t d, uint64_t off, uint64_t F, hipStream_t s);
// Layer d + 1 from layer d: every neighbour is tested against `seen`.
// `most`: states layer d may hold (sizes the launch only).
void launch_rb_step(int n, const RbArgs &a, uint32_t d, uint64_t most, PipeWork &w);

// Words of the bitmap: 2^ceil(log2 n!) bits.
uint64_t rb_bitmap_words(int n);

// A large step: layer d (off, F) in launches of its own. Its neighbours' bit
// numbers go to 512 x blocks parts of cap words (part) with their counts.
struct RbPlan {
    uint32_t tiles = 0, ranges = 0, blocks = 0, cap = 0;
    uint64_t parts() const { return (uint64_t)blocks << kRbLgDigits; }
    uint64_t bytes() const { return parts() * cap * 4; }
};
RbPlan rb_plan(uint64_t F, uint32_t k);
void launch_rb_large(int n, const RbArgs &a, uint32_t d, uint64_t off, uint64_t F, const RbPlan &p, uint32_t *part,
                     uint32_t *count, PipeWork &w);

// A step by the unseen states: needs the bit numbers of no rank marked as
// seen (once), the inverse generators and a second bitmap, which holds the
// seen states afterwards.
void launch_rb_mark_unused(int n, uint32_t *seen, hipStream_t s);
void launch_rb_pull(int n, const RbArgs &a, uint32_t d, uint64_t off, uint64_t F, const GenSel *inv, uint32_t *to,
                    PipeWork &w);

}  // namespace cg
