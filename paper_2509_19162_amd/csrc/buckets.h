// Layers by hash buckets (buckets.hip): host-side declarations.
#pragma once

#include "internal.h"

namespace cg {

// ---- limits shared with the kernels ------------------------------------------
constexpr uint32_t kHashMaxLgDigits = 10;    // digits of one partition: 512 of the first, 1024 of the second
constexpr uint32_t kHashMaxLgSub = 6;        // buckets per partition beyond the second level: 64
constexpr uint32_t kHashLgSlots = 13;        // slots of a bucket's table, 64 KB: two workgroups per CU
constexpr uint32_t kHashBucket = 3072;       // states a bucket is planned for at most
constexpr uint32_t kHashMaxNew = 4096;       // new states of a bucket
constexpr int kHashStartBits = 40;           // bucket entry: start (40 bits) | count (24 bits)
constexpr uint64_t kHashStartMask = (1ull << kHashStartBits) - 1;
// device counters of one layer step
constexpr uint32_t kHashCount = 0;           // new states
constexpr uint32_t kHashFlags = 1;           // kHashFlag*
constexpr uint32_t kHashCounters = 2;
constexpr uint32_t kHashCounterStride = 64;  // words between the two sets
constexpr uint32_t kHashFlagPart = 1;        // a part of a partition overran
constexpr uint32_t kHashFlagTable = 2;       // a bucket's table overran

// one-workgroup layers: states of three layers together, candidates of one
constexpr uint32_t kSmallStates = 9216;
constexpr uint32_t kSmallMaxCand = 16384;
constexpr uint32_t kSmallSortStates = 16384; // longest run that launch_hash_sort_small takes
constexpr uint32_t kSmallMaxLayers = 1024;   // layers of one launch
// why a launch ended: buffers full or the next layer beyond the limits; the
// growth's end; a stop rule; the next layer's states did not fit the table
enum : uint32_t { kSmallMore = 0, kSmallDone = 1, kSmallStopped = 2, kSmallFull = 3 };

// A bit permutation as masked shifts (binary states).
struct BitTerm {
    uint64_t mask;
    uint32_t by;
    uint32_t left;
};

// Generators on the device: selectors (4-bit states) or masked shifts.
struct HashGens {
    bool binary = false;
    uint32_t k = 0;
    const GenSel *sel = nullptr;
    const BitTerm *term = nullptr;
    const uint32_t *first = nullptr;
};
// Masked shifts of k generators (rows of n bytes): terms of all generators,
// and per generator its first term (k + 1 entries).
void make_bit_terms(int n, const uint8_t *gens, int k, std::vector<BitTerm> &terms, std::vector<uint32_t> &first);

// Tags. A state's neighbours in layer d-1 are those it came from. So a
// candidate carries, above the state in its key, the bit of the generator
// that undoes its own; the bits of equal candidates are OR-ed; and the
// generators that take a state of a tagged layer back are left out, with
// them the look at layer d-1. For the LRX moves a state forms two neighbours
// or one instead of three: S_16 with layers up to 2^29 91 -> 73 ms, the
// C(32,16) binary states 44 -> 30. A key has 64 - 4n bits left (binary 64 -
// n), and four more in place of entry 0, which follows from the others, as
// the entries' sum is the orbit's. Where they suffice for half of the
// generators or more but not for all, those are left out and layer d-1 is
// looked at as without (14 entries, 13 adjacent swaps: 9.1 -> 8.3 ms).
constexpr uint32_t kHashMaxTags = 28;
struct HashTags {
    uint32_t mask_hi = ~0u;  // of a key's high word: the state without its tags
    uint32_t shift = 0;      // the tags: the high word from this bit on
    uint32_t sum = 0;        // entry 0 left out: 16 + the sum of a state's entries modulo 16
    uint32_t place = 0;      // ... and its first bit in the high word
    uint32_t all = 0;        // every generator has a tag
    uint32_t undo[kHashMaxTags] = {};  // the tag of the generator that undoes generator g (0: none)
    bool on() const { return mask_hi != ~0u; }
};

// A layer in buckets: 2^lg of them, each one run of `keys`; bucket[i] =
// start | count << kHashStartBits. lg == 0: the whole of keys[0..n), no table.
struct HashLayer {
    const uint64_t *keys = nullptr;
    uint64_t n = 0;
    const uint64_t *bucket = nullptr;
    uint32_t lg = 0;
    bool tagged = false;
};

// How one layer step is split.
struct HashPlan {
    uint64_t C = 0;
    uint32_t tiles = 0, ranges = 0, blocks = 0;  // first partition: items and workgroups
    uint32_t lg1 = 0, lg2 = 0, lg_sub = 0;       // digits, second-level digits, buckets per partition
    uint32_t cap1 = 0, cap2 = 0;                 // keys per part
    uint32_t lg_slots = 0;                       // of a bucket's table
    uint32_t lg_q() const { return lg1 + lg2 + lg_sub; }
    uint64_t bytes1() const { return ((uint64_t)blocks << lg1) * cap1 * 8; }
    uint64_t bytes2() const { return lg2 ? (1ull << (lg1 + lg2)) * cap2 * 8 : 0; }
    uint64_t counts1() const { return (uint64_t)blocks << lg1; }
    uint64_t counts2() const { return lg2 ? 1ull << (lg1 + lg2) : 0; }
};
// F states under k generators; `states`: the expected number of different
// states among the candidates and both reference layers. False when it needs
// more buckets than there are.
bool hash_plan(uint64_t F, uint32_t k, uint64_t states, HashPlan *p);

struct HashBufs {
    uint64_t *part1, *part2;
    uint32_t *count1, *count2;
    uint64_t *counters;  // kHashCounters words, zero before the step
    uint64_t *next;      // those of the next step (another line), cleared by this one
};
// Partitions the candidates of `cur`.
// (Those of a layer with all tags: each state's k - 1 at most; the plan is
// for as many.)
void launch_hash_partition(const HashPlan &p, const HashGens &g, const HashTags &t, const HashLayer &cur,
                           const HashBufs &b, PipeWork &w);
// dst[i] = the whole key of the state src[i] (dst may be src).
void launch_hash_strip(uint64_t *dst, const uint64_t *src, uint64_t n, const HashTags &t, hipStream_t s);
// Buckets: new states to out[0..out_cap) (the count in counters[kHashCount]
// goes on past out_cap), their buckets to out_bucket[0 .. 2^lg_q).
void launch_hash_buckets(const HashPlan &p, const HashLayer &prev, const HashLayer &cur, const HashBufs &b,
                         const HashTags &t, uint64_t *out, uint64_t out_cap, uint64_t *out_bucket, PipeWork &w);

struct HashSmallArgs {
    const uint64_t *prev, *cur;
    uint32_t np, nc, k;
    uint32_t max_new;          // layers this launch may add (at most kSmallMaxLayers)
    uint32_t max_new_is_rule;  // reaching max_new is the caller's max_layers rule
    uint64_t max_frontier;
    uint64_t *out;             // the new layers, one after another
    uint64_t out_cap;
    uint64_t *sizes;           // sizes of the new layers (the last may be 0)
    uint32_t *state;           // [0] layers added (an empty one included), [1] kSmall*
};
void launch_hash_small(const HashSmallArgs &a, const HashGens &g, const HashTags &t, PipeWork &w);
// Sorts `layers` consecutive runs of keys (at most kSmallSortStates each) in
// place; the runs' lengths are at sizes[0..layers).
void launch_hash_sort_small(uint64_t *keys, const uint64_t *sizes, uint32_t layers, hipStream_t s);

}  // namespace cg
