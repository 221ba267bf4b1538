// Layers by hash buckets: the layer step of sets closed under inverses,
// without a sort.
//
// A candidate (a neighbour s.g of a layer-d state) is a new state iff it is
// the first of its copies and lies neither in layer d nor in layer d-1. No
// order is needed to decide that, only that equal keys meet. So the
// candidates are partitioned by a hash of their key into buckets whose
// states, those of all three layers together, fit a hash table in LDS; one
// workgroup per bucket inserts the bucket's states of layers d-1 and d,
// then its candidates. Whole keys are compared, so nothing rests on the
// hash but the balance of the buckets: a bucket or a table that overruns
// raises a flag, and the host takes more buckets or hands the layer to the
// sort path.
//
//   hash_expand_kernel  expand + first partition (partition_device.h): candidates are formed in
//                       registers and go to up to 512 digits;
//   hash_split_kernel   second partition (large layers): one workgroup per
//                       first-level digit;
//   hash_bucket_kernel  one workgroup per bucket: the LDS table; survivors
//                       go to the new layer, bucket by bucket;
//   hash_small_kernel   whole layers, one after another, in one workgroup
//                       while the three layers fit one table.
//
// Traffic per candidate: 8 bytes written, then 8 read and 8 written when
// there is a second partition, then 8 read; per state 8 written once and
// read three times. An LSD sort of the same candidates moves 16 bytes per
// pass and takes 6 passes for S_16, 4 for binary states of n = 32.
#include "buckets.h"

#include <algorithm>
#include <cstring>

#include "device_util.h"
#include "expand_device.h"
#include "partition_device.h"

namespace cg {

namespace {

constexpr int kPartRows = 4;               // candidates per thread and round
constexpr uint32_t kPartTile = kPartBlock * kPartRows;
static_assert(kHashMaxLgDigits <= kPartMaxLgDigits, "digits of a partition");

constexpr int kBucketBlock = 1024;         // threads of a bucket workgroup
constexpr uint32_t kBucketWaves = kBucketBlock / kWave;
constexpr uint32_t kMaxProbes = 512;       // a longer probe means an overfull table

constexpr uint32_t kSmallLgSlots = 14;     // table of the one-workgroup kernel: 128 KB
constexpr uint32_t kSmallSlots = 1u << kSmallLgSlots;

// ---- hash -------------------------------------------------------------------
// The top bits pick the digits of both partitions. Two rounds of a 32 x 32 -> 64-bit product of two halves
// that both depend on the key. A linear hash (multiplications by constants)
// will not do: it commutes with the moves that shift a state, so the
// neighbours of one bucket's states met in a few digits (12 times the
// spread of uniform draws on binary Coxeter layers, 7 on LRX). With these
// two rounds the parts of one workgroup spread as uniform draws on layers of
// LRX, Coxeter, pancake, star, 3-cycle and reversal growths of
// permutations, multisets and binary states.
__device__ __forceinline__ uint32_t key_hash(uint64_t key) {
    const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
    const uint64_t r = (uint64_t)(lo ^ 0x9E3779B1u) * (((lo << 16) | (lo >> 16)) ^ hi ^ 0x85EBCA77u);
    const uint32_t rl = (uint32_t)r, rh = (uint32_t)(r >> 32);
    const uint64_t t = (uint64_t)(rl ^ rh ^ 0x27D4EB2Fu) * ((rh ^ 0x165667B1u) | 1u);
    return (uint32_t)t ^ (uint32_t)(t >> 32);
}

// ---- generators -----------------------------------------------------------------
// Generators are read-only and the same in every lane: read through the
// constant address space they come by scalar loads (the kernels' stores
// would otherwise have to be assumed to change them).
template <class T>
using ConstPtr = const T __attribute__((address_space(4))) *;
template <class T>
__device__ __forceinline__ ConstPtr<T> const_ptr(const T *p) {
    return (ConstPtr<T>)(uintptr_t)p;
}
struct NibbleGens {
    const GenSel *sel;
    __device__ __forceinline__ uint64_t apply(uint64_t s, uint32_t g) const {
        ConstPtr<uint32_t> p = const_ptr(&sel[g].sel[0]);
        GenSel v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v.sel[i] = p[i];
        return apply_gensel(s, v);
    }
    // the same where g differs from lane to lane
    __device__ __forceinline__ uint64_t apply_lane(uint64_t s, uint32_t g) const { return apply_gensel(s, sel[g]); }
};
// Binary states: a generator moves key bit p to bit p + shift; the bits that
// share a shift are one mask, so a candidate is the OR of a few masked
// shifts (2 or 3 for the LRX moves), the same in every lane.
struct BitGens {
    const BitTerm *term;
    const uint32_t *first;  // terms of generator g: first[g] .. first[g+1]
    __device__ __forceinline__ uint64_t apply(uint64_t s, uint32_t g) const {
        uint64_t t = 0;
        const uint32_t end = const_ptr(first)[g + 1];
        for (uint32_t i = const_ptr(first)[g]; i < end; ++i) {
            const uint64_t x = s & const_ptr(&term[i].mask)[0];
            const uint32_t by = const_ptr(&term[i].by)[0];
            t |= const_ptr(&term[i].left)[0] ? x << by : x >> by;
        }
        return t;
    }
    __device__ __forceinline__ uint64_t apply_lane(uint64_t s, uint32_t g) const {
        uint64_t t = 0;
        for (uint32_t i = first[g]; i < first[g + 1]; ++i) {
            const BitTerm x = term[i];
            t |= x.left ? (s & x.mask) << x.by : (s & x.mask) >> x.by;
        }
        return t;
    }
};

// ---- tags --------------------------------------------------------------------------
__device__ __forceinline__ uint64_t tag_off(uint64_t key, uint32_t mask_hi) {
    return (uint64_t)((uint32_t)(key >> 32) & mask_hi) << 32 | (uint32_t)key;
}
// The whole key: without its tags, entry 0 put back where it was left out.
__device__ __forceinline__ uint64_t tag_strip(uint64_t key, const HashTags &t) {
    key = tag_off(key, t.mask_hi);
    if (t.sum) {
        const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32), m = 0x0F0F0F0Fu;
        const uint32_t four = (lo & m) + ((lo >> 4) & m) + (hi & m) + ((hi >> 4) & m);  // bytes up to 60
        key |= (uint64_t)(((t.sum - __builtin_amdgcn_sad_u8(four, 0u, 0u)) & 15u) << t.place) << 32;
    }
    return key;
}

// Items of (4096 frontier states) x (a range of generators), dealt to the
// blocks in turn. The item's states stay in registers; each round maps them
// through one generator. A candidate equal to its state is dropped here. Of
// a layer with all tags there are k - 1 rounds: in the first that would take
// a state back it takes the last generator (if that does not).
// kTags: the growth has tags (without, nothing is spent on them: the checks
// cost the Coxeter growth of a 14-entry coset graph 9%).
template <class G, bool kTags>
__global__ __launch_bounds__(kPartBlock) void hash_expand_kernel(const uint64_t *__restrict__ frontier, uint64_t F,
                                                                 G gens, uint32_t k, HashTags tags, bool tagged,
                                                                 uint32_t tiles, uint32_t ranges, uint32_t lg,
                                                                 PartOut<uint64_t> o, uint64_t *next) {
    __shared__ PartLds<uint64_t> L;
    const uint32_t tid = threadIdx.x;
    // the next step's counters, not this one's: a plain store would reach
    // memory after other workgroups' atomics on the same line
    if (blockIdx.x == 0 && tid < kHashCounters) next[tid] = 0;
    part_begin(L, 1u << lg);
    o.base += (uint64_t)blockIdx.x * o.cap;
    o.count += blockIdx.x;
    uint32_t parity = 0;
    const bool swap = kTags && tagged && tags.all;
    const uint32_t rounds = swap ? k - 1 : k;
    for (uint32_t it = blockIdx.x; it < tiles * ranges; it += gridDim.x) {
        const uint32_t tile = it / ranges, range = it - tile * ranges;
        const uint32_t g0 = (uint32_t)((uint64_t)rounds * range / ranges);
        const uint32_t g1 = (uint32_t)((uint64_t)rounds * (range + 1) / ranges);
        uint64_t s[kPartRows], last[kPartRows];
        uint32_t back[kPartRows], in = 0;
#pragma unroll
        for (int j = 0; j < kPartRows; ++j) {
            const uint64_t f = (uint64_t)tile * kPartTile + (uint32_t)j * kPartBlock + tid;
            const uint64_t x = f < F ? frontier[f] : 0ull;
            if (f < F) in |= 1u << j;
            s[j] = kTags ? tag_strip(x, tags) : x;
            back[j] = kTags && tagged ? (uint32_t)(x >> 32) >> tags.shift : 0u;
        }
        if (swap) {
#pragma unroll
            for (int j = 0; j < kPartRows; ++j) last[j] = gens.apply(s[j], k - 1);
        }
        for (uint32_t g = g0; g < g1; ++g) {
            uint64_t c[kPartRows];
            uint32_t pend = in, tag[kPartRows];
#pragma unroll
            for (int j = 0; j < kPartRows; ++j) {
                c[j] = gens.apply(s[j], g);
                if constexpr (kTags) {
                    // g takes the state back, as the first that does: -x & x is its bit
                    const uint32_t x = back[j];
                    const bool over = (x >> g) & 1u;
                    const bool instead = swap && over && (x & (0u - x)) >> g == 1u && !((x >> (k - 1)) & 1u);
                    if (instead) c[j] = last[j];
                    if (over && !instead) pend &= ~(1u << j);
                    tag[j] = instead ? tags.undo[k - 1] : tags.undo[g];
                }
                if (c[j] == s[j]) pend &= ~(1u << j);
            }
            uint32_t dig[kPartRows];
#pragma unroll
            for (int j = 0; j < kPartRows; ++j) {
                if constexpr (kTags) c[j] = tag_off(c[j], tags.mask_hi);
                dig[j] = key_hash(c[j]) >> (32 - lg);
                if constexpr (kTags) c[j] |= (uint64_t)tag[j] << 32;
            }
            part_round(L, c, dig, pend, lg, o, parity);
        }
    }
    part_end(L, lg, o);
}

// Second partition: block d takes digit d's keys from every first-level
// block. A wave walks its share of the source blocks' parts; the block goes
// on while any wave has keys left.
template <bool kTags>
__global__ __launch_bounds__(kPartBlock) void hash_split_kernel(const uint64_t *__restrict__ in,
                                                                const uint32_t *__restrict__ in_count, uint32_t nsrc,
                                                                uint32_t in_cap, uint32_t mask_hi, uint32_t lg1,
                                                                uint32_t lg2, PartOut<uint64_t> o) {
    __shared__ PartLds<uint64_t> L;
    constexpr uint32_t kWaves = kPartBlock / kWave;
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t d = blockIdx.x;
    part_begin(L, 1u << lg2);
    o.base += (uint64_t)d * (o.stride << lg2);
    o.count += (uint64_t)d << lg2;
    uint32_t parity = 0;
    uint32_t src = wave, at = 0;
    uint32_t n = src < nsrc ? in_count[(uint64_t)d * nsrc + src] : 0u;
    for (;;) {
        while (src < nsrc && at >= n) {
            src += kWaves;
            at = 0;
            n = src < nsrc ? in_count[(uint64_t)d * nsrc + src] : 0u;
        }
        const bool any = src < nsrc;
        uint64_t key[kPartRows];
        uint32_t pend = 0;
        if (any) {
            const uint64_t *p = in + ((uint64_t)d * nsrc + src) * in_cap;
#pragma unroll
            for (int j = 0; j < kPartRows; ++j) {
                const uint32_t i = at + (uint32_t)j * kWave + lane;
                key[j] = i < n ? p[i] : 0ull;
                if (i < n) pend |= 1u << j;
            }
            at += kPartRows * kWave;
        } else {
#pragma unroll
            for (int j = 0; j < kPartRows; ++j) key[j] = 0;
        }
        if (!__syncthreads_or(any)) break;
        uint32_t dig[kPartRows];
#pragma unroll
        for (int j = 0; j < kPartRows; ++j) dig[j] = (key_hash(kTags ? tag_off(key[j], mask_hi) : key[j]) << lg1) >> (32 - lg2);
        part_round(L, key, dig, pend, lg2, o, parity);
    }
    part_end(L, lg2, o);
}

// Values that are the same in every lane but were loaded per lane: in scalar
// registers from here on.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint64_t uniform(uint64_t x) {
    return (uint64_t)uniform((uint32_t)(x >> 32)) << 32 | uniform((uint32_t)x);
}

// ---- LDS tables ----------------------------------------------------------------
// Open addressing over whole 64-bit keys (kSentinel = free), 2^lg slots, an
// odd stride per key. The compare-and-swap is the probe: it reads, and takes
// a free slot at once. One key per lane at a time: with tables at most 3/8
// full a wave is done after about three probes. True when the key was not
// in the table (its slot in `slot`); keys that differ in their tags only are
// the same, and their tags are OR-ed. A probe past kMaxProbes raises *over.
template <bool kTags>
__device__ __forceinline__ bool table_insert(uint64_t *tab, uint32_t lg, uint64_t key, uint32_t mask_hi, bool on,
                                             uint32_t &slot, uint32_t *over) {
    // linear in the key's halves: enough among the states of one bucket,
    // which are a random subset (slots fill as by uniform draws on the
    // layers named at the hash above)
    const uint32_t hi = kTags ? (uint32_t)(key >> 32) & mask_hi : (uint32_t)(key >> 32);
    const uint32_t h = (uint32_t)key * 0x9E3779B1u + hi * 0x85EBCA77u;
    const uint32_t mask = (1u << lg) - 1u, step = h | 1u;
    slot = h >> (32 - lg);
    bool fresh = false;
    uint32_t probes = 0;
    while (on) {
        const uint64_t old = atomicCAS((unsigned long long *)&tab[slot], (unsigned long long)kSentinel,
                                       (unsigned long long)key);
        fresh = old == kSentinel;
        if (fresh || (!kTags && old == key)) break;
        if (kTags && tag_off(old ^ key, mask_hi) == 0) {
            const uint32_t tags = (uint32_t)(key >> 32) & ~mask_hi;
            if (tags & ~(uint32_t)(old >> 32)) atomicOr(reinterpret_cast<uint32_t *>(&tab[slot]) + 1, tags);
            break;
        }
        slot = (slot + step) & mask;
        if (++probes > kMaxProbes) {
            *over = 1;
            break;
        }
    }
    return fresh;
}

struct alignas(16) BucketLds {
    uint64_t tab[1u << kHashLgSlots];
    uint16_t list[kHashMaxNew];  // slots of the new states
    uint32_t found, over;
    uint64_t base;
};

struct LayerRef {
    const uint64_t *keys;
    const uint64_t *bucket;  // start | count << 40 per bucket
    uint64_t n;
    uint32_t lg;             // log2 of its buckets (0: one, without a table)
};

struct BucketArgs {
    const uint64_t *in;        // candidates: nsrc parts of in_cap keys per partition
    const uint32_t *in_count;
    uint32_t nsrc, in_cap;
    uint32_t lg_q, lg_sub;     // bucket q of 2^lg_q lies in partition q >> lg_sub
    uint32_t lg_slots;
    uint32_t mask_hi;          // of the keys' tags
    LayerRef A, B;             // layers d and d-1
    uint64_t *out;
    uint64_t out_cap;
    uint64_t *out_bucket;
    uint64_t *counters;
};

// A layer's run for bucket q, where the layer has no more buckets than the
// step: start | count << 40.
__device__ __forceinline__ uint64_t run_of(const LayerRef &R, uint32_t q, uint32_t lg_q) {
    if (!R.n) return 0;
    return R.lg ? uniform(R.bucket[q >> (lg_q - R.lg)]) : R.n << kHashStartBits;
}

// Inserts the keys of `act` that lie in bucket q; the slots of those that
// were new go to the list (candidates) or are forgotten (references).
template <bool kTags, int R>
__device__ __forceinline__ void bucket_insert(BucketLds &L, const BucketArgs &a, const uint64_t (&key)[R],
                                              uint32_t act, uint32_t q, bool filter, bool refs) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
        bool on = (act >> u) & 1u;
        const uint32_t mask_hi = kTags ? a.mask_hi : ~0u;
        if (filter) on = on && (key_hash(tag_off(key[u], mask_hi)) >> (32 - a.lg_q)) == q;
        uint32_t slot;
        // references: with all tags, so that none are added
        const uint64_t x = refs ? key[u] | (uint64_t)~mask_hi << 32 : key[u];
        const bool fresh = table_insert<kTags>(L.tab, a.lg_slots, x, mask_hi, on, slot, &L.over);
        if (refs) continue;
        const uint64_t m = __ballot(fresh);
        if (!m) continue;
        uint32_t at = 0;
        if (lane_id() == 0) at = atomicAdd(&L.found, (uint32_t)__popcll(m));
        at = uniform(at) + mask_rank(m);
        if (fresh && at < kHashMaxNew) L.list[at] = (uint16_t)slot;
    }
}

__device__ __forceinline__ void bucket_begin(BucketLds &L, uint32_t lg_slots) {
    // two slots per store (lg_slots >= 9)
    ulonglong2 *const t = reinterpret_cast<ulonglong2 *>(L.tab);
    for (uint32_t i = threadIdx.x; i < (1u << lg_slots) / 2; i += kBucketBlock) t[i] = make_ulonglong2(kSentinel, kSentinel);
    if (threadIdx.x == 0) L.found = L.over = 0;
    __syncthreads();
}

__device__ __forceinline__ void bucket_end(BucketLds &L, const BucketArgs &a, uint32_t q) {
    __syncthreads();
    const uint32_t n = L.found;
    if (threadIdx.x == 0) {
        const uint64_t base =
            n ? atomicAdd((unsigned long long *)&a.counters[kHashCount], (unsigned long long)n) : 0ull;
        L.base = base;
        a.out_bucket[q] = (base & kHashStartMask) | (uint64_t)n << kHashStartBits;
        if (L.over || n > kHashMaxNew) atomicOr((uint32_t *)&a.counters[kHashFlags], kHashFlagTable);
    }
    __syncthreads();
    const uint64_t base = L.base;
    for (uint32_t i = threadIdx.x; i < n && i < kHashMaxNew; i += kBucketBlock)
        if (base + i < a.out_cap) a.out[base + i] = L.tab[L.list[i]];
    __syncthreads();
}

// Large layers: one run of candidates per partition (nsrc == 1), and both
// reference layers with no more buckets than this step. The blocks are
// persistent and take the buckets in turn; two stages each: the reference
// states (layer d's run, then layer d-1's, as one sequence), the candidates.
// A bucket is two or three keys per thread, so what is loaded has to be on
// its way long before: the first keys of either stage while the previous
// bucket's same stage goes into the table, where they lie a bucket earlier
// still. (Loaded a stage ahead, with the places
// read just before: S_16, layers up to 2^29, 33.4 ms in this kernel, now 29.7.)
template <bool kTags>
__global__ __launch_bounds__(kBucketBlock) __attribute__((amdgpu_waves_per_eu(8))) void hash_bucket_kernel(
    BucketArgs a) {
    __shared__ BucketLds L;
    constexpr int kRows = 2;
    constexpr uint32_t kStep = kRows * kBucketBlock;
    const uint32_t tid = threadIdx.x, Q = 1u << a.lg_q;
    struct Runs {  // a bucket's runs: layer d's, layer d-1's, candidates
        uint64_t ea, eb;
        uint32_t nc;
    };
    auto look = [&](uint32_t q) {  // as loaded
        Runs r{0, 0, 0};
        if (q < Q) {
            if (a.A.n) r.ea = a.A.lg ? a.A.bucket[q >> (a.lg_q - a.A.lg)] : a.A.n << kHashStartBits;
            if (a.B.n) r.eb = a.B.lg ? a.B.bucket[q >> (a.lg_q - a.B.lg)] : a.B.n << kHashStartBits;
            r.nc = a.in_count[q >> a.lg_sub];
        }
        return r;
    };
    auto settle = [&](const Runs &r) { return Runs{uniform(r.ea), uniform(r.eb), uniform(r.nc)}; };
    auto total = [&](const Runs &r, uint32_t stage) -> uint32_t {
        return stage ? r.nc : (uint32_t)(r.ea >> kHashStartBits) + (uint32_t)(r.eb >> kHashStartBits);
    };
    auto load = [&](uint64_t (&key)[kRows], const Runs &r, uint32_t q, uint32_t stage, uint32_t b) -> uint32_t {
        uint32_t act = 0;
        const uint32_t n = total(r, stage), na = (uint32_t)(r.ea >> kHashStartBits);
        const uint64_t *pa = stage ? a.in + (uint64_t)(q >> a.lg_sub) * a.in_cap : a.A.keys + (r.ea & kHashStartMask);
        const uint64_t *pb = stage ? pa : a.B.keys + (r.eb & kHashStartMask) - na;
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const uint32_t i = b + (uint32_t)u * kBucketBlock + tid;
            key[u] = 0;
            if (i < n) {
                const uint64_t *p = i < na ? pa : pb;
                key[u] = p[i];
                act |= 1u << u;
            }
        }
        return act;
    };
    const bool filter0 = a.A.lg < a.lg_q || a.B.lg < a.lg_q;
    const uint32_t G = gridDim.x;
    uint32_t q = blockIdx.x;
    Runs now = settle(look(q)), next = settle(look(q + G));
    uint64_t pre[2][kRows];
    uint32_t pact[2];
#pragma unroll
    for (uint32_t stage = 0; stage < 2; ++stage) pact[stage] = load(pre[stage], now, q, stage, 0);
    for (; q < Q; q += G) {
        const Runs after = look(q + 2 * G);
        bucket_begin(L, a.lg_slots);
#pragma unroll
        for (uint32_t stage = 0; stage < 2; ++stage) {
            uint64_t key[kRows];
            uint32_t act = pact[stage];
#pragma unroll
            for (int u = 0; u < kRows; ++u) key[u] = pre[stage][u];
            pact[stage] = load(pre[stage], next, q + G, stage, 0);
            const uint32_t n = total(now, stage);
            for (uint32_t b = 0;;) {
                bucket_insert<kTags>(L, a, key, act, q, stage ? a.lg_sub != 0 : filter0, stage == 0);
                b += kStep;
                if (b >= n) break;
                act = load(key, now, q, stage, b);
            }
            if (stage == 0) __syncthreads();
        }
        bucket_end(L, a, q);
        now = next;
        next = settle(after);
    }
}

// Any other step: candidates in several parts (one partition), or reference
// layers with more buckets than this step. One block per bucket; its waves
// take pieces in turn: 256 keys of a run, or a whole (small) run.
template <bool kTags>
__global__ __launch_bounds__(kBucketBlock) __attribute__((amdgpu_waves_per_eu(8))) void hash_bucket_pieces_kernel(
    BucketArgs a) {
    __shared__ BucketLds L;
    constexpr uint32_t kPiece = 4 * kWave;
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, q = blockIdx.x;
    auto pieces = [&](const LayerRef &R) -> uint32_t {
        if (!R.n) return 0;
        if (R.lg > a.lg_q) return 1u << (R.lg - a.lg_q);
        return ((uint32_t)(run_of(R, q, a.lg_q) >> kHashStartBits) + kPiece - 1) / kPiece;
    };
    const uint32_t na = pieces(a.A), nb = pieces(a.B);
    bucket_begin(L, a.lg_slots);
    for (uint32_t stage = 0; stage < 2; ++stage) {
        const uint32_t np = stage ? a.nsrc : na + nb;
        for (uint32_t i = wave; i < np; i += kBucketWaves) {
            const uint64_t *p;
            uint32_t n, b = 0;
            bool filter = a.lg_sub != 0;
            if (stage) {
                const uint64_t part = (uint64_t)(q >> a.lg_sub) * a.nsrc + i;
                p = a.in + part * a.in_cap;
                n = a.in_count[part];
            } else {
                const LayerRef &R = i < na ? a.A : a.B;
                const uint32_t j = i < na ? i : i - na;
                const bool many = R.lg > a.lg_q;
                const uint64_t e = many ? R.bucket[((uint64_t)q << (R.lg - a.lg_q)) + j] : run_of(R, q, a.lg_q);
                p = R.keys + (e & kHashStartMask);
                n = (uint32_t)(e >> kHashStartBits);
                if (!many) {
                    b = j * kPiece;
                    n = n < b + kPiece ? n : b + kPiece;
                }
                filter = R.lg < a.lg_q;
            }
            for (; b < n; b += kPiece) {
                uint64_t key[4];
                uint32_t act = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t k = b + (uint32_t)u * kWave + lane;
                    key[u] = k < n ? p[k] : 0ull;
                    if (k < n) act |= 1u << u;
                }
                bucket_insert<kTags>(L, a, key, act, q, filter, stage == 0);
            }
        }
        if (stage == 0) __syncthreads();
    }
    bucket_end(L, a, q);
}

// ---- small layers ---------------------------------------------------------------
// Whole layers in one workgroup while layers d-1, d and d+1 fit its table.
// Layers follow one another in `out` (a ring is not needed: the caller
// bounds the total). Ends when the growth ends, a stop rule holds, the next
// layer might be too large, or the buffers are full.
struct SmallLds {
    uint64_t tab[1u << kSmallLgSlots];
    uint32_t count, over;
};

template <class G, bool kTags>
__global__ __launch_bounds__(kPartBlock) void hash_small_kernel(HashSmallArgs a, G gens, HashTags tags) {
    __shared__ SmallLds L;
    const uint32_t tid = threadIdx.x;
    const uint64_t *prev = a.prev, *cur = a.cur;
    uint32_t np = a.np, nc = a.nc;
    uint32_t used = 0, made = 0, code = kSmallMore;
    for (;;) {
        if (a.max_frontier && nc > a.max_frontier) {
            code = kSmallStopped;
            break;
        }
        if (made >= a.max_new) {
            code = a.max_new_is_rule ? kSmallStopped : kSmallMore;
            break;
        }
        const uint64_t C = (uint64_t)nc * a.k;
        if (C > kSmallMaxCand || np + nc > kSmallStates || used + kSmallStates > a.out_cap) break;
        for (uint32_t i = tid; i < kSmallSlots; i += kPartBlock) L.tab[i] = kSentinel;
        if (tid == 0) L.count = L.over = 0;
        __syncthreads();
        for (int which = 0; which < 2; ++which) {
            const uint64_t *p = which ? cur : prev;
            const uint32_t n = which ? nc : np;
            for (uint32_t i = tid; i < n; i += kPartBlock) {
                uint32_t slot;
                (void)table_insert<false>(L.tab, kSmallLgSlots, kTags ? tag_strip(p[i], tags) : p[i], ~0u, true, slot, &L.over);
            }
        }
        __syncthreads();
        const uint32_t budget = kSmallStates - np - nc;
        uint64_t *o = a.out + used;
        // a thread takes a state under one generator; whole waves go round
        // together (the ballot below)
        const uint32_t work = nc * a.k;
        // w / nc for w < 2^15: one multiplication
        const uint32_t inv = (uint32_t)(((1ull << 32) + nc - 1) / nc);
        static_assert(kSmallMaxCand + kPartBlock <= (1u << 15) && kSmallStates <= (1u << 14), "exact quotients");
        for (uint32_t w0 = 0; w0 < work; w0 += kPartBlock) {
            const uint32_t w = w0 + tid, g = nc == 1 ? w : __umulhi(w, inv), f = w - g * nc;
            uint64_t s = 0, key = 0;
            if (w < work) {
                s = kTags ? tag_strip(cur[f], tags) : cur[f];
                key = gens.apply_lane(s, g);
            }
            uint32_t slot;
            const bool fresh = table_insert<false>(L.tab, kSmallLgSlots, key, ~0u, key != s, slot, &L.over);
            const uint64_t m = __ballot(fresh);
            if (!m) continue;
            uint32_t at = 0;
            if (lane_id() == 0) at = atomicAdd(&L.count, (uint32_t)__popcll(m));
            const uint32_t base = uniform(at);
            at = base + mask_rank(m);
            if (fresh && at < kSmallStates) o[at] = key;
            if (base > budget) break;  // too many for the table: the layer is done again elsewhere
        }
        __syncthreads();
        const uint32_t n = L.count, over = L.over;
        if (n > budget || over) {
            code = kSmallFull;
            break;
        }
        if (tid == 0) a.sizes[made] = n;
        __syncthreads();  // the layer's stores are done (and L.count is read) before it is expanded
        ++made;
        prev = cur;
        np = nc;
        cur = o;
        nc = n;
        used += n;
        if (n == 0) {
            code = kSmallDone;
            break;
        }
    }
    if (tid == 0) {
        a.state[0] = made;
        a.state[1] = code;
    }
}

}  // namespace

namespace {
__global__ __launch_bounds__(256) void hash_strip_kernel(uint64_t *dst, const uint64_t *src, uint64_t n, HashTags t) {
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
        dst[i] = tag_strip(src[i], t);
}
}  // namespace

void launch_hash_strip(uint64_t *dst, const uint64_t *src, uint64_t n, const HashTags &t, hipStream_t s) {
    const uint64_t blocks = std::min<uint64_t>((n + 255) / 256, 4096);
    if (!blocks) return;
    hipLaunchKernelGGL(hash_strip_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, dst, src, n, t);
    CG_HIP(hipGetLastError());
}

// ---- sorted small layers (for callers that read states back) -----------------------
namespace {

// One workgroup per layer: bitonic sort in LDS.
__global__ __launch_bounds__(kPartBlock) void hash_sort_small_kernel(uint64_t *keys, const uint64_t *sizes) {
    __shared__ uint64_t s[kSmallSlots];
    uint64_t start = 0;
    for (uint32_t i = 0; i < blockIdx.x; ++i) start += sizes[i];
    const uint32_t n = (uint32_t)sizes[blockIdx.x];
    if (n > kSmallSlots) return;
    uint32_t m = 2;
    while (m < n) m <<= 1;
    for (uint32_t i = threadIdx.x; i < m; i += kPartBlock) s[i] = i < n ? keys[start + i] : kSentinel;
    __syncthreads();
    for (uint32_t span = 2; span <= m; span <<= 1)
        for (uint32_t step = span >> 1; step; step >>= 1) {
            for (uint32_t t = threadIdx.x; t < m / 2; t += kPartBlock) {
                const uint32_t i = 2 * t - (t & (step - 1));
                const uint64_t a = s[i], b = s[i + step];
                if ((a > b) == ((i & span) == 0)) {
                    s[i] = b;
                    s[i + step] = a;
                }
            }
            __syncthreads();
        }
    for (uint32_t i = threadIdx.x; i < n; i += kPartBlock) keys[start + i] = s[i];
}

uint32_t ceil_log2(uint64_t x) {
    uint32_t l = 0;
    while ((1ull << l) < x) ++l;
    return l;
}

}  // namespace

void launch_hash_sort_small(uint64_t *keys, const uint64_t *sizes, uint32_t layers, hipStream_t s) {
    if (!layers) return;
    hipLaunchKernelGGL(hash_sort_small_kernel, dim3(layers), dim3(kPartBlock), 0, s, keys, sizes);
    CG_HIP(hipGetLastError());
}

void make_bit_terms(int n, const uint8_t *gens, int k, std::vector<BitTerm> &terms, std::vector<uint32_t> &first) {
    terms.clear();
    first.assign(1, 0);
    for (int g = 0; g < k; ++g) {
        const uint8_t *r = gens + (size_t)g * n;
        // candidate entry i (bit n-1-i) is entry r[i] (bit n-1-r[i]): left by r[i] - i
        for (int d = -(n - 1); d <= n - 1; ++d) {
            uint64_t mask = 0;
            for (int i = 0; i < n; ++i)
                if ((int)r[i] - i == d) mask |= 1ull << (n - 1 - r[i]);
            if (mask) terms.push_back(BitTerm{mask, (uint32_t)(d < 0 ? -d : d), d > 0 ? 1u : 0u});
        }
        first.push_back((uint32_t)terms.size());
    }
}

bool hash_plan(uint64_t F, uint32_t k, uint64_t states, HashPlan *p) {
    p->C = F * (uint64_t)k;
    const uint64_t tiles = (F + kPartTile - 1) / kPartTile;
    if (tiles * k >= (1ull << 31)) return false;
    p->tiles = (uint32_t)tiles;
    // a workgroup per CU; a small frontier is dealt out by generator too
    p->ranges = tiles >= 512 ? 1u : (uint32_t)std::min<uint64_t>(k, (512 + tiles - 1) / tiles);
    const uint64_t items = tiles * p->ranges;
    p->blocks = (uint32_t)std::min<uint64_t>(items, 256);
    const double per_item = (double)std::min<uint64_t>(F, kPartTile) * (double)((k + p->ranges - 1) / p->ranges);
    const double per_block = per_item * (double)((items + p->blocks - 1) / p->blocks);
    p->lg2 = p->lg_sub = 0;
    // one partition while its 512 digits leave buckets of at most
    // kHashBucket states (a table then stays 3/8 full at most)
    if (states <= ((uint64_t)kHashBucket << 9)) {
        p->lg1 = std::max(4u, std::min(9u, ceil_log2((states + 511) / 512)));
    } else {
        const uint32_t lg = ceil_log2((states + kHashBucket - 1) / kHashBucket);
        // a workgroup of the second one per digit: one per CU, where that
        // makes buckets enough (of 8192 small ones their number is what
        // costs: 12 ns each for their place in the layer; 14-entry coset
        // graph under 13 swaps with 512 digits throughout 9.4 ms, now 8.0,
        // C(32,16) binary LRX 29.5 and 28.8)
        p->lg1 = lg <= 12 ? 8u : 9u;
        p->lg2 = std::min(kHashMaxLgDigits, std::max(4u, lg - p->lg1));
        if (lg > p->lg1 + p->lg2) p->lg_sub = lg - p->lg1 - p->lg2;
        if (p->lg_sub > kHashMaxLgSub) return false;
    }
    p->cap1 = part_cap(per_block / (double)(1u << p->lg1), k);
    p->cap2 = p->lg2 ? part_cap((double)p->C / (double)(1ull << (p->lg1 + p->lg2)), k) : 0;
    // table: at least 8/3 of the expected states, and room to spare for few
    const uint64_t per_bucket = states >> p->lg_q();
    p->lg_slots = std::min(kHashLgSlots, std::max(9u, ceil_log2(8 * per_bucket / 3 + 128)));
    return true;
}

namespace {

template <class Fn>
void with_gens(const HashGens &g, Fn &&fn) {
    if (g.binary)
        fn(BitGens{g.term, g.first});
    else
        fn(NibbleGens{g.sel});
}

}  // namespace

void launch_hash_partition(const HashPlan &p, const HashGens &g, const HashTags &t, const HashLayer &cur,
                           const HashBufs &b, PipeWork &w) {
    if (w.prof) w.prof->begin(K_EXPAND);
    PartOut<uint64_t> o{b.part1, (uint64_t)p.blocks * p.cap1, p.cap1, b.count1, p.blocks,
                        (uint32_t *)&b.counters[kHashFlags], kHashFlagPart};
    with_gens(g, [&](auto gens) {
        auto kernel = t.on() ? hash_expand_kernel<decltype(gens), true> : hash_expand_kernel<decltype(gens), false>;
        hipLaunchKernelGGL(kernel, dim3(p.blocks), dim3(kPartBlock), 0, w.stream, cur.keys, cur.n, gens, g.k, t,
                           cur.tagged, p.tiles, p.ranges, p.lg1, o, b.next);
    });
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->end(K_EXPAND, 8.0 * (double)cur.n + 8.0 * (double)p.C, (double)p.C);
    if (p.lg2) {
        if (w.prof) w.prof->begin(K_SPLIT);
        PartOut<uint64_t> o2{b.part2, p.cap2, p.cap2, b.count2, 1, (uint32_t *)&b.counters[kHashFlags], kHashFlagPart};
        hipLaunchKernelGGL(t.on() ? hash_split_kernel<true> : hash_split_kernel<false>, dim3(1u << p.lg1), dim3(kPartBlock), 0, w.stream, b.part1, b.count1,
                           p.blocks, p.cap1, t.mask_hi, p.lg1, p.lg2, o2);
        CG_HIP(hipGetLastError());
        if (w.prof) w.prof->end(K_SPLIT, 16.0 * (double)p.C, (double)p.C);
    }
}

void launch_hash_buckets(const HashPlan &p, const HashLayer &prev, const HashLayer &cur, const HashBufs &b,
                         const HashTags &t, uint64_t *out, uint64_t out_cap, uint64_t *out_bucket, PipeWork &w) {
    if (w.prof) w.prof->begin(K_BUCKET);
    const LayerRef A{cur.keys, cur.bucket, cur.n, cur.lg};
    const LayerRef B = cur.tagged && t.all ? LayerRef{nullptr, nullptr, 0, 0} : LayerRef{prev.keys, prev.bucket, prev.n, prev.lg};
    const bool two = p.lg2 != 0;
    const uint32_t lg_q = p.lg_q();
    BucketArgs a{two ? b.part2 : b.part1, two ? b.count2 : b.count1, two ? 1u : p.blocks, two ? p.cap2 : p.cap1,
                 lg_q, p.lg_sub, p.lg_slots, t.mask_hi, A, B, out, out_cap, out_bucket, b.counters};
    if (two && A.lg <= lg_q && B.lg <= lg_q)
        hipLaunchKernelGGL(t.on() ? hash_bucket_kernel<true> : hash_bucket_kernel<false>,
                           dim3(std::min(1u << lg_q, 512u)), dim3(kBucketBlock), 0, w.stream, a);
    else
        hipLaunchKernelGGL(t.on() ? hash_bucket_pieces_kernel<true> : hash_bucket_pieces_kernel<false>,
                           dim3(1u << lg_q), dim3(kBucketBlock), 0, w.stream, a);
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->end(K_BUCKET, 8.0 * (double)(p.C + A.n + B.n), (double)p.C);
}

void launch_hash_small(const HashSmallArgs &a, const HashGens &g, const HashTags &t, PipeWork &w) {
    if (w.prof) w.prof->begin(K_SMALL);
    with_gens(g, [&](auto gens) {
        auto kernel = t.on() ? hash_small_kernel<decltype(gens), true> : hash_small_kernel<decltype(gens), false>;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kPartBlock), 0, w.stream, a, gens, t);
    });
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->end(K_SMALL, 0, 0);
}

}  // namespace cg
