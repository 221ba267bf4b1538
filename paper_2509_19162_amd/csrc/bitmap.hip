// Growth over rank-space bitmaps: the small-job engine (one workgroup per
// job, one persistent launch for a whole batch) and the bitmask engine (one
// job over the whole device, 3 bits per state). The layer rule is the
// breadth-first one of the definition of growth (paper, section "Reminder
// on Cayley graphs, diameters, growth"): layer d+1 holds the neighbours
// s.g of layer d that no earlier layer holds. A visited bitmap stands for
// "every earlier layer", so no closure under inverses is assumed.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>

#include "bitmap.h"
#include "device_util.h"
#include "expand_device.h"
#include "internal.h"
#include "partition_device.h"
#include "perm_rank.h"

// Device memory of cg_growth_batch_noalloc: every buffer its launch needs
// beyond the caller's inputs and outputs (job table, generator table,
// layer-size and outcome staging, the job-queue tickets, the per-workgroup
// bitmap slots of n = 10 jobs). Each GPU the library runs on holds its
// own copy until the process ends. Host code never uses this name as an
// address: it takes the device address once per device from
// hipGetSymbolAddress (cg::noalloc_scratch).
constexpr size_t kNoAllocScratchBytes = 64ull << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace cg {

namespace {

__host__ __device__ constexpr uint64_t factorial(int n) { return n <= 1 ? 1ull : (uint64_t)n * factorial(n - 1); }

template <int N>
using RankOf = typename std::conditional<(N <= 12), uint32_t, uint64_t>::type;

// Lexicographic rank on the host for any n <= 16 (64-bit).
uint64_t host_rank64(uint64_t key, int n) {
    uint64_t rank = 0;
    uint32_t used = 0;
    for (int i = 0; i < n; ++i) {
        const uint32_t v = (uint32_t)(key >> (4 * (n - 1 - i))) & 15u;
        const uint32_t c = v - (uint32_t)__builtin_popcount(used & ((1u << v) - 1u));
        rank = rank * (uint64_t)(n - i) + c;
        used |= 1u << v;
    }
    return rank;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// ---------------------------------------------------------------------------
// Small-job engine
// ---------------------------------------------------------------------------
struct WgJobDev {
    uint32_t n, k, goff, start_rank;
    uint32_t max_layers, pad;
    uint64_t max_frontier;  // 0 = none
    uint64_t sizes_off;     // first entry of the job's layer sizes
};
struct WgOutDev {
    int32_t status, num_layers;
    uint64_t expanded;
};

constexpr uint32_t kWgLdsN = 9;  // largest n whose bitmaps live in LDS
constexpr int kWgMaxBlock = 1024;
constexpr uint32_t kWgWaves = kWgMaxBlock / kWave;
constexpr uint32_t kWgChunk = 16;  // bitmap words a wave lists at a time
constexpr uint32_t wg_words(int n) { return (uint32_t)((factorial(n) + 31) / 32); }
// n = 10: the bitmap in parts of 2^20 bits.
constexpr uint32_t kWgLgPart = 20, kWgParts = 4;
constexpr uint32_t kWgPartWords = 1u << (kWgLgPart - 5);
static_assert((uint64_t)kWgParts << kWgLgPart >= factorial(10), "parts cover the bitmap");
// Words of a slot: three bitmaps and the lists of neighbours (their length
// is divided among the waves and parts).
constexpr uint64_t kWgSlotBits = (wg_words(10) + 63) / 64 * 64;
constexpr uint64_t kWgListWords = 1u << 20;
constexpr uint64_t kWgListWordsLeast = 16u << 10;
// Slots for `jobs` of n = 10 in `words` words: the fewer, the longer their
// lists and the fewer passes over a job's bitmaps. A round of S_10 growths by
// two random generators and their inverses takes 21 ms times 1 + 28600 /
// (words of a slot's lists), measured from 23000 to 250000 of these. (35 jobs
// 44 ms in two rounds of 29 slots, 25 in one; 46 jobs 48 ms in one round, 43
// in two; a batch with 1365 in 48 MB 846 ms with 32 slots, 669 with 28.)
struct WgSlots {
    uint32_t slots = 0;
    uint64_t words = 0;  // of a slot
};
WgSlots wg_slots(uint64_t words, uint32_t jobs, uint32_t blocks) {
    WgSlots s;
    double least = 0;
    for (uint32_t n = 1; n <= std::min(jobs, blocks); ++n) {
        const uint64_t w = std::min(words / n / 64 * 64, 3 * kWgSlotBits + kWgListWords);
        if (w < 3 * kWgSlotBits + kWgListWordsLeast) break;
        const double t = (double)((jobs + n - 1) / n) * (1.0 + 28600.0 / (double)(w - 3 * kWgSlotBits));
        if (!s.slots || t <= least) {
            least = t;
            s = WgSlots{n, w};
        }
    }
    return s;
}

// ---- states of n <= 8 ------------------------------------------------------------
// A state is eight bytes, entry i in byte i (fewer than eight entries are the
// last ones, above others that stay in place: S_n as a subgroup of S_8, whose
// ranks are the first n!; with the others past them, S_n's ranks lay spread
// over all 40320, and S_5 by LRX took 131 us, now 35). A generator is
// two byte permutes. The rank is that of the first four entries times 24 plus
// the order among the last four: two table lookups, each at the 12-bit number
// made of four 3-bit entries; the way back is two lookups and one byte
// permute.
struct Wg8Tables {
    uint32_t from[2 * 1680];  // first four entries, the other four in order
    uint32_t order[24];       // the 24 orders of four bytes, as selectors
    uint16_t first[4096];     // rank of four entries in S_8, without the factor 24
    uint8_t last[4096];       // order (0..23) among four entries
};
__device__ __forceinline__ uint32_t wg8_index(uint32_t x) {
    return __builtin_amdgcn_udot4(x, 0x00400801u, (x >> 24) << 9, false);
}
__device__ __forceinline__ void wg8_build(Wg8Tables &t) {
    for (uint32_t q = threadIdx.x; q < 1680u; q += blockDim.x) {
        uint64_t left = 0x0706050403020100ull;
        const uint32_t c[4] = {q / 210u, q / 30u % 7u, q / 5u % 6u, q % 5u};
        uint32_t x = 0;
        for (int i = 0; i < 4; ++i) {
            const uint32_t sh = 8u * c[i];
            x |= (uint32_t)((left >> sh) & 255u) << (8 * i);
            left = (left & ((1ull << sh) - 1ull)) | ((left >> 8) & ~((1ull << sh) - 1ull));
        }
        uint32_t o = 0;
        for (int i = 0; i < 3; ++i) {
            uint32_t less = 0;
            for (int j = i + 1; j < 4; ++j) less += ((x >> (8 * j)) & 255u) < ((x >> (8 * i)) & 255u) ? 1u : 0u;
            o = o * (uint32_t)(4 - i) + less;  // radices 4, 3, 2
        }
        t.from[2 * q] = x;
        t.from[2 * q + 1] = (uint32_t)left;
        t.first[wg8_index(x)] = (uint16_t)q;
        t.last[wg8_index(x)] = (uint8_t)o;
    }
    for (uint32_t o = threadIdx.x; o < 24u; o += blockDim.x) {
        uint32_t left = 0x03020100u, x = 0;
        const uint32_t c[4] = {o / 6u, o / 2u % 3u, o % 2u, 0u};
        for (int i = 0; i < 4; ++i) {
            const uint32_t sh = 8u * c[i], keep = (1u << sh) - 1u;
            x |= ((left >> sh) & 255u) << (8 * i);
            left = (left & keep) | ((left >> 8) & ~keep);
        }
        t.order[o] = x;
    }
}

struct Wg8 {
    const Wg8Tables &t;
    const GenSel *sel;  // words 0 and 1: the byte selectors
    struct State {
        uint32_t lo, hi;
    };
    __device__ __forceinline__ State unrank(uint32_t r) const {
        const uint32_t q = r / 24u, o = r - 24u * q;
        return {t.from[2 * q], __builtin_amdgcn_perm(0u, t.from[2 * q + 1], t.order[o])};
    }
    __device__ __forceinline__ uint32_t neighbour(const State &s, uint32_t g) const {
        const uint32_t lo = __builtin_amdgcn_perm(s.hi, s.lo, sel[g].sel[0]);
        const uint32_t hi = __builtin_amdgcn_perm(s.hi, s.lo, sel[g].sel[1]);
        return (uint32_t)t.first[wg8_index(lo)] * 24u + (uint32_t)t.last[wg8_index(hi)];
    }
};

template <int N>
struct WgN {
    const GenSel *sel;  // in device memory
    using State = Nibbles;
    __device__ __forceinline__ State unrank(uint32_t r) const { return split_nibbles(perm_unrank_t<N>(r)); }
    __device__ __forceinline__ uint32_t neighbour(const State &s, uint32_t g) const {
        return nibbles_rank_t<N>(apply_gensel_nibbles(s, uniform_gensel(sel, g)));
    }
};

// The set bits of 16 words (16 c ..) in `list`: bit numbers from the first
// word on. Returns how many.
__device__ __forceinline__ uint32_t wg_list(const uint32_t *words, bool unset, uint32_t c, uint32_t W, uint16_t *list) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t w = c * kWgChunk + (lane >> 2);
    uint32_t x = 0;
    if (w < W) x = unset ? ~words[w] : words[w];
    x = (x >> (8u * (lane & 3u))) & 255u;
    uint32_t n = 0;
#pragma unroll
    for (uint32_t b = 0; b < 8; ++b) {
        const bool on = (x >> b) & 1u;
        const uint64_t m = __ballot(on);
        if (on) list[n + mask_rank(m)] = (uint16_t)(lane << 3 | b);
        n += (uint32_t)__popcll(m);
    }
    return n;
}
__device__ __forceinline__ void wg_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// The unseen states of chunk c that have a seen predecessor (under the
// inverse generators, after the k generators in the codec's table): their
// bits in `fresh`, 16 words of the wave's own, zero before.
template <class C>
__device__ __forceinline__ void wg_pull(const C &codec, uint32_t k, const uint32_t *vis, uint32_t c, uint32_t W,
                                        uint16_t *list, uint32_t *fresh) {
    const uint32_t n = wg_list(vis, true, c, W, list);
    wg_wave_sync();
    for (uint32_t i = threadIdx.x & (kWave - 1); i < n; i += kWave) {
        const uint32_t bit = list[i];
        const typename C::State s = codec.unrank(c * (kWgChunk * 32u) + bit);
        for (uint32_t g = k; g < 2 * k; ++g) {
            const uint32_t q = codec.neighbour(s, g);
            if ((vis[q >> 5] >> (q & 31u)) & 1u) {
                atomicOr(&fresh[bit >> 5], 1u << (bit & 31u));
                break;
            }
        }
    }
    wg_wave_sync();
}

// What a growth keeps between its layers, and the stop rules.
struct WgLayers {
    uint64_t F = 1, before = 0, expanded = 0, seen = 1;
    uint32_t layers = 1;
    int status = CG_OK;
    __device__ __forceinline__ bool done(const WgJobDev &J) {
        if (J.k == 0) return true;
        if ((J.max_frontier && F > J.max_frontier) || layers >= J.max_layers) {
            status = CG_TRUNCATED;
            return true;
        }
        return false;
    }
    // the next layer has n1 states; false: none
    __device__ __forceinline__ bool next(uint32_t n1, uint64_t *sizes) {
        expanded += F;
        if (n1 == 0) return false;
        if (threadIdx.x == 0) sizes[layers] = n1;
        ++layers;
        before = F;
        F = n1;
        seen += n1;
        return true;
    }
    __device__ __forceinline__ void store(WgOutDev *out) const {
        if (threadIdx.x == 0) {
            out->status = status;
            out->num_layers = (int32_t)layers;
            out->expanded = expanded;
        }
    }
};

// One job with its bitmaps in LDS. A layer's states are the set bits of
// `cur`; a wave lists those of 16 words at a time, so that its lanes take
// one state each however the bits lie. Either every state of the layer forms
// its neighbours, and those not seen are set in `nxt`; or, when few states
// are left, every unseen state looks for a seen predecessor and is set in
// `nxt` at the first (the wave owns its word). Bits of no state, in the last
// word, are marked as seen.
// A job alone is bound by what its one CU issues: S_8 by three random
// permutations and their inverses (10 layers, 242,000 neighbours) is 94 us,
// VALU busy for 0.52 of the CU's cycles, LDS for 0.37 (39% of that in
// conflicts); the call takes 154 us, and 440 when each lane looped over a
// word's bits and computed ranks. A small layer is its passes and barriers,
// 10 us (S_8 Coxeter, 29 layers: 300 us). 1024 growths of S_9 take 6.9 ms.
template <class C>
__device__ __forceinline__ void wg_run(const WgJobDev &J, const C &codec, uint32_t states, uint32_t *vis, uint32_t *cur,
                                       uint32_t *nxt, uint16_t *list, uint32_t *fresh, uint64_t *__restrict__ sizes,
                                       WgOutDev *__restrict__ out, uint32_t *s_acc) {
    const uint32_t tid = threadIdx.x, nt = blockDim.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint32_t waves = nt / kWave, W = (states + 31u) / 32u;
    const uint32_t k = J.k;
    for (uint32_t w = tid; w < W; w += nt) {
        vis[w] = 0u;
        cur[w] = 0u;
        nxt[w] = 0u;
    }
    if (tid == 0) *s_acc = 0;
    if (lane < kWgChunk) fresh[lane] = 0;
    __syncthreads();
    if (tid == 0) {
        const uint32_t r = J.start_rank;
        if (states % 32u) vis[W - 1] = ~0u << (states % 32u);
        vis[r >> 5] |= 1u << (r & 31u);
        cur[r >> 5] = 1u << (r & 31u);
        sizes[0] = 1;
    }
    __syncthreads();
    WgLayers L;
    while (!L.done(J)) {
        const bool pull = pull_is_less(states - L.seen, L.F, L.before, k);
        for (uint32_t c = wave; c * kWgChunk < W; c += waves) {
            if (pull) {
                wg_pull(codec, k, vis, c, W, list, fresh);
                if (lane < kWgChunk) {
                    const uint32_t x = fresh[lane];
                    if (x) {
                        nxt[c * kWgChunk + lane] = x;
                        fresh[lane] = 0;
                    }
                }
                continue;
            }
            const uint32_t n = wg_list(cur, false, c, W, list);
            if (!n) continue;
            wg_wave_sync();
            for (uint32_t i = lane; i < n; i += kWave) {
                const typename C::State s = codec.unrank(c * (kWgChunk * 32u) + list[i]);
                for (uint32_t g = 0; g < k; ++g) {
                    const uint32_t q = codec.neighbour(s, g), m = 1u << (q & 31u);
                    if (!(vis[q >> 5] & m)) atomicOr(&nxt[q >> 5], m);
                }
            }
            wg_wave_sync();
        }
        __syncthreads();
        // fold: visited |= next, count it, clear the expanded layer
        uint32_t cnt = 0;
        for (uint32_t w = tid; w < W; w += nt) {
            const uint32_t x = nxt[w];
            if (x) {
                vis[w] |= x;
                cnt += (uint32_t)__popc(x);
            }
            cur[w] = 0u;
        }
        cnt = wave_sum(cnt);
        if (lane == 0 && cnt) atomicAdd(s_acc, cnt);
        __syncthreads();
        const uint32_t n1 = *s_acc;
        uint32_t *t = cur;
        cur = nxt;
        nxt = t;
        if (!L.next(n1, sizes)) break;
        __syncthreads();  // every thread has read s_acc before it is reset
        if (tid == 0) *s_acc = 0;
    }
    L.store(out);
}

// One job of n = 10: its bitmaps (454 KB each) lie in device memory, where
// tests and ORs at random addresses run at 53 and 27 G/s for the whole chip.
// So neighbours are not tested one by one: each wave appends them to four
// lists of its own, one per part of the bitmap, in order (16-lane pieces of
// whole lines); then, part by part, the workgroup ORs its lists into a part
// in LDS, takes away what was seen and writes the next layer's words. A list
// that is full ends the round of its wave; the others end theirs likewise,
// the lists are applied and the waves go on where they were. Late in a growth
// the unseen states look for a seen predecessor in the bitmap in memory; such
// a test weighs four neighbours here.
// A batch of 4096 jobs (1365 of n = 10, four or more generators): this launch
// 75 ms, 222 ms with tests and ORs in the bitmaps in memory; bound by the
// instructions that form the neighbours' ranks.
// A layer goes over whole bitmaps then, 285 us in a job alone on the chip
// however few its states are. So until a layer has more than kWgThin
// neighbours its states are two lists in the LDS of the part: a wave maps 64
// of them under one generator, and a neighbour is claimed in the visited
// bitmap. (One directed generator of order 30: 2.8 us a layer; LRX up to a
// layer of 4000 states 0.10 ms, 3.84 over bitmaps, 1.33 with tests in memory.)
constexpr uint32_t kWgSpan = 8;                            // words listed at a time
constexpr uint32_t kWgQueue = kWgSpan * 32 + kWave;        // states a wave holds
constexpr uint32_t kWgThin = kWgPartWords / 2;             // neighbours of a thin layer: a list's room
template <class C>
__device__ __forceinline__ void wg_run_parts(const WgJobDev &J, const C &codec, uint32_t *vis, uint32_t *cur,
                                             uint32_t *nxt, uint32_t *lists, uint32_t cap, uint32_t *part,
                                             uint32_t *queue, uint32_t *fresh, uint64_t *__restrict__ sizes,
                                             WgOutDev *__restrict__ out, uint32_t *s_acc, uint32_t *s_more) {
    constexpr uint32_t W = wg_words(10), kSpans = kWave / kWgSpan;
    static_assert(W % 4 == 0, "bitmaps of whole uint4");
    const uint32_t tid = threadIdx.x, nt = blockDim.x, lane = tid & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave)), waves = nt / kWave;
    const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)J.k);
    uint32_t *const mine = lists + (uint64_t)wave * kWgParts * cap;
    for (uint32_t w = tid; w < W; w += nt) {
        vis[w] = 0u;
        cur[w] = 0u;
    }
    if (tid == 0) *s_acc = *s_more = 0;
    if (lane < kWgChunk) fresh[lane] = 0;
    __syncthreads();
    uint32_t *from = part, *to = part + kWgThin;  // states of a thin layer and of the next
    if (tid == 0) {
        const uint32_t r = J.start_rank;
        vis[r >> 5] = 1u << (r & 31u);
        from[0] = r;
        sizes[0] = 1;
    }
    __syncthreads();
    WgLayers L;
    bool thin = true;
    while (!L.done(J)) {
        if (thin && L.F * k <= kWgThin) {
            const uint32_t F = (uint32_t)L.F, items = (F + kWave - 1) / kWave * k;
            for (uint32_t it = wave; it < items; it += waves) {
                const uint32_t c = it / k, i = c * kWave + lane;
                const typename C::State s = codec.unrank(from[i < F ? i : 0u]);
                const uint32_t q = codec.neighbour(s, it - c * k), m = 1u << (q & 31u);
                // (a word read from a stale line costs an atomic, no more)
                bool won = i < F && !(vis[q >> 5] & m);
                if (won) won = !(atomicOr(&vis[q >> 5], m) & m);
                const uint64_t b = __ballot(won);
                if (!b) continue;
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(s_acc, (uint32_t)__popcll(b));
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + mask_rank(b);
                if (won) to[at] = q;
            }
            __syncthreads();
            const uint32_t n1 = *s_acc;
            uint32_t *t = from;
            from = to;
            to = t;
            if (!L.next(n1, sizes)) break;
            __syncthreads();  // every thread has read s_acc before it is reset
            if (tid == 0) *s_acc = 0;
            __syncthreads();
            continue;
        }
        if (thin) {
            // the layer's states as bits of `cur`; the part is empty again
            thin = false;
            for (uint32_t i = tid; i < (uint32_t)L.F; i += nt) atomicOr(&cur[from[i] >> 5], 1u << (from[i] & 31u));
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // no line of the bitmaps from before the atomics
            for (uint32_t w = tid; w < kWgPartWords; w += nt) part[w] = 0u;
            __syncthreads();
        }
        uint32_t cnt = 0;
        if (pull_is_less(factorial(10) - L.seen, L.F, L.before, k, 4.0)) {
            for (uint32_t c = wave; c * kWgChunk < W; c += waves) {
                wg_pull(codec, k, vis, c, W, (uint16_t *)queue, fresh);
                if (lane < kWgChunk && c * kWgChunk + lane < W) {
                    nxt[c * kWgChunk + lane] = fresh[lane];
                    fresh[lane] = 0;
                }
            }
            __syncthreads();
            for (uint32_t w = tid; w < W; w += nt) {
                const uint32_t x = nxt[w];
                if (x) {
                    vis[w] |= x;
                    cnt += (uint32_t)__popc(x);
                }
            }
        } else {
            // where the wave is: its span of the 64 words of which a lane
            // holds one, the states in its queue, and the next generator
            uint32_t block = wave, span = kSpans, held = 0, g = 0, x = 0;
            uint64_t some = 0;  // lanes with states left
            for (bool first = true;; first = false) {
                uint32_t fill[kWgParts] = {0, 0, 0, 0};
                bool full = false;
                while (!full) {
                    if (held < kWave && g == 0) {
                        if (span == kSpans) {
                            if (block * kWave < W) {
                                const uint32_t w = block * kWave + lane;
                                x = w < W ? cur[w] : 0u;
                                some = __ballot(x != 0);
                                block += waves;
                                span = 0;
                                continue;
                            }
                        } else {
                            if ((some >> (kWgSpan * span)) & ((1u << kWgSpan) - 1u)) {
                                // four bits of a word per lane
                                const uint32_t from = span * kWgSpan + lane / 8u;
                                const uint32_t y = __shfl(x, (int)from, kWave) >> (4u * (lane & 7u));
                                const uint32_t r0 = ((block - waves) * kWave + from) * 32u + 4u * (lane & 7u);
#pragma unroll
                                for (uint32_t b = 0; b < 4; ++b) {
                                    const bool on = (y >> b) & 1u;
                                    const uint64_t m = __ballot(on);
                                    if (on) queue[held + mask_rank(m)] = r0 + b;
                                    held += (uint32_t)__popcll(m);
                                }
                                wg_wave_sync();
                            }
                            ++span;
                            continue;
                        }
                        if (held == 0) break;
                    }
                    const uint32_t take = held < kWave ? held : (uint32_t)kWave;
                    const bool on = lane < take;
                    const uint64_t in = __ballot(on);
                    const typename C::State s = codec.unrank(queue[held - take + (on ? lane : 0u)]);
                    for (; g < k; ++g) {
                        if (max(max(fill[0], fill[1]), max(fill[2], fill[3])) + kWave > cap) {
                            full = true;
                            break;
                        }
                        const uint32_t q = codec.neighbour(s, g), d = q >> kWgLgPart;
                        const uint64_t b0 = __ballot(d & 1u), b1 = __ballot(d & 2u);
                        const uint64_t m[kWgParts] = {in & ~b1 & ~b0, in & ~b1 & b0, in & b1 & ~b0, in & b1 & b0};
                        uint32_t at = 0;
#pragma unroll
                        for (uint32_t p = 0; p < kWgParts; ++p) {
                            const uint32_t pos = __builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(m[p] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[p], fill[p]));
                            at = d == p ? p * cap + pos : at;
                            fill[p] += (uint32_t)__popcll(m[p]);
                        }
                        if (on) mine[at] = q & ((1u << kWgLgPart) - 1u);
                    }
                    if (!full) {
                        held -= take;
                        g = 0;
                    }
                }
                if (full && lane == 0) *s_more = 1;
                __syncthreads();
                const bool more = *s_more != 0;
#pragma unroll
                for (uint32_t p = 0; p < kWgParts; ++p) {
                    const uint32_t *const in = mine + (uint64_t)p * cap;
                    for (uint32_t i = 4u * lane; i < fill[p]; i += 4u * kWave) {
                        const uint4 v = *reinterpret_cast<const uint4 *>(in + i);
                        const uint32_t q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j)
                            if (i + j < fill[p]) atomicOr(&part[q[j] >> 5], 1u << (q[j] & 31u));
                    }
                    __syncthreads();
                    if (tid == 0) *s_more = 0;  // every thread has read it
                    constexpr uint32_t kAll = kWgPartWords / 4;
                    const uint32_t n4 = min(kAll, W / 4 - p * kAll);
                    uint4 *const pt = reinterpret_cast<uint4 *>(part);
                    uint4 *const vs = reinterpret_cast<uint4 *>(vis) + p * kAll;
                    uint4 *const nx = reinterpret_cast<uint4 *>(nxt) + p * kAll;
                    for (uint32_t i = tid; i < n4; i += nt) {
                        uint4 f = pt[i];
                        const bool any = (f.x | f.y | f.z | f.w) != 0;
                        if (any) {
                            uint4 v = vs[i];
                            f = make_uint4(f.x & ~v.x, f.y & ~v.y, f.z & ~v.z, f.w & ~v.w);
                            cnt += (uint32_t)(__popc(f.x) + __popc(f.y) + __popc(f.z) + __popc(f.w));
                            pt[i] = make_uint4(0, 0, 0, 0);
                            vs[i] = make_uint4(v.x | f.x, v.y | f.y, v.z | f.z, v.w | f.w);
                            if (!first) {
                                v = nx[i];
                                f = make_uint4(v.x | f.x, v.y | f.y, v.z | f.z, v.w | f.w);
                            }
                        }
                        if (first || any) nx[i] = f;
                    }
                    __syncthreads();
                }
                if (!more) break;
            }
        }
        cnt = wave_sum(cnt);
        if (lane == 0 && cnt) atomicAdd(s_acc, cnt);
        __syncthreads();
        const uint32_t n1 = *s_acc;
        uint32_t *t = cur;
        cur = nxt;
        nxt = t;
        if (!L.next(n1, sizes)) break;
        __syncthreads();  // every thread has read s_acc before it is reset
        if (tid == 0) *s_acc = 0;
    }
    L.store(out);
}

// The jobs of a launch, in order: n = 10 (bitmaps in device slots), n = 9
// (bitmaps in LDS, one workgroup per CU), n <= 8 (LDS, two per CU).
struct WgLaunch {
    const WgJobDev *jobs;
    uint32_t n10, n9, njobs;
    uint32_t slot_blocks;  // workgroups that own a slot
    const GenSel *gtab;
    uint64_t *sizes;
    WgOutDev *outs;
    uint32_t *ticket;      // three queues
    uint32_t *gbits;       // slots of slot_words words
    uint64_t slot_words;
};

// A persistent launch: each workgroup takes the next job from a queue (jobs
// are ordered by decreasing size within their range) and runs it to
// completion. ticket[0] hands the jobs of n = 10 to the workgroups that own a
// slot, ticket[1] those of n = 9, ticket[2] the others. kBig: the launch with
// the LDS of a whole CU, which takes from all three; else from the last only.
template <bool kBig>
__global__ __launch_bounds__(kWgMaxBlock) __attribute__((amdgpu_waves_per_eu(kBig ? 4 : 8))) void wg_growth_kernel(
    WgLaunch a) {
    struct Small {
        uint32_t bits[3 * wg_words(8)];
        Wg8Tables tables;
        GenSel sel[2 * kBitmapMaxK];
    };
    constexpr uint32_t kBytes = kBig ? 3 * 4 * wg_words(9) : (uint32_t)sizeof(Small);
    static_assert(kBytes >= sizeof(Small) && (!kBig || kBytes >= 4 * kWgPartWords), "one area for every range");
    __shared__ __align__(16) unsigned char s_area[kBytes];
    __shared__ __align__(16) uint32_t s_list[kWgWaves][kBig ? kWgQueue : kWgChunk * 16];
    __shared__ uint32_t s_fresh[kWgWaves][kWgChunk];
    __shared__ uint32_t s_acc, s_more, s_job;
    const uint32_t wave = threadIdx.x / kWave;
    uint32_t *const queue = s_list[wave], *const fresh = s_fresh[wave];
    uint16_t *const list = reinterpret_cast<uint16_t *>(queue);
    Small &sm = *reinterpret_cast<Small *>(s_area);
    bool built = false;
    const bool has_slot = kBig && a.gbits && blockIdx.x < a.slot_blocks;
    for (uint32_t q = kBig ? (has_slot ? 0u : 1u) : 2u; q < 3u; ++q) {
        const uint32_t lo = q == 0 ? 0u : (q == 1 ? a.n10 : a.n10 + a.n9);
        const uint32_t hi = q == 0 ? a.n10 : (q == 1 ? a.n10 + a.n9 : a.njobs);
        for (;;) {
            if (threadIdx.x == 0) s_job = atomicAdd(a.ticket + q, 1u);
            __syncthreads();
            const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_job);
            __syncthreads();
            if (t >= hi - lo) break;
            const uint32_t j = lo + t;
            const WgJobDev J = a.jobs[j];
            const GenSel *gens = a.gtab + (uint32_t)__builtin_amdgcn_readfirstlane((int)J.goff);
            uint64_t *sz = a.sizes + J.sizes_off;
            WgOutDev *out = a.outs + j;
            if (q == 2) {
                constexpr uint32_t W = wg_words(8);
                if (!built) wg8_build(sm.tables);
                built = true;
                for (uint32_t i = threadIdx.x; i < 2 * J.k * 8u; i += blockDim.x)
                    (&sm.sel[0].sel[0])[i] = (&gens[0].sel[0])[i];
                uint32_t states = 1;
                for (uint32_t i = 2; i <= J.n; ++i) states *= i;
                wg_run(J, Wg8{sm.tables, sm.sel}, states, sm.bits, sm.bits + W, sm.bits + 2 * W, list, fresh, sz, out,
                       &s_acc);
            } else if constexpr (kBig) {
                uint32_t *bits = reinterpret_cast<uint32_t *>(s_area);
                if (q == 1) {
                    constexpr uint32_t W = wg_words(9);
                    wg_run(J, WgN<9>{gens}, (uint32_t)factorial(9), bits, bits + W, bits + 2 * W, list, fresh, sz, out,
                           &s_acc);
                } else {
                    uint32_t *slot = a.gbits + (uint64_t)blockIdx.x * a.slot_words;
                    const uint32_t cap = (uint32_t)(a.slot_words - 3 * kWgSlotBits) / (kWgParts * (blockDim.x / kWave));
                    wg_run_parts(J, WgN<10>{gens}, slot, slot + kWgSlotBits, slot + 2 * kWgSlotBits,
                                 slot + 3 * kWgSlotBits, cap & ~3u, bits, queue, fresh, sz, out, &s_acc, &s_more);
                }
            }
            __syncthreads();
        }
    }
}

__global__ void clear_u32_kernel(uint32_t *p, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------
// Bitmask engine (one job, whole device)
// ---------------------------------------------------------------------------
constexpr uint32_t kChunkWords = 1024;  // bitmap words per summary bit
constexpr int kBmBlock = 256;

template <int N>
__global__ __launch_bounds__(kBmBlock) void bm_expand_kernel(const uint32_t *__restrict__ cur,
                                                             const uint32_t *__restrict__ scur,
                                                             const uint32_t *__restrict__ vis, uint32_t *nxt,
                                                             uint32_t *snxt, uint64_t W, uint64_t nchunks,
                                                             const GenSel *__restrict__ gsel, int k,
                                                             const uint32_t *go) {
    using R = RankOf<N>;
    __shared__ GenSel s_sel[kBitmapMaxK];
    if (go && !*go) return;  // the lists held everything
    for (int i = threadIdx.x; i < k * 8; i += kBmBlock) (&s_sel[0].sel[0])[i] = (&gsel[0].sel[0])[i];
    __syncthreads();
    for (uint64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        if (!((scur[c >> 5] >> (c & 31u)) & 1u)) continue;  // no state of layer d here
        const uint64_t w_end = (c + 1) * kChunkWords < W ? (c + 1) * kChunkWords : W;
        for (uint64_t w = c * kChunkWords + threadIdx.x; w < w_end; w += kBmBlock) {
            uint32_t bits = cur[w];
            while (bits) {
                const uint32_t b = (uint32_t)__builtin_ctz(bits);
                bits &= bits - 1u;
                const Nibbles s = split_nibbles(perm_unrank_t<N, R>((R)(w * 32u + b)));
                for (int g = 0; g < k; ++g) {
                    const uint64_t q = (uint64_t)nibbles_rank_t<N, R>(apply_gensel_nibbles(s, s_sel[g]));
                    const uint64_t qw = q >> 5;
                    const uint32_t m = 1u << (uint32_t)(q & 31u);
                    if (vis[qw] & m) continue;
                    if (nxt[qw] & m) continue;  // may read stale: then the atomic below decides
                    const uint32_t old = atomicOr(&nxt[qw], m);
                    if (old == 0u) {  // first bit of this word in layer d+1: mark its chunk
                        const uint64_t qc = qw / kChunkWords;
                        atomicOr(&snxt[qc >> 5], 1u << (uint32_t)(qc & 31u));
                    }
                }
            }
        }
    }
}

// ---- large layers through lists --------------------------------------------------
// A test at a random address of the bitmaps costs 19 ps of the whole chip's
// time (53 G/s), the atomic of a new state 37. For n = 11..13 a large layer
// goes through lists instead: a piece of its neighbours is split by segment
// of the bitmap (bm_part_kernel: 512 digits, each the segments digit,
// digit + 512, ..., so that crowded ranks spread), then a workgroup per
// segment ORs its words into LDS, takes away what was seen and adds the rest
// to the next layer (bm_apply_kernel). The workgroups of one digit run side
// by side on one XCD: its words, read by each of them, come from that L2.
// States next to each other share their first entries, and so do their
// neighbours under one generator: hundreds of words of one digit at a time,
// so the workgroups share the digits' parts (with parts of their own, of
// 2000 words, one in ten overran).
// OR may be repeated, so a piece whose lists overran goes through
// bm_expand_kernel as if nothing had happened (on S_11, whose bitmaps fit the
// caches, even that is faster: most bits are set by then).
// S_13 by two random generators and their inverses: 617 -> 260 ms, of which
// the split takes 60% (8.9 ps a neighbour: ranks, ring slots and barriers)
// and the ORs 30% (4.4).
constexpr uint32_t kBmLgDigits = 9;
constexpr uint32_t kBmPartBlocks = 256;
constexpr uint32_t kBmSets = 2;  // cursors of a digit: workgroups take turns
constexpr uint32_t kBmCursors = (kBmSets * PartShared<uint32_t>::kStep) << kBmLgDigits;
template <int N>
struct BmSeg {
    static constexpr uint32_t kLg = N >= 12 ? 20 : 17;  // bits of a segment
    static constexpr uint32_t kSegs = (uint32_t)((factorial(N) + (1ull << kLg) - 1) >> kLg);
    static constexpr uint32_t kSubs = (kSegs + (1u << kBmLgDigits) - 1) >> kBmLgDigits;  // per digit
    static_assert((uint64_t)kSubs << kLg <= 1ull << 32, "words of 32 bits");
};
constexpr uint32_t kBmSpan = 4, kBmTake = 2 * kWave;  // words listed at a time; states a wave takes

// Piece `piece` of `pieces` of the layer: every pieces-th block of 64 words.
// A round forms eight neighbours per thread, of two states and four
// generators; a wave queues states so that its rounds are full.
template <int N>
__global__ __launch_bounds__(kPartBlock) void bm_part_kernel(const uint32_t *__restrict__ cur, uint64_t W,
                                                             uint32_t piece, uint32_t pieces,
                                                             const GenSel *__restrict__ sel, uint32_t k,
                                                             PartShared<uint32_t> o) {
    using R = RankOf<N>;
    constexpr uint32_t kWaves = kPartBlock / kWave, kLg = BmSeg<N>::kLg, kSpans = kWave / kBmSpan;
    constexpr uint32_t kQueue = kBmTake + kBmSpan * 32;
    __shared__ PartLds<uint32_t> L;
    __shared__ uint32_t s_queue[kWaves][kQueue];
    __shared__ uint32_t s_any[2];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    uint32_t *const queue = s_queue[wave];
    if (threadIdx.x < 2) s_any[threadIdx.x] = 0;
    part_begin(L, 1u << kBmLgDigits);
    o.base += (uint64_t)(blockIdx.x / 8u % kBmSets) * o.cap;
    o.cursor += (blockIdx.x / 8u % kBmSets) * (kBmCursors / kBmSets);
    // block of 64 words number i of this wave
    const uint32_t id = blockIdx.x * kWaves + wave, stride = gridDim.x * kWaves;
    auto word_of = [&](uint32_t i) { return ((uint64_t)((uint64_t)i * stride + id) * pieces + piece) * kWave; };
    uint32_t parity = 0, turn = 0, i = 0, span = kSpans, held = 0, x = 0;
    uint64_t some = 0;
    for (;;) {
        while (held < kBmTake) {
            if (span == kSpans) {
                const uint64_t w0 = word_of(i);
                if (w0 >= W) break;
                x = w0 + lane < W ? cur[w0 + lane] : 0u;
                some = __ballot(x != 0);
                span = 0;
                ++i;
                continue;
            }
            if ((some >> (kBmSpan * span)) & ((1u << kBmSpan) - 1u)) {
                // two bits of a word per lane
                const uint32_t from = span * kBmSpan + lane / 16u;
                const uint32_t y = __shfl(x, (int)from, kWave) >> (2u * (lane & 15u));
                const uint32_t r0 = ((i - 1) * kWave + from) * 32u + 2u * (lane & 15u);
#pragma unroll
                for (uint32_t b = 0; b < 2; ++b) {
                    const bool on = (y >> b) & 1u;
                    const uint64_t m = __ballot(on);
                    if (on) queue[held + mask_rank(m)] = r0 + b;
                    held += (uint32_t)__popcll(m);
                }
                wg_wave_sync();
            }
            ++span;
        }
        if (held && lane == 0) s_any[turn] = 1;
        __syncthreads();
        if (!s_any[turn]) break;
        turn ^= 1u;
        if (threadIdx.x == 0) s_any[turn] = 0;  // read before the last barrier
        const uint32_t take = held < kBmTake ? held : kBmTake;
        held -= take;
        Nibbles s[2];
        uint32_t in = 0;
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j) {
            const uint32_t at = j * kWave + lane;
            const bool on = at < take;
            const uint32_t e = queue[on ? held + at : 0];
            const uint64_t r = on ? word_of(e >> 11) * 32u + (e & 2047u) : 0ull;
            s[j] = split_nibbles(perm_unrank_t<N, R>((R)r));
            if (on) in |= 1u << j;
        }
        for (uint32_t g0 = 0; g0 < k; g0 += 4) {
            uint32_t v[8], dig[8], pend = 0;
#pragma unroll
            for (uint32_t h = 0; h < 4; ++h) {
                const uint32_t g = g0 + h < k ? g0 + h : k - 1;
                if (g0 + h < k) pend |= in << (2 * h);
                const GenSel G = uniform_gensel(sel, g);
#pragma unroll
                for (uint32_t j = 0; j < 2; ++j) {
                    const R q = nibbles_rank_t<N, R>(apply_gensel_nibbles(s[j], G));
                    const uint32_t seg = (uint32_t)(q >> kLg);
                    dig[2 * h + j] = seg & ((1u << kBmLgDigits) - 1u);
                    v[2 * h + j] = (seg >> kBmLgDigits) << kLg | ((uint32_t)q & ((1u << kLg) - 1u));
                }
            }
            part_round(L, v, dig, pend, kBmLgDigits, o, parity);
        }
    }
    part_end(L, kBmLgDigits, o);
}

template <int N>
__global__ __launch_bounds__(kPartBlock) void bm_apply_kernel(const uint32_t *__restrict__ in,
                                                              const uint32_t *__restrict__ cursor, uint32_t cap,
                                                              const uint32_t *__restrict__ vis,
                                                              uint32_t *__restrict__ nxt, uint32_t *snxt, uint64_t W,
                                                              uint32_t *overrun) {
    constexpr uint32_t kLg = BmSeg<N>::kLg, kSubs = BmSeg<N>::kSubs, kWords = 1u << (kLg - 5);
    constexpr uint32_t kRows = 4;  // loads of a lane under way
    static_assert(kWords % kChunkWords == 0 && kChunkWords % 256 == 0, "whole summary bits, a wave in one");
    __shared__ __align__(16) uint32_t s_bits[kWords];
    __shared__ uint32_t s_sum;
    // blocks go to the XCDs in turn
    const uint32_t xcd = blockIdx.x % 8u, at = blockIdx.x / 8u;
    const uint32_t digit = at / kSubs * 8u + xcd, sub = at % kSubs, seg = sub << kBmLgDigits | digit;
    if (seg >= BmSeg<N>::kSegs) return;
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    uint4 *const bits4 = reinterpret_cast<uint4 *>(s_bits);
    for (uint32_t w = tid; w < kWords / 4; w += kPartBlock) bits4[w] = make_uint4(0, 0, 0, 0);
    if (tid == 0) s_sum = 0;
    __syncthreads();
    for (uint32_t set = 0; set < kBmSets; ++set) {
        const uint32_t given = cursor[set * (kBmCursors / kBmSets) + digit * PartShared<uint32_t>::kStep];
        const uint32_t n = min(given, cap) / 4;
        if (given > cap && tid == 0) *overrun = 1;
        const uint4 *const p = reinterpret_cast<const uint4 *>(in + ((uint64_t)digit * kBmSets + set) * cap);
        for (uint32_t b = tid; b < n; b += kRows * kPartBlock) {
            uint4 q[kRows];
#pragma unroll
            for (uint32_t j = 0; j < kRows; ++j)
                q[j] = b + j * kPartBlock < n ? p[b + j * kPartBlock] : make_uint4(~0u, ~0u, ~0u, ~0u);
#pragma unroll
            for (uint32_t j = 0; j < kRows; ++j) {
                const uint32_t x[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u)
                    if (x[u] >> kLg == sub) {  // not of a place that holds no word
                        const uint32_t y = x[u] & ((1u << kLg) - 1u);
                        atomicOr(&s_bits[y >> 5], 1u << (y & 31u));
                    }
            }
        }
    }
    __syncthreads();
    const uint64_t w0 = (uint64_t)seg * kWords;
    const uint32_t n4 = (uint32_t)(min((uint64_t)kWords, W - w0) / 4);
    static_assert(factorial(N) % 128 == 0, "bitmaps of whole uint4");
    const uint4 *const v4 = reinterpret_cast<const uint4 *>(vis + w0);
    uint4 *const x4 = reinterpret_cast<uint4 *>(nxt + w0);
    for (uint32_t i = tid; i < kWords / 4; i += kPartBlock) {
        const uint4 f = bits4[i];
        bool some = false;
        if (i < n4 && (f.x | f.y | f.z | f.w)) {
            const uint4 v = v4[i], x = x4[i];
            const uint4 y = make_uint4(x.x | (f.x & ~v.x), x.y | (f.y & ~v.y), x.z | (f.z & ~v.z), x.w | (f.w & ~v.w));
            some = y.x != x.x || y.y != x.y || y.z != x.z || y.w != x.w;
            if (some) x4[i] = y;
        }
        if (__ballot(some) && lane == 0) atomicOr(&s_sum, 1u << (4 * i / kChunkWords));
    }
    __syncthreads();
    const uint64_t c = w0 / kChunkWords;
    if (tid == 0 && s_sum) atomicOr(&snxt[c >> 5], s_sum << (uint32_t)(c & 31u));
}

// Lists of a layer step: `pieces` launches of at most `per_piece` neighbours.
struct BmLists {
    uint64_t per_piece = 0;  // 0: n has none
    uint32_t cap = 0;        // words of a part (one of kBmSets) of a digit
    uint64_t words() const { return (uint64_t)kBmSets * cap << kBmLgDigits; }
};
BmLists bm_lists(int n, uint32_t k) {
    BmLists l;
    auto set = [&](auto NN) {
        constexpr int N = decltype(NN)::value;
        // about a sixteenth of the states, 1 GiB of words at most
        l.per_piece = std::min<uint64_t>(1ull << 28, std::max<uint64_t>(1ull << 24, factorial(N) / 16));
        const double share = (double)BmSeg<N>::kSubs / (double)BmSeg<N>::kSegs;  // of the fullest digit
        // (workgroups end a part in the middle of a line)
        l.cap = part_cap(1.3 * (double)l.per_piece * share / kBmSets + 32.0 * kBmPartBlocks / kBmSets, k);
    };
    if (n == 11) set(std::integral_constant<int, 11>{});
    if (n == 12) set(std::integral_constant<int, 12>{});
    if (n == 13) set(std::integral_constant<int, 13>{});
    return l;
}
template <class F>
void with_bm_lists_n(int n, F &&f) {
    switch (n) {
        case 11: f(std::integral_constant<int, 11>{}); break;
        case 12: f(std::integral_constant<int, 12>{}); break;
        default: f(std::integral_constant<int, 13>{}); break;
    }
}
// Lists are for generators that scatter. Where g leaves the last entries in
// place, or moves late ones only, the neighbours of states with nearby ranks
// lie in a few lines, and testing them directly takes 3 to 6 ps (S_12 under
// all 66 transpositions 230 ms, through lists 2100; S_13 2.9 s and 7.7),
// where scattered ones take 31 and the lists 9 to 13 (by the rules here 160 ms
// and 1.9 s; star S_13 690 -> 484, pancake 1046 -> 525, LRX 760 to 830 -> 597,
// against direct tests of all). It depends on how near
// the layer's ranks are: lines that 64 of them come to under g, per rank, in
// two places, for one in 1, 4, 16 or 64 ranks in the layer.
constexpr int kBmDensities = 4;
struct BmSpread {
    double at[kBmDensities];
};
constexpr uint32_t kBmSpreadRanks = 64, kBmSpreadPlaces = 2;
constexpr uint32_t kBmSpreadKeys = kBmDensities * kBmSpreadPlaces * kBmSpreadRanks;
// The permutations looked at, the same for every generator.
template <int N>
void bm_spread_keys(uint64_t *key) {
    for (int d = 0; d < kBmDensities; ++d)
        for (uint64_t place = 0; place < kBmSpreadPlaces; ++place) {
            const uint64_t r0 = (factorial(N) / 5 * (2 * place + 1)) / 4096 * 4096;
            for (uint32_t i = 0; i < kBmSpreadRanks; ++i)
                *key++ = perm_unrank_t<N, RankOf<N>>((RankOf<N>)(r0 + ((uint64_t)i << (2 * d))));
        }
}
template <int N>
BmSpread bm_spread(const uint8_t *row, const uint64_t *key) {
    constexpr uint32_t kLgLine = 10;
    BmSpread out;
    for (int d = 0; d < kBmDensities; ++d) {
        uint32_t lines = 0;
        for (uint32_t place = 0; place < kBmSpreadPlaces; ++place) {
            uint64_t line[kBmSpreadRanks];
            for (uint64_t &x : line) {
                uint64_t t = 0;
                for (int j = 0; j < N; ++j) t = t << 4 | ((*key >> (4 * (N - 1 - row[j]))) & 15u);
                ++key;
                x = (uint64_t)perm_rank_t<N, RankOf<N>>(t) >> kLgLine;
            }
            std::sort(line, line + kBmSpreadRanks);
            lines += (uint32_t)(std::unique(line, line + kBmSpreadRanks) - line);
        }
        out.at[d] = (double)lines / (2.0 * kBmSpreadRanks);
    }
    return out;
}
int bm_density(uint64_t F, uint64_t S) { return 2 * F >= S ? 0 : (8 * F >= S ? 1 : (32 * F >= S ? 2 : 3)); }
// From this many lines per neighbour on a generator goes through lists, at 13
// ps. A direct test takes 28 ps per line, and its 95 instructions, with its
// share of the state's 250, more of a wave the fewer of its lanes have a
// state (0.0256 ps each when all have).
double bm_scattered(int density, int k) {
    constexpr double kLanes[kBmDensities] = {1.2, 1.5, 2.5, 4.0};
    return std::max(0.0, (13.0 - (95.0 + 250.0 / k) * 0.0256 * kLanes[density]) / 28.0);
}

// From this many neighbours on a layer goes through lists: below, clearing
// and writing back every segment is more than the tests (at n = 13, 2.5 ms; by
// two random generators and their inverses 8e6 neighbours 3.5 ms and 3.2
// directly, 2.5e7 3.8 and 5.1).
constexpr uint64_t kBmListsMin = 1ull << 23, kBmListsMin13 = 1ull << 24;
uint64_t bm_lists_min(int n) { return n >= 13 ? kBmListsMin13 : kBmListsMin; }
// Early layers crowd near the start state, and late ones at the other end.
// There direct tests are cheap, as neighbours share lines (S_13 Coxeter, 8e5
// to 2e8 states, 82 to 15 ps), and a digit's list overruns (lists 900 to 62
// ps). So a layer goes through lists up to this many times its even share in
// the fullest digit. One segment to a digit (n = 11, 12): lists are faster on
// S_11 up to 3.8 (pancake 320 ps directly, 116 through lists, transpositions
// 46 and 22), slower for reversals at 4.4 (40, 118) and for Coxeter, none of
// whose generators goes far, at 3.7 (136, 200); on S_12 faster up to 2.2 (LRX
// 175, 70), slower for Coxeter at 2.7 (42, 146) and reversals at 2.9 (11, 53).
// A digit of n = 13 holds 12 segments: faster up to 1.43 (LRX 74, 45), slower
// at 1.51 (Coxeter 15, 62) and 1.61 (pancake 19, 28). Where every generator
// takes ranks as near as the layer's to a quarter of a line each or more, no
// neighbours share lines, whatever part of the ranks the orbit lies in: up to
// 3 (S_12 as a subgroup of S_13, at 2.2: 34 to 207 ps, 16 to 133).
constexpr double kBmFar = 0.25, kBmCrowdedMost = 4.0;
double bm_crowded(int n, bool all_far, bool some_far) {
    if (n <= 11) return some_far ? kBmCrowdedMost : 3.5;
    return all_far ? 3.0 : (n == 12 ? 2.4 : 1.45);
}
// From this many states on a layer is worth finding out which generators
// scatter: up to 17 us of host time per generator, and lists save 100 ps and
// more of a neighbour's time in the first layers that take them.
constexpr uint64_t kBmSpreadMin = 1ull << 18;

// The step from the other side, late in a growth: every unseen state looks
// for a seen predecessor (its images under the inverse generators) and is in
// the next layer iff there is one. No atomics: a state's bit is set by the
// wave that owns its word. A wave lists the unseen bits of 16 words at a
// time in LDS, so that its lanes take one state each. Bound by the tests at
// random addresses (53 G/s in 780 MB), of which there are fewer: S_13 by two
// random generators and their inverses 794 -> 617 ms. Sets of even
// permutations reach half of S_n, the other half stays unseen, and the rule
// stays with the expansion.
template <int N>
__global__ __launch_bounds__(kBmBlock) void bm_pull_kernel(const uint32_t *__restrict__ vis,
                                                           uint32_t *__restrict__ nxt, uint32_t *snxt, uint64_t W,
                                                           const GenSel *__restrict__ ginv, int k) {
    using R = RankOf<N>;
    constexpr uint32_t kWords = 16, kWaves = kBmBlock / kWave;
    __shared__ GenSel s_sel[kBitmapMaxK];
    __shared__ uint16_t s_list[kWaves][kWords * 32];
    __shared__ uint32_t s_new[kWaves][kWords];
    for (int i = threadIdx.x; i < k * 8; i += kBmBlock) (&s_sel[0].sel[0])[i] = (&ginv[0].sel[0])[i];
    __syncthreads();
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint16_t *list = s_list[wave];
    uint32_t *fresh = s_new[wave];
    const uint64_t pieces = (W + kWords - 1) / kWords;
    for (uint64_t c = (uint64_t)blockIdx.x * kWaves + wave; c < pieces; c += (uint64_t)gridDim.x * kWaves) {
        const uint64_t w = c * kWords + (lane >> 2);
        uint32_t x = w < W ? ~vis[w] : 0u;
        if (lane < kWords) fresh[lane] = 0;
        x = (x >> (8u * (lane & 3u))) & 255u;
        uint32_t n = 0;
#pragma unroll
        for (uint32_t b = 0; b < 8; ++b) {
            const bool on = (x >> b) & 1u;
            const uint64_t m = __ballot(on);
            if (on) list[n + mask_rank(m)] = (uint16_t)(lane << 3 | b);
            n += (uint32_t)__popcll(m);
        }
        if (!n) continue;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (uint32_t i = lane; i < n; i += kWave) {
            const uint32_t bit = list[i];
            const R r = (R)(c * (kWords * 32)) + (R)bit;
            if ((uint64_t)r >= factorial(N)) continue;  // past the last rank, in the last word
            const Nibbles s = split_nibbles(perm_unrank_t<N, R>(r));
            for (int g = 0; g < k; ++g) {
                const uint64_t q = (uint64_t)nibbles_rank_t<N, R>(apply_gensel_nibbles(s, s_sel[g]));
                if ((vis[q >> 5] >> (uint32_t)(q & 31u)) & 1u) {
                    atomicOr(&fresh[bit >> 5], 1u << (bit & 31u));
                    break;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t f = lane < kWords ? fresh[lane] : 0u;
        if (f) {
            nxt[c * kWords + lane] = f;
            const uint64_t qc = (c * kWords) / kChunkWords;
            atomicOr(&snxt[qc >> 5], 1u << (uint32_t)(qc & 31u));
        }
    }
}

// visited |= next (counted), and the expanded layer is cleared, over the
// chunks that either touches. digits (or null): new states by the digit of
// their segment, of 2^lg bits.
__global__ __launch_bounds__(kBmBlock) void bm_fold_kernel(uint32_t *__restrict__ vis, uint32_t *__restrict__ cur,
                                                           const uint32_t *__restrict__ scur,
                                                           const uint32_t *__restrict__ nxt,
                                                           const uint32_t *__restrict__ snxt, uint64_t W,
                                                           uint64_t nchunks, unsigned long long *count,
                                                           uint32_t *digits, uint32_t lg) {
    __shared__ uint32_t s_acc, s_digit[1u << kBmLgDigits];
    if (threadIdx.x == 0) s_acc = 0;
    if (digits)
        for (uint32_t d = threadIdx.x; d < (1u << kBmLgDigits); d += kBmBlock) s_digit[d] = 0;
    __syncthreads();
    uint32_t cnt = 0;
    for (uint64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const bool in_next = (snxt[c >> 5] >> (c & 31u)) & 1u;
        const bool in_cur = (scur[c >> 5] >> (c & 31u)) & 1u;
        if (!in_next && !in_cur) continue;
        const uint64_t w_end = (c + 1) * kChunkWords < W ? (c + 1) * kChunkWords : W;
        uint32_t here = 0;
        for (uint64_t w = c * kChunkWords + threadIdx.x; w < w_end; w += kBmBlock) {
            if (in_next) {
                const uint32_t x = nxt[w];
                if (x) {
                    vis[w] |= x;
                    here += (uint32_t)__popc(x);
                }
            }
            if (in_cur) cur[w] = 0u;
        }
        cnt += here;
        if (digits && in_next) {
            here = wave_sum(here);
            const uint32_t d = (uint32_t)(c * kChunkWords * 32 >> lg) & ((1u << kBmLgDigits) - 1u);
            if ((threadIdx.x & (kWave - 1)) == 0 && here) atomicAdd(&s_digit[d], here);
        }
    }
    cnt = wave_sum(cnt);
    if ((threadIdx.x & (kWave - 1)) == 0 && cnt) atomicAdd(&s_acc, cnt);
    __syncthreads();
    if (threadIdx.x == 0 && s_acc) atomicAdd(count, (unsigned long long)s_acc);
    if (digits)
        for (uint32_t d = threadIdx.x; d < (1u << kBmLgDigits); d += kBmBlock)
            if (s_digit[d]) atomicAdd(&digits[d], s_digit[d]);
}

__global__ void bm_seed_kernel(uint32_t *vis, uint32_t *cur, uint32_t *scur, uint64_t r,
                               unsigned long long *count) {
    const uint64_t w = r >> 5;
    const uint32_t m = 1u << (uint32_t)(r & 31u);
    vis[w] = m;
    cur[w] = m;
    const uint64_t c = w / kChunkWords;
    scur[c >> 5] = 1u << (uint32_t)(c & 31u);
    count[0] = 0;
}

__global__ void bm_clear_kernel(uint32_t *a, uint64_t na, unsigned long long *count) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < na; i += (uint64_t)gridDim.x * blockDim.x)
        a[i] = 0u;
    if (count && blockIdx.x == 0 && threadIdx.x == 0) *count = 0;
}

template <class F>
void with_bm_n(int n, F &&f) {
    switch (n) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 5: f(std::integral_constant<int, 5>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 7: f(std::integral_constant<int, 7>{}); break;
        case 8: f(std::integral_constant<int, 8>{}); break;
        case 9: f(std::integral_constant<int, 9>{}); break;
        case 10: f(std::integral_constant<int, 10>{}); break;
        case 11: f(std::integral_constant<int, 11>{}); break;
        case 12: f(std::integral_constant<int, 12>{}); break;
        case 13: f(std::integral_constant<int, 13>{}); break;
        default: f(std::integral_constant<int, 14>{}); break;
    }
}

int device_cus() {
    int dev = 0, cus = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    return cus;
}

}  // namespace

bool start_is_permutation(const JobSpec &spec) {
    bool seen[16] = {false};
    for (int i = 0; i < spec.n; ++i) {
        if (spec.start[i] >= spec.n || seen[spec.start[i]]) return false;
        seen[spec.start[i]] = true;
    }
    return true;
}

bool wg_eligible(const JobSpec &spec) {
    return spec.n <= kWgMaxN && spec.k <= kBitmapMaxK && start_is_permutation(spec) && !spec.layers_out &&
           !(spec.flags & CG_KEEP_ALL_LAYERS) && spec.max_layers <= (int)0x7fffffff;
}

// ---------------------------------------------------------------------------
// WgRunner
// ---------------------------------------------------------------------------
WgRunner::WgRunner(hipStream_t s) : stream_(s) {
    for (DevBuf *b : {&jobs_, &gsel_, &outs_, &ws_, &ticket_}) b->stream = s;
}

WgRunner::~WgRunner() {
    if (exec_) (void)hipGraphExecDestroy(exec_);
    if (graph_) (void)hipGraphDestroy(graph_);
    const bool idle = hipStreamSynchronize(stream_) == hipSuccess;
    for (DevBuf *b : {&jobs_, &gsel_, &outs_, &ws_, &ticket_}) b->release();
    give_kit(kit_, idle);
}

namespace {

// Host tables of one small-job launch, jobs in launch order.
struct WgTables {
    std::vector<uint32_t> order;  // launch position -> item index
    std::vector<WgJobDev> jobs;
    std::vector<GenSel> gsel;
    uint64_t sizes_total = 0;     // layer-size entries of all jobs
    uint32_t n10 = 0, n9 = 0;     // jobs of n = 10 (first) and n = 9 (next)
    uint32_t k10 = 0;             // most generators of a job of n = 10
    int n_max = 0;
};

// Selectors of generator g of a job, or of its inverse: up to n = 8 the two
// byte selectors of the eight-byte states, else the nibble selectors.
GenSel wg_gensel(const JobSpec &s, int g, bool inverse) {
    const uint8_t *row = s.gens.data() + (size_t)g * s.n;
    const int low = std::max(0, 8 - s.n);  // entries that stay in place
    uint8_t r[16];
    for (int i = 0; i < 16; ++i) r[i] = (uint8_t)i;
    for (int i = 0; i < s.n; ++i) {
        if (inverse)
            r[low + row[i]] = (uint8_t)(low + i);
        else
            r[low + i] = (uint8_t)(low + row[i]);
    }
    if (s.n > 8) return make_gensel(s.n, r);
    GenSel v{};
    std::memcpy(&v.sel[0], r, 8);
    return v;
}

// Jobs of n = 10 first, then n = 9, then the others; within these the largest
// first (the queue then balances like longest-first). A job records at most
// min(max_layers, orbit) layer sizes: every recorded layer holds at least
// one state of the orbit.
WgTables wg_tables(const std::vector<WgItem> &items) {
    const uint32_t nj = (uint32_t)items.size();
    WgTables T;
    T.order.resize(nj);
    for (uint32_t i = 0; i < nj; ++i) T.order[i] = i;
    auto range = [](int n) { return n > (int)kWgLdsN ? 0 : (n == 9 ? 1 : 2); };
    std::stable_sort(T.order.begin(), T.order.end(), [&](uint32_t a, uint32_t b) {
        const JobSpec &x = *items[a].spec, &y = *items[b].spec;
        if (range(x.n) != range(y.n)) return range(x.n) < range(y.n);
        const double cx = (double)factorial(x.n) * (x.k + 1), cy = (double)factorial(y.n) * (y.k + 1);
        return cx > cy;
    });
    T.jobs.resize(nj);
    for (uint32_t i = 0; i < nj; ++i) {
        const JobSpec &s = *items[T.order[i]].spec;
        if (!wg_eligible(s)) throw Error(CG_E_INVAL, "job not eligible for the small-job engine");
        WgJobDev &d = T.jobs[i];
        d.n = (uint32_t)s.n;
        d.k = (uint32_t)s.k;
        d.goff = (uint32_t)T.gsel.size();
        // up to n = 8 the states are those of S_8 that fix the first 8 - n
        const int m = std::max(s.n, 8), low = m - s.n;
        uint64_t key = 0;
        for (int q = 0; q < m; ++q) key |= (uint64_t)(q < low ? q : low + s.start[q - low]) << (4 * (m - 1 - q));
        d.start_rank = (uint32_t)host_rank64(key, m);
        d.max_layers = (uint32_t)s.max_layers;
        d.pad = 0;
        d.max_frontier = s.max_frontier;
        d.sizes_off = T.sizes_total;
        T.sizes_total += std::min<uint64_t>((uint64_t)s.max_layers, factorial(s.n));
        // the generators, then their inverses
        for (int g = 0; g < 2 * s.k; ++g) T.gsel.push_back(wg_gensel(s, g < s.k ? g : g - s.k, g >= s.k));
        T.n10 += s.n > (int)kWgLdsN;
        if (s.n > (int)kWgLdsN) T.k10 = std::max(T.k10, (uint32_t)s.k);
        T.n9 += s.n == 9;
        T.n_max = std::max(T.n_max, s.n);
    }
    if (T.gsel.empty()) T.gsel.push_back(GenSel{});
    return T;
}

// Copies the launch's outcomes into the callers' results.
void wg_results(std::vector<WgItem> &items, const WgTables &T, const uint64_t *hsz, const WgOutDev *ho, double ms,
                double t_submit, double t_admit, double t_done) {
    for (uint32_t i = 0; i < (uint32_t)T.jobs.size(); ++i) {
        const JobSpec &s = *items[T.order[i]].spec;
        cg_result_t *r = items[T.order[i]].res;
        const WgOutDev &o = ho[i];
        std::memset(r->layer_sizes, 0, sizeof(uint64_t) * (size_t)s.max_layers);
        const int nl = std::max(0, std::min(o.num_layers, s.max_layers));
        std::memcpy(r->layer_sizes, hsz + T.jobs[i].sizes_off, sizeof(uint64_t) * (size_t)nl);
        r->status = o.status;
        r->num_layers = nl;
        r->states_expanded = o.expanded;
        r->candidates = o.expanded * (uint64_t)s.k;
        r->device_ms = ms;
        r->n_kstats = 0;
        r->t_submit = t_submit;
        r->t_admit = t_admit;
        r->t_done = t_done;
    }
}

}  // namespace

// Workgroups of the two launches: every job its own, at most as many as are
// resident at once. The one for n <= 8 is there for the CUs that the other
// leaves free; when it leaves none, it runs those jobs as well, at its end.
struct WgGrid {
    uint32_t big = 0, small = 0;
};
static WgGrid wg_grid(const WgTables &T, int block) {
    const uint32_t cus = (uint32_t)device_cus();
    const uint32_t bigs = T.n10 + T.n9, others = (uint32_t)T.jobs.size() - bigs;
    WgGrid g;
    g.big = std::min(bigs, cus);  // the LDS of a whole CU
    if (others && g.big < cus) {
        int occ = 0;
        CG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, wg_growth_kernel<false>, block, 0));
        g.small = (uint32_t)std::min<uint64_t>(others, (uint64_t)cus * (uint64_t)std::max(occ, 1));
    }
    return g;
}
// Words of a slot where there is memory for all. (One generator makes layers
// of one state, or two.)
uint64_t wg_slot_words(const WgTables &T) { return 3 * kWgSlotBits + (T.k10 > 1 ? kWgListWords : kWgListWordsLeast); }

uint64_t WgRunner::launch_bytes(const std::vector<WgItem> &items, const WgTuning &t) {
    if (items.empty()) return 0;
    const WgTables T = wg_tables(items);
    const uint32_t nj = (uint32_t)items.size();
    const uint64_t slots = std::min(wg_grid(T, t.block).big, T.n10);
    // every buffer as DevBuf rounds it (64 KiB) with its growth slack
    auto r = [](uint64_t b) { return ((uint64_t)(1.5 * (double)b) + (64u << 10) - 1) / (64u << 10) * (64u << 10); };
    return r(sizeof(WgJobDev) * nj) + r(sizeof(GenSel) * T.gsel.size()) +
           r(sizeof(WgOutDev) * nj + sizeof(uint64_t) * T.sizes_total) + r(256) + r(slots * wg_slot_words(T) * sizeof(uint32_t));
}

uint64_t WgRunner::device_bytes() const {
    return jobs_.bytes + gsel_.bytes + outs_.bytes + ws_.bytes + ticket_.bytes;
}

void WgRunner::release() {
    if (exec_) (void)hipGraphExecDestroy(exec_);
    if (graph_) (void)hipGraphDestroy(graph_);
    exec_ = nullptr;
    graph_ = nullptr;
    graph_key_.clear();
    for (DevBuf *b : {&jobs_, &gsel_, &outs_, &ws_, &ticket_}) b->release();
    give_kit(kit_, hipStreamSynchronize(stream_) == hipSuccess);
}

double WgRunner::run(std::vector<WgItem> &items, const WgTuning &t, double t_submit) {
    const uint32_t nj = (uint32_t)items.size();
    if (!nj) return 0.0;
    if (t.block < 64 || t.block > kWgMaxBlock || t.block % kWave) throw Error(CG_E_INVAL, "bad workgroup size");
    // jobs that need a device slot first: only as many workgroups as there
    // are such jobs own one
    const WgTables T = wg_tables(items);
    const uint64_t sizes_total = T.sizes_total;
    const WgGrid grid = wg_grid(T, t.block);

    jobs_.ensure(sizeof(WgJobDev) * nj, 1.25);
    gsel_.ensure(sizeof(GenSel) * T.gsel.size(), 1.25);
    static_assert(sizeof(WgOutDev) % sizeof(uint64_t) == 0, "sizes follow the outcomes");
    const size_t outs_bytes = sizeof(WgOutDev) * nj, back = outs_bytes + sizeof(uint64_t) * sizes_total;
    outs_.ensure(back, 1.25);
    uint64_t *const d_sizes = reinterpret_cast<uint64_t *>(outs_.as<char>() + outs_bytes);
    ticket_.ensure(256);
    // a slot for every workgroup with a job of n = 10, or as many as there is
    // memory for
    WgSlots slots{std::min(grid.big, T.n10), wg_slot_words(T)};
    for (uint64_t words = slots.slots * slots.words; words;) {
        try {
            ws_.ensure(slots.slots * slots.words * sizeof(uint32_t));
            break;
        } catch (const Error &e) {
            if (e.code != CG_E_NOMEM) throw;
            words = words / 4 * 3;
            slots = wg_slots(words, T.n10, grid.big);
            if (!slots.slots) throw;
        }
    }
    CG_HIP(hipMemcpyAsync(jobs_.p, T.jobs.data(), sizeof(WgJobDev) * nj, hipMemcpyHostToDevice, stream_));
    CG_HIP(hipMemcpyAsync(gsel_.p, T.gsel.data(), sizeof(GenSel) * T.gsel.size(), hipMemcpyHostToDevice, stream_));

    uint32_t *gbits = slots.slots ? ws_.as<uint32_t>() : nullptr;
    WgLaunch args{jobs_.as<const WgJobDev>(), T.n10, T.n9, nj, slots.slots, gsel_.as<const GenSel>(),
                  d_sizes, outs_.as<WgOutDev>(), ticket_.as<uint32_t>(), gbits, slots.words};
    const std::vector<uint64_t> key = {(uint64_t)(uintptr_t)jobs_.p,   nj,
                                       (uint64_t)(uintptr_t)gsel_.p,   (uint64_t)(uintptr_t)d_sizes,
                                       (uint64_t)(uintptr_t)outs_.p,   (uint64_t)(uintptr_t)ticket_.p,
                                       (uint64_t)(uintptr_t)gbits,     (uint64_t)t.block,
                                       T.n10,                          T.n9,
                                       slots.slots,                    slots.words,
                                       grid.big,                       grid.small};
    auto enqueue = [&]() {
        hipLaunchKernelGGL(clear_u32_kernel, dim3(1), dim3(64), 0, stream_, ticket_.as<uint32_t>(), 3u);
        if (grid.big) hipLaunchKernelGGL(wg_growth_kernel<true>, dim3(grid.big), dim3(t.block), 0, stream_, args);
        if (grid.small)
            hipLaunchKernelGGL(wg_growth_kernel<false>, dim3(grid.small), dim3(t.block), 0, stream_, args);
    };
    if (key != graph_key_) {
        // the graph is built node by node (no stream capture): a queue
        // reset, then the persistent kernels side by side
        if (exec_) (void)hipGraphExecDestroy(exec_);
        if (graph_) (void)hipGraphDestroy(graph_);
        exec_ = nullptr;
        graph_ = nullptr;
        graph_key_.clear();
        uint32_t *tk = ticket_.as<uint32_t>();
        uint32_t three = 3;
        void *clear_args[] = {&tk, &three};
        void *wg_args[] = {&args};
        auto node = [](void *func, uint32_t grid_x, int block, void **kernel_args) {
            hipKernelNodeParams p{};
            p.func = func;
            p.gridDim = dim3(grid_x);
            p.blockDim = dim3(block);
            p.sharedMemBytes = 0;
            p.kernelParams = kernel_args;
            p.extra = nullptr;
            return p;
        };
        hipGraphNode_t n0 = nullptr, n1 = nullptr;
        bool ok = hipGraphCreate(&graph_, 0) == hipSuccess;
        const hipKernelNodeParams p0 = node(reinterpret_cast<void *>(clear_u32_kernel), 1, 64, clear_args);
        ok = ok && hipGraphAddKernelNode(&n0, graph_, nullptr, 0, &p0) == hipSuccess;
        if (grid.big) {
            const hipKernelNodeParams p =
                node(reinterpret_cast<void *>(wg_growth_kernel<true>), grid.big, t.block, wg_args);
            ok = ok && hipGraphAddKernelNode(&n1, graph_, &n0, 1, &p) == hipSuccess;
        }
        if (grid.small) {
            const hipKernelNodeParams p =
                node(reinterpret_cast<void *>(wg_growth_kernel<false>), grid.small, t.block, wg_args);
            ok = ok && hipGraphAddKernelNode(&n1, graph_, &n0, 1, &p) == hipSuccess;
        }
        ok = ok && hipGraphInstantiate(&exec_, graph_, nullptr, nullptr, 0) == hipSuccess;
        if (ok) {
            graph_key_ = key;
            ++graph_captures_;
        } else {
            (void)hipGetLastError();
            if (exec_) (void)hipGraphExecDestroy(exec_);
            if (graph_) (void)hipGraphDestroy(graph_);
            exec_ = nullptr;
            graph_ = nullptr;
        }
    }
    hipEvent_t e0, e1;
    CG_HIP(hipEventCreate(&e0));
    CG_HIP(hipEventCreate(&e1));
    const double t_admit = now_seconds();
    CG_HIP(hipEventRecord(e0, stream_));
    if (exec_) {
        CG_HIP(hipGraphLaunch(exec_, stream_));
        ++graph_launches_;
    } else {
        enqueue();
        CG_HIP(hipGetLastError());
    }
    CG_HIP(hipEventRecord(e1, stream_));
    // one copy, into pinned memory where that is kept (large batches: their
    // sizes take milliseconds either way)
    std::vector<uint64_t> pageable;
    const char *h;
    if (back <= kMaxKitBytes) {
        if (kit_.bytes < back) {
            give_kit(kit_, true);
            kit_ = take_kit(back, false);
        }
        h = static_cast<const char *>(kit_.host);
    } else {
        pageable.resize(back / sizeof(uint64_t));
        h = reinterpret_cast<const char *>(pageable.data());
    }
    CG_HIP(hipMemcpyAsync(const_cast<char *>(h), outs_.p, back, hipMemcpyDeviceToHost, stream_));
    CG_HIP(hipStreamSynchronize(stream_));
    float ms = 0;
    CG_HIP(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    const double t_done = now_seconds();
    wg_results(items, T, reinterpret_cast<const uint64_t *>(h + outs_bytes), reinterpret_cast<const WgOutDev *>(h), ms,
               t_submit, t_admit, t_done);
    return ms;
}

WgTuning tune_wg(std::vector<WgItem> &sample, WgRunner &r, double *best_ms_out) {
    WgTuning best;
    double best_ms = -1;
    for (int block : {256, 512, 1024}) {
        WgTuning t;
        t.block = block;
        r.run(sample, t, now_seconds());  // first run: graph build, warm caches
        const double ms = r.run(sample, t, now_seconds());
        if (best_ms < 0 || ms < best_ms) {
            best_ms = ms;
            best = t;
        }
    }
    if (best_ms_out) *best_ms_out = best_ms;
    return best;
}

// ---------------------------------------------------------------------------
// Small-job batches without allocation (cg_growth_batch_noalloc)
// ---------------------------------------------------------------------------
namespace {

constexpr size_t na_align(size_t x) { return (x + 255) & ~(size_t)255; }
// layout of the scratch array: three uint32 queue tickets, then what this
// call's jobs need; the slots of n = 10 take the rest
struct NaLayout {
    size_t outs, jobs, gsel, sizes, slots;
};
constexpr NaLayout na_layout(size_t n_jobs, size_t n_gsel, size_t n_sizes) {
    NaLayout l{};
    l.outs = 256;
    l.jobs = na_align(l.outs + sizeof(WgOutDev) * n_jobs);
    l.gsel = na_align(l.jobs + sizeof(WgJobDev) * n_jobs);
    l.sizes = na_align(l.gsel + sizeof(GenSel) * n_gsel);
    l.slots = na_align(l.sizes + sizeof(uint64_t) * n_sizes);
    return l;
}
static_assert(na_layout(kNoAllocMaxJobs, 2 * kNoAllocMaxGens, kNoAllocMaxSizes).slots +
                      16 * (3 * kWgSlotBits + kWgListWordsLeast) * sizeof(uint32_t) <= kNoAllocScratchBytes,
              "room for at least 16 slots of n = 10");

constexpr int kNaMaxDevices = 64;
struct NaDevice {
    std::once_flag once;
    hipError_t err = hipSuccess;
    void *ptr = nullptr;  // the device's address of `scratch`
    std::mutex mu;        // one call at a time per device in this process
};
NaDevice g_na[kNaMaxDevices];

}  // namespace

void *noalloc_scratch(int dev) {
    if (dev < 0 || dev >= kNaMaxDevices) throw Error(CG_E_DEVICE, "device index beyond the no-allocation table");
    NaDevice &d = g_na[dev];
    // once per device, with that device current (the caller's): each GPU
    // holds its own copy of the array at its own address
    std::call_once(d.once, [&] { d.err = hipGetSymbolAddress(&d.ptr, HIP_SYMBOL(scratch)); });
    if (d.err != hipSuccess || !d.ptr)
        throw Error(CG_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(d.err));
    return d.ptr;
}

void run_batch_noalloc(int n_jobs, const cg_job_t *jobs, cg_result_t *results, hipStream_t stream) {
    const double t0 = now_seconds();
    if (n_jobs < 0 || n_jobs > (int)kNoAllocMaxJobs)
        throw Error(CG_E_INVAL, "cg_growth_batch_noalloc takes at most 4096 jobs");
    std::vector<JobSpec> specs;
    specs.reserve((size_t)n_jobs);
    std::vector<WgItem> items;
    std::vector<int> idx;
    for (int i = 0; i < n_jobs; ++i) {
        cg_result_t *r = &results[i];
        if (!r->layer_sizes) {
            r->status = CG_E_INVAL;
            r->num_layers = 0;
            continue;
        }
        try {
            specs.push_back(canonicalize(jobs[i], true));
        } catch (const Error &e) {
            r->status = e.code;
            r->num_layers = 0;
            continue;
        }
        if (!wg_eligible(specs.back())) {
            char buf[160];
            std::snprintf(buf, sizeof buf,
                          "job %d: cg_growth_batch_noalloc needs n <= 10, a permutation start and at most 128 "
                          "generators",
                          i);
            throw Error(CG_E_INVAL, buf);
        }
        idx.push_back(i);
    }
    for (size_t j = 0; j < specs.size(); ++j) items.push_back({&specs[j], &results[idx[j]]});
    if (items.empty()) return;
    const WgTables T = wg_tables(items);
    if (T.gsel.size() > 2 * kNoAllocMaxGens)  // with their inverses
        throw Error(CG_E_INVAL, "cg_growth_batch_noalloc takes at most 32768 distinct generators in all");
    if (T.sizes_total > kNoAllocMaxSizes)
        throw Error(CG_E_INVAL, "cg_growth_batch_noalloc records at most 2^21 layer sizes in all "
                                "(sum over jobs of min(max_layers, n!))");
    const uint32_t nj = (uint32_t)items.size();
    int dev = 0;
    CG_HIP(hipGetDevice(&dev));
    unsigned char *base = static_cast<unsigned char *>(noalloc_scratch(dev));
    std::lock_guard<std::mutex> lk(g_na[dev].mu);

    const NaLayout at = na_layout(nj, T.gsel.size(), T.sizes_total);
    uint32_t *ticket = reinterpret_cast<uint32_t *>(base);
    WgOutDev *outs = reinterpret_cast<WgOutDev *>(base + at.outs);
    WgJobDev *djobs = reinterpret_cast<WgJobDev *>(base + at.jobs);
    GenSel *dgsel = reinterpret_cast<GenSel *>(base + at.gsel);
    uint64_t *dsizes = reinterpret_cast<uint64_t *>(base + at.sizes);
    uint32_t *gbits = T.n10 ? reinterpret_cast<uint32_t *>(base + at.slots) : nullptr;

    // the launch shape of cg_growth_batch for the batch's largest n
    const int block = wg_block(T.n_max);
    const WgGrid grid = wg_grid(T, block);
    // workgroups that own a slot
    WgSlots slots;
    if (gbits) {
        slots = wg_slots((kNoAllocScratchBytes - at.slots) / sizeof(uint32_t), T.n10, grid.big);
        if (!slots.slots || at.slots + slots.slots * slots.words * sizeof(uint32_t) > kNoAllocScratchBytes)
            throw Error(CG_E_DEVICE, "no-allocation slot layout");
    }
    CG_HIP(hipMemcpyAsync(djobs, T.jobs.data(), sizeof(WgJobDev) * nj, hipMemcpyHostToDevice, stream));
    CG_HIP(hipMemcpyAsync(dgsel, T.gsel.data(), sizeof(GenSel) * T.gsel.size(), hipMemcpyHostToDevice, stream));
    // the array keeps the last call's contents: the tickets start at zero
    hipLaunchKernelGGL(clear_u32_kernel, dim3(1), dim3(64), 0, stream, ticket, 3u);
    CG_HIP(hipGetLastError());
    const double t_admit = now_seconds();
    const WgLaunch args{djobs, T.n10, T.n9, nj, slots.slots, dgsel, dsizes, outs, ticket, gbits, slots.words};
    if (grid.big) hipLaunchKernelGGL(wg_growth_kernel<true>, dim3(grid.big), dim3(block), 0, stream, args);
    CG_HIP(hipGetLastError());
    if (grid.small) hipLaunchKernelGGL(wg_growth_kernel<false>, dim3(grid.small), dim3(block), 0, stream, args);
    CG_HIP(hipGetLastError());
    std::vector<uint64_t> hsz(T.sizes_total);
    std::vector<WgOutDev> ho(nj);
    CG_HIP(hipMemcpyAsync(hsz.data(), dsizes, sizeof(uint64_t) * T.sizes_total, hipMemcpyDeviceToHost, stream));
    CG_HIP(hipMemcpyAsync(ho.data(), outs, sizeof(WgOutDev) * nj, hipMemcpyDeviceToHost, stream));
    CG_HIP(hipStreamSynchronize(stream));
    const double t_done = now_seconds();
    // no events (they would be allocated): device_ms is the host-timed span
    // from the launch to the end of the read-back
    wg_results(items, T, hsz.data(), ho.data(), 1e3 * (t_done - t_admit), t0, t_admit, t_done);
}

// ---------------------------------------------------------------------------
// Bitmask engine host loop
// ---------------------------------------------------------------------------
std::string bitmask_unsupported(const JobSpec &spec) {
    if (spec.n > kBitmaskMaxN) return "the bitmask engine covers n <= 14";
    if (!start_is_permutation(spec)) return "the bitmask engine needs a start state that is a permutation";
    if (spec.k > kBitmapMaxK) return "the bitmask engine takes at most 128 generators";
    if (spec.layers_out || (spec.flags & CG_KEEP_ALL_LAYERS)) return "the bitmask engine does not export layers";
    return "";
}

uint64_t bitmask_list_bytes(const JobSpec &spec) {
    const uint64_t k = (uint64_t)spec.k;
    if (spec.max_frontier && spec.max_frontier < bm_lists_min(spec.n) / std::max<uint64_t>(1, k)) return 0;
    const BmLists l = bm_lists(spec.n, (uint32_t)spec.k);
    return l.per_piece ? (l.words() + kBmCursors) * sizeof(uint32_t) : 0;
}

void run_bitmask(const JobSpec &spec, cg_result_t *res, hipStream_t s, HeldBytes *held) {
    const std::string why = bitmask_unsupported(spec);
    if (!why.empty()) throw Error(CG_E_INVAL, why);
    const double t0 = now_seconds();
    const int n = spec.n, k = spec.k;
    uint64_t *sizes = res->layer_sizes;
    std::memset(sizes, 0, sizeof(uint64_t) * (size_t)spec.max_layers);
    sizes[0] = 1;
    res->status = CG_OK;
    res->num_layers = 1;
    res->states_expanded = 0;
    res->candidates = 0;
    res->n_kstats = 0;

    const uint64_t S = factorial(n);
    const uint64_t W = (S + 31) / 32;
    const uint64_t nchunks = (W + kChunkWords - 1) / kChunkWords;
    const uint64_t sw = (nchunks + 31) / 32;
    DevBuf vis, cur, nxt, scur, snxt, gsel, cnt, lists, list_cnt;
    for (DevBuf *b : {&vis, &cur, &nxt, &scur, &snxt, &gsel, &cnt, &lists, &list_cnt}) {
        b->stream = s;
        b->held = held;
    }
    vis.ensure(W * 4);
    cur.ensure(W * 4);
    nxt.ensure(W * 4);
    scur.ensure(sw * 4);
    snxt.ensure(sw * 4);
    // the layer's count, the lists' flag, and states by digit
    constexpr uint32_t kFlagAt = 2, kDigitsAt = 16, kCounts = kDigitsAt + (1u << kBmLgDigits);
    cnt.ensure(kCounts * sizeof(uint32_t));
    // the generators, then the inverses
    std::vector<GenSel> hs(std::max(1, 2 * k));
    std::vector<int> order(k);
    for (int g = 0; g < k; ++g) order[g] = g;
    auto upload = [&]() {
        for (int g = 0; g < k; ++g) {
            const uint8_t *row = spec.gens.data() + (size_t)order[g] * n;
            uint8_t inv[16] = {0};
            for (int i = 0; i < n; ++i) inv[row[i]] = (uint8_t)i;
            hs[g] = make_gensel(n, row);
            hs[k + g] = make_gensel(n, inv);
        }
        CG_HIP(hipMemcpyAsync(gsel.p, hs.data(), sizeof(GenSel) * hs.size(), hipMemcpyHostToDevice, s));
    };
    gsel.ensure(sizeof(GenSel) * hs.size());
    upload();
    // how many generators go through lists, by the layer's density; these
    // come first then (nothing is under way between two layers)
    int scattered[kBmDensities] = {0};
    bool looked = false, all_far[kBmDensities] = {false}, some_far[kBmDensities] = {false};
    double crowd = 1e9;  // the fullest digit of the layer, in even shares
    auto look_for_scattered = [&]() {
        looked = true;
        std::vector<BmSpread> spread(k, BmSpread{});
        with_bm_lists_n(n, [&](auto NN) {
            constexpr int N = decltype(NN)::value;
            uint64_t keys[kBmSpreadKeys];
            bm_spread_keys<N>(keys);
            for (int g = 0; g < k; ++g) spread[g] = bm_spread<N>(spec.gens.data() + (size_t)g * n, keys);
        });
        auto sum = [&](int g) { return spread[g].at[0] + spread[g].at[1] + spread[g].at[2] + spread[g].at[3]; };
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return sum(a) > sum(b); });
        for (int d = 0; d < kBmDensities; ++d) {
            for (int g = 0; g < k; ++g) scattered[d] += spread[g].at[d] >= bm_scattered(d, k);
            scattered[d] = std::min(k, (scattered[d] + 3) / 4 * 4);  // (a round takes four)
            auto far = [&](const BmSpread &x) { return x.at[d] >= kBmFar; };
            all_far[d] = std::all_of(spread.begin(), spread.end(), far);
            some_far[d] = std::any_of(spread.begin(), spread.end(), far);
        }
        upload();
    };
    CG_HIP(hipMemsetAsync(vis.p, 0, W * 4, s));
    CG_HIP(hipMemsetAsync(cur.p, 0, W * 4, s));
    CG_HIP(hipMemsetAsync(nxt.p, 0, W * 4, s));
    CG_HIP(hipMemsetAsync(scur.p, 0, sw * 4, s));
    CG_HIP(hipMemsetAsync(snxt.p, 0, sw * 4, s));
    uint64_t key0 = 0;
    for (int q = 0; q < n; ++q) key0 |= (uint64_t)spec.start[q] << (4 * (n - 1 - q));
    hipLaunchKernelGGL(bm_seed_kernel, dim3(1), dim3(1), 0, s, vis.as<uint32_t>(), cur.as<uint32_t>(),
                       scur.as<uint32_t>(), host_rank64(key0, n), cnt.as<unsigned long long>());
    CG_HIP(hipGetLastError());
    hipLaunchKernelGGL(bm_clear_kernel, dim3(1), dim3(256), 0, s, cnt.as<uint32_t>() + kFlagAt,
                       (uint64_t)(kCounts - kFlagAt), (unsigned long long *)nullptr);
    CG_HIP(hipGetLastError());

    hipEvent_t e0, e1;
    CG_HIP(hipEventCreate(&e0));
    CG_HIP(hipEventCreate(&e1));
    CG_HIP(hipEventRecord(e0, s));
    const uint32_t grid = (uint32_t)std::min<uint64_t>(nchunks, (uint64_t)device_cus() * 16);
    HostKit kit = take_kit(kCounts * sizeof(uint32_t), false);
    const uint32_t *const host_cnt = static_cast<const uint32_t *>(kit.host);
    uint32_t *pc = cur.as<uint32_t>(), *pn = nxt.as<uint32_t>(), *sc = scur.as<uint32_t>(),
             *sn = snxt.as<uint32_t>();
    uint64_t F = 1, before = 0, seen = 1;
    int layers = 1, status = CG_OK;
    // every step from the unseen side goes over the whole bitmap: not for
    // layers whose neighbours are fewer than its words
    const uint32_t grid_all = (uint32_t)std::min<uint64_t>((W + 63) / 64, (uint64_t)device_cus() * 32);
    BmLists L = bm_lists(n, (uint32_t)k);
    uint32_t lg_seg = 0;
    double share = 1;  // of the fullest digit, spread evenly
    if (L.per_piece)
        with_bm_lists_n(n, [&](auto NN) {
            using Seg = BmSeg<decltype(NN)::value>;
            lg_seg = Seg::kLg;
            share = (double)Seg::kSubs / (double)Seg::kSegs;
        });
    // the lists are there from the first large layer on, if memory allows
    auto room_for_lists = [&]() {
        if (!lists.p) {
            try {
                lists.ensure(L.words() * 4);
                list_cnt.ensure(kBmCursors * sizeof(uint32_t));
            } catch (const Error &e) {
                if (e.code != CG_E_NOMEM) throw;
                lists.release();
                L.per_piece = 0;
                return false;
            }
        }
        return true;
    };
    try {
        for (;;) {
            if (k == 0) break;
            if (spec.max_frontier && F > spec.max_frontier) {
                status = CG_TRUNCATED;
                break;
            }
            if (layers >= spec.max_layers) {
                status = CG_TRUNCATED;
                break;
            }
            // (a next layer too small for lists is not counted by digit)
            const bool by_digit = L.per_piece && F * (uint64_t)k >= kBmSpreadMin;
            if (!looked && L.per_piece && crowd <= kBmCrowdedMost && F >= kBmSpreadMin &&
                F * (uint64_t)k >= bm_lists_min(n))
                look_for_scattered();
            const int density = bm_density(F, S), kf = scattered[density];
            const bool even = crowd <= bm_crowded(n, all_far[density], some_far[density]);
            const bool large = L.per_piece && even && F * (uint64_t)kf >= bm_lists_min(n);
            // (a scattered test costs two and a half neighbours that go through lists)
            const bool pull = F * (uint64_t)k >= W && pull_is_less(S - seen, F, before, (uint64_t)k,
                                                                   large ? 1.0 + 1.5 * (double)kf / (double)k : 1.0);
            bool by_lists = large && !pull && room_for_lists();
            if (by_lists) {
                // (the fullest list has a third more room than its even share)
                const uint32_t pieces = (uint32_t)std::ceil(std::max(1.0, crowd / 1.2) * (double)F * (double)kf /
                                                            (double)L.per_piece);
                uint32_t *const flag = cnt.as<uint32_t>() + kFlagAt;
                const PartShared<uint32_t> o{lists.as<uint32_t>(), (uint64_t)kBmSets * L.cap, L.cap,
                                             list_cnt.as<uint32_t>()};
                with_bm_lists_n(n, [&](auto NN) {
                    constexpr int N = decltype(NN)::value;
                    for (uint32_t p = 0; p < pieces; ++p) {
                        hipLaunchKernelGGL(bm_clear_kernel, dim3(kBmCursors / 256), dim3(256), 0, s,
                                           list_cnt.as<uint32_t>(), (uint64_t)kBmCursors,
                                           (unsigned long long *)nullptr);
                        hipLaunchKernelGGL(bm_part_kernel<N>, dim3(kBmPartBlocks), dim3(kPartBlock), 0, s, pc, W, p,
                                           pieces, gsel.as<const GenSel>(), (uint32_t)kf, o);
                        hipLaunchKernelGGL(bm_apply_kernel<N>, dim3(BmSeg<N>::kSubs << kBmLgDigits), dim3(kPartBlock),
                                           0, s, lists.as<const uint32_t>(), list_cnt.as<const uint32_t>(), L.cap,
                                           vis.as<const uint32_t>(), pn, sn, W, flag);
                    }
                });
                CG_HIP(hipGetLastError());
            }
            with_bm_n(n, [&](auto NN) {
                constexpr int N = decltype(NN)::value;
                const GenSel *const sel = gsel.as<const GenSel>();
                auto expand = [&](int g0, int g1, const uint32_t *go) {
                    if (g0 < g1)
                        hipLaunchKernelGGL(bm_expand_kernel<N>, dim3(grid), dim3(kBmBlock), 0, s, pc, sc,
                                           vis.as<const uint32_t>(), pn, sn, W, nchunks, sel + g0, g1 - g0, go);
                };
                if (pull) {
                    hipLaunchKernelGGL(bm_pull_kernel<N>, dim3(grid_all), dim3(kBmBlock), 0, s,
                                       vis.as<const uint32_t>(), pn, sn, W, sel + k, k);
                } else if (by_lists) {
                    expand(0, kf, cnt.as<const uint32_t>() + kFlagAt);  // if lists overran
                    expand(kf, k, nullptr);
                } else {
                    expand(0, k, nullptr);
                }
            });
            CG_HIP(hipGetLastError());
            hipLaunchKernelGGL(bm_fold_kernel, dim3(grid), dim3(kBmBlock), 0, s, vis.as<uint32_t>(), pc, sc, pn, sn,
                               W, nchunks, cnt.as<unsigned long long>(),
                               by_digit ? cnt.as<uint32_t>() + kDigitsAt : nullptr, lg_seg);
            CG_HIP(hipGetLastError());
            // the expanded layer's summary becomes the next layer's: clear it
            hipLaunchKernelGGL(bm_clear_kernel, dim3((uint32_t)std::min<uint64_t>((sw + 255) / 256, 4096)),
                               dim3(256), 0, s, sc, sw, (unsigned long long *)nullptr);
            CG_HIP(hipGetLastError());
            CG_HIP(hipMemcpyAsync(kit.host, cnt.p, (by_digit ? kCounts : 2) * sizeof(uint32_t),
                                  hipMemcpyDeviceToHost, s));
            hipLaunchKernelGGL(bm_clear_kernel, dim3(1), dim3(256), 0, s, cnt.as<uint32_t>() + kFlagAt,
                               (uint64_t)(by_digit ? kCounts - kFlagAt : 1u), cnt.as<unsigned long long>());
            CG_HIP(hipStreamSynchronize(s));
            const uint64_t N = host_cnt[0] | (uint64_t)host_cnt[1] << 32;
            crowd = 1e9;
            if (by_digit && N)
                crowd = (double)*std::max_element(host_cnt + kDigitsAt, host_cnt + kCounts) / ((double)N * share);
            res->states_expanded += F;
            res->candidates += F * (uint64_t)k;
            std::swap(pc, pn);
            std::swap(sc, sn);
            if (N == 0) break;
            sizes[layers++] = N;
            before = F;
            F = N;
            seen += N;
        }
    } catch (...) {
        give_kit(kit, hipStreamSynchronize(s) == hipSuccess);
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        throw;
    }
    CG_HIP(hipEventRecord(e1, s));
    CG_HIP(hipEventSynchronize(e1));
    float ms = 0;
    CG_HIP(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    give_kit(kit, true);
    for (DevBuf *b : {&vis, &cur, &nxt, &scur, &snxt, &gsel, &cnt, &lists, &list_cnt}) b->release();
    res->device_ms = ms;
    res->status = status;
    res->num_layers = layers;
    res->t_submit = t0;
    res->t_admit = t0;
    res->t_done = now_seconds();
}

}  // namespace cg
