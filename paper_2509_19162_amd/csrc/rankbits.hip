// Layers over a rank-space bitmap: the layer step of permutations of up to
// 12 entries, without a sort.
//
// A state of S_n has one bit, at a bijective scramble of its lexicographic
// rank (on ceil(log2 n!) bits: 64 MB at n = 12), so one bitmap holds every
// state seen so far, exactly, and a neighbour is new iff its bit was clear.
// The bitmap stands for all earlier layers: the generating set need not be
// closed under inverses. Layers stay packed keys, one layer after another in
// one array, in no order.
//
// Three forms of the step:
//   rb_step_kernel   small layers: every neighbour is tested and claimed in
//                    memory. The kernel reads the layer's place and size from
//                    device counters and leaves the next layer's there, so
//                    several layers are launched one behind another and read
//                    back together;
//   rb_part_kernel + rb_segment_kernel   large layers: device atomics run at
//                    27 G/s on this chip whatever the bitmap's size, LDS
//                    atomics at 2000 G/s. So the neighbours' bit numbers are
//                    partitioned into 512 segments of the bitmap (4 bytes
//                    written and read per neighbour), and one workgroup per
//                    segment sets them in LDS, takes off the visited bits and
//                    writes out the new states;
//   rb_pull_kernel   large layers late in a growth: the unseen states look
//                    for a seen predecessor instead.
//
// S_12 pancake (479,001,600 states, 5.3e9 neighbours, every layer kept): 76.3
// ms by sorting, 36 with the first two forms (partition 23.7 ms, 2.2e11
// neighbours/s, bound by the rank arithmetic; segments 9.3), 27.7 with the
// third (9.3 + 5.1 + 10.1). S_10 with six random generators 1.66 -> 0.37 ms,
// a directed pair on S_11 12.0 -> 1.46.
#include "rankbits.h"

#include <algorithm>

#include "device_util.h"
#include "expand_device.h"
#include "partition_device.h"
#include "perm_rank.h"

namespace cg {

namespace {

constexpr int kRbBlock = 1024;
constexpr uint32_t kRbWaves = kRbBlock / kWave;
constexpr int kRbRows = 4;  // neighbours per thread and round

__host__ __device__ __forceinline__ uint32_t rb_word(uint32_t d) { return (d % kRbWindow) * kRbStride; }

__device__ __forceinline__ uint64_t rb_uniform(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return (uint64_t)hi << 32 | lo;
}

// ---- bit numbers ---------------------------------------------------------------
// The scramble spreads the layers (whose ranks crowd: few inversions, common
// leading entries) evenly over the segments, and the neighbours of one
// segment's states over all segments. Shifts by at least half the width are
// their own inverse.
template <int N>
struct RbBits {
    static constexpr int bits() {
        uint64_t f = 1;
        for (int i = 2; i <= N; ++i) f *= (uint64_t)i;
        int b = 0;
        while ((1ull << b) < f) ++b;
        return b;
    }
    static constexpr int B = bits() < 5 ? 5 : bits();
    static constexpr uint32_t kMask = (uint32_t)((1ull << B) - 1);
    static constexpr int kShift = (B + 1) / 2;
    static constexpr uint32_t kMul1 = 0x2C1B3C6Du, kMul2 = 0x297A2D39u;
    static constexpr uint32_t inverse(uint32_t a) {  // of an odd a, modulo 2^32 (Newton)
        uint32_t x = a;
        for (int i = 0; i < 5; ++i) x *= 2u - a * x;
        return x;
    }
    static constexpr uint32_t kInv1 = inverse(kMul1), kInv2 = inverse(kMul2);
    static __device__ __forceinline__ uint32_t of_rank(uint32_t r) {
        r ^= r >> kShift;
        r = (r * kMul1) & kMask;
        r ^= r >> kShift;
        return (r * kMul2) & kMask;
    }
    static __device__ __forceinline__ uint32_t to_rank(uint32_t x) {
        x = (x * kInv2) & kMask;
        x ^= x >> kShift;
        x = (x * kInv1) & kMask;
        return x ^ (x >> kShift);
    }
    static __device__ __forceinline__ uint32_t of_key(uint64_t key) { return of_rank(perm_rank_t<N>(key)); }
    static __device__ __forceinline__ uint32_t of_state(const Nibbles &y) { return of_rank(nibbles_rank_t<N>(y)); }
    // bits of a segment: 512 segments
    static constexpr int kLgSeg = B - (int)kRbLgDigits;
};

__global__ void rb_set_kernel(RbArgs a, uint32_t d, uint64_t off, uint64_t F) {
    const uint32_t i = threadIdx.x;
    if (i < kRbWindow) {
        const bool here = i == d % kRbWindow;
        a.cnt[i * kRbStride] = here ? F : 0ull;
        a.off[i * kRbStride] = here ? off : 0ull;
    }
    if (i == 0) *a.flags = 0;
}

template <int N>
__global__ __launch_bounds__(256) void rb_mark_kernel(const uint64_t *__restrict__ keys, uint64_t n, uint32_t *seen) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t r = RbBits<N>::of_key(keys[i]);
    atomicOr(&seen[r >> 5], 1u << (r & 31u));
}

// A block takes items of (1024 states) x (a range of generators); a round
// maps the item's states through four generators. A neighbour whose bit
// reads as clear is claimed by an atomic OR: whoever finds the bit still
// clear owns the state (a stale read costs an atomic, never a state). The
// round's new states are appended together, one global atomic per round.
template <int N>
__global__ __launch_bounds__(kRbBlock) __attribute__((amdgpu_waves_per_eu(8))) void rb_step_kernel(RbArgs a,
                                                                                                   uint32_t d) {
    __shared__ uint32_t s_n[2][kRbWaves];
    __shared__ uint64_t s_base[2];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint64_t F = rb_uniform(a.cnt[rb_word(d)]), off = rb_uniform(a.off[rb_word(d)]);
    if (blockIdx.x == 0 && tid == 0) {
        a.off[rb_word(d + 1)] = off + F;
        a.cnt[rb_word(d + 2)] = 0;
    }
    if (F == 0 || (a.max_frontier && F > a.max_frontier)) return;
    uint64_t *const next = a.all + off + F;
    const uint64_t room = a.cap - (off + F);
    const uint32_t tiles = (uint32_t)((F + kRbBlock - 1) / kRbBlock);
    const uint32_t quads = (a.k + kRbRows - 1) / kRbRows;
    uint32_t ranges = gridDim.x / tiles;  // enough items for every block
    ranges = ranges < 1 ? 1 : (ranges > quads ? quads : ranges);
    uint32_t parity = 0;
    for (uint64_t it = blockIdx.x; it < (uint64_t)tiles * ranges; it += gridDim.x) {
        const uint32_t tile = (uint32_t)(it / ranges), range = (uint32_t)(it - (uint64_t)tile * ranges);
        const uint32_t q0 = (uint32_t)((uint64_t)quads * range / ranges);
        const uint32_t q1 = (uint32_t)((uint64_t)quads * (range + 1) / ranges);
        const uint64_t f = (uint64_t)tile * kRbBlock + tid;
        const bool in = f < F;
        const uint64_t key = in ? a.all[off + f] : 0ull;
        const Nibbles s = split_nibbles(key);
        for (uint32_t q = q0; q < q1; ++q) {
            uint64_t t[kRbRows];
            uint32_t r[kRbRows], word[kRbRows];
            bool fresh[kRbRows];
#pragma unroll
            for (int j = 0; j < kRbRows; ++j) {
                const uint32_t g = q * kRbRows + j < a.k ? q * kRbRows + j : a.k - 1;
                const Nibbles y = apply_gensel_nibbles(s, uniform_gensel(a.sel, g));
                t[j] = join_nibbles(y);
                r[j] = RbBits<N>::of_state(y);
                fresh[j] = in && q * kRbRows + j < a.k;
                word[j] = fresh[j] ? a.seen[r[j] >> 5] : ~0u;
            }
            uint32_t mine = 0;
            uint64_t m[kRbRows];
#pragma unroll
            for (int j = 0; j < kRbRows; ++j) {
                const uint32_t bit = 1u << (r[j] & 31u);
                fresh[j] = fresh[j] && !(word[j] & bit);
                if (fresh[j]) fresh[j] = !(atomicOr(&a.seen[r[j] >> 5], bit) & bit);
                m[j] = __ballot(fresh[j]);
                mine += (uint32_t)__popcll(m[j]);
            }
            if (lane == 0) s_n[parity][wave] = mine;
            __syncthreads();
            uint32_t before = 0, total = 0;
#pragma unroll
            for (uint32_t w = 0; w < kRbWaves; ++w) {
                const uint32_t c = s_n[parity][w];
                before += w < wave ? c : 0;
                total += c;
            }
            if (tid == 0 && total)
                s_base[parity] = atomicAdd((unsigned long long *)&a.cnt[rb_word(d + 1)], (unsigned long long)total);
            __syncthreads();
            if (total) {
                uint64_t at = s_base[parity] + before;
#pragma unroll
                for (int j = 0; j < kRbRows; ++j) {
                    if (fresh[j]) {
                        const uint64_t x = at + mask_rank(m[j]);
                        if (x < room)
                            next[x] = t[j];
                        else
                            atomicOr(a.flags, kRbFlagRoom);
                    }
                    at += (uint32_t)__popcll(m[j]);
                }
            }
            parity ^= 1u;
        }
    }
}

// ---- large layers ----------------------------------------------------------------
constexpr int kRbPartStates = 4, kRbPartGens = 2;  // states and generators of a round, per thread
constexpr int kRbPartRows = kRbPartStates * kRbPartGens;
constexpr uint32_t kRbPartTile = kPartBlock * kRbPartStates;

// Items of (4096 states) x (a range of pairs of generators), dealt to the
// blocks in turn; a round forms eight neighbours per thread.
template <int N>
__global__ __launch_bounds__(kPartBlock) void rb_part_kernel(const uint64_t *__restrict__ layer, uint64_t F,
                                                             const GenSel *sel, uint32_t k, uint32_t tiles,
                                                             uint32_t ranges, PartOut<uint32_t> o) {
    __shared__ PartLds<uint32_t> L;
    constexpr uint32_t lg = kRbLgDigits;
    const uint32_t tid = threadIdx.x;
    part_begin(L, 1u << lg);
    o.base += (uint64_t)blockIdx.x * o.cap;
    o.count += blockIdx.x;
    uint32_t parity = 0;
    const uint32_t pairs = (k + kRbPartGens - 1) / kRbPartGens;
    for (uint32_t it = blockIdx.x; it < tiles * ranges; it += gridDim.x) {
        const uint32_t tile = it / ranges, range = it - tile * ranges;
        const uint32_t p0 = (uint32_t)((uint64_t)pairs * range / ranges);
        const uint32_t p1 = (uint32_t)((uint64_t)pairs * (range + 1) / ranges);
        Nibbles s[kRbPartStates];
        uint32_t in = 0;
#pragma unroll
        for (int j = 0; j < kRbPartStates; ++j) {
            const uint64_t f = (uint64_t)tile * kRbPartTile + (uint32_t)j * kPartBlock + tid;
            s[j] = split_nibbles(f < F ? layer[f] : 0ull);
            if (f < F) in |= 1u << j;
        }
        for (uint32_t p = p0; p < p1; ++p) {
            uint32_t x[kRbPartRows], dig[kRbPartRows], pend = 0;
#pragma unroll
            for (int h = 0; h < kRbPartGens; ++h) {
                const uint32_t g = p * kRbPartGens + h;
                if (g < k) pend |= in << (h * kRbPartStates);
                const GenSel G = uniform_gensel(sel, g < k ? g : k - 1);
#pragma unroll
                for (int j = 0; j < kRbPartStates; ++j) {
                    const uint32_t r = RbBits<N>::of_state(apply_gensel_nibbles(s[j], G));
                    x[h * kRbPartStates + j] = r & ((1u << RbBits<N>::kLgSeg) - 1u);
                    dig[h * kRbPartStates + j] = r >> RbBits<N>::kLgSeg;
                }
            }
            part_round(L, x, dig, pend, lg, o, parity);
        }
    }
    part_end(L, lg, o);
}

// One segment: the neighbours' bits in LDS, less the visited ones; the new
// states' keys are appended to the next layer (their bits taken back to
// ranks and unranked).
template <int N>
__global__ __launch_bounds__(kRbBlock) void rb_segment_kernel(RbArgs a, uint32_t d, const uint32_t *__restrict__ in,
                                                              const uint32_t *__restrict__ in_count, uint32_t nsrc,
                                                              uint32_t in_cap, uint32_t width) {
    constexpr uint32_t kWords = 1u << (RbBits<N>::kLgSeg - 5), kWaves = kRbWaves, BLOCK = kRbBlock;
    __shared__ uint32_t s_bits[kWords];
    __shared__ uint32_t s_scan[kWaves];
    __shared__ uint64_t s_base;
    const uint32_t tid = threadIdx.x, seg = blockIdx.x;
    for (uint32_t w = tid; w < kWords; w += BLOCK) s_bits[w] = 0;
    __syncthreads();
    // `width` lanes to a part (16 where the parts are short)
    const uint32_t sub = tid & (width - 1u), step = 4 * width;
    for (uint32_t i = tid / width; i < nsrc; i += BLOCK / width) {
        const uint64_t part = (uint64_t)seg * nsrc + i;
        const uint32_t *p = in + part * in_cap;
        const uint32_t n = in_count[part];
        for (uint32_t b = sub; b < n; b += step) {
            uint32_t x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = b + (uint32_t)u * width;
                x[u] = j < n ? p[j] : ~0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (x[u] != ~0u) atomicOr(&s_bits[x[u] >> 5], 1u << (x[u] & 31u));
        }
    }
    __syncthreads();
    uint32_t *seen = a.seen + (uint64_t)seg * kWords;
    uint32_t mine = 0;
    for (uint32_t w = tid; w < kWords; w += BLOCK) {
        const uint32_t x = s_bits[w];
        if (!x) continue;
        const uint32_t v = seen[w], fresh = x & ~v;
        s_bits[w] = fresh;
        if (fresh) seen[w] = v | fresh;
        mine += (uint32_t)__popc(fresh);
    }
    uint32_t total;
    uint32_t at = block_excl_scan<kWaves>(mine, s_scan, &total);
    if (total == 0) return;
    if (tid == 0) s_base = atomicAdd((unsigned long long *)&a.cnt[rb_word(d + 1)], (unsigned long long)total);
    __syncthreads();
    const uint64_t off = a.off[rb_word(d + 1)];
    if (off + s_base + total > a.cap) {
        if (tid == 0) atomicOr(a.flags, kRbFlagRoom);
        return;
    }
    uint64_t *next = a.all + off + s_base;
    for (uint32_t w = tid; w < kWords; w += BLOCK) {
        uint32_t x = s_bits[w];
        while (x) {
            const uint32_t b = (uint32_t)__builtin_ctz(x);
            x &= x - 1u;
            next[at++] = perm_unrank_t<N>(RbBits<N>::to_rank(seg << RbBits<N>::kLgSeg | w << 5 | b));
        }
    }
}

// ---- the step from the other side --------------------------------------------------
// Late in a growth few states are left unseen while the frontier is large.
// Then each unseen state asks whether a state it comes from (its image under
// an inverse generator) has been seen, and stops at the first that has: a
// state unseen so far with a seen predecessor is in the next layer, and no
// other is. Seen bits are read from one bitmap and written to another
// (`to`), so bits found on the way are not mistaken for earlier ones.
// Bit numbers of no rank are marked seen beforehand.
template <int N>
__global__ __launch_bounds__(256) void rb_mark_unused_kernel(uint32_t *seen) {
    constexpr uint32_t kWords = 1u << (RbBits<N>::B - 5);
    constexpr uint64_t kStates = [] {
        uint64_t f = 1;
        for (int i = 2; i <= N; ++i) f *= (uint64_t)i;
        return f;
    }();
    for (uint32_t w = blockIdx.x * 256 + threadIdx.x; w < kWords; w += gridDim.x * 256) {
        uint32_t x = 0;
        for (uint32_t b = 0; b < 32; ++b)
            if (RbBits<N>::to_rank(w << 5 | b) >= kStates) x |= 1u << b;
        if (x) seen[w] |= x;
    }
}

// A block takes 256 words of the bitmap at a time: their unseen bits are
// listed in LDS, then every thread takes one listed state per round.
template <int N>
__global__ __launch_bounds__(kRbBlock) __attribute__((amdgpu_waves_per_eu(8))) void rb_pull_kernel(
    RbArgs a, uint32_t d, const GenSel *inv, uint32_t *__restrict__ to) {
    constexpr uint32_t kWords = 1u << (RbBits<N>::B - 5), kChunk = 256;
    __shared__ uint16_t s_list[kChunk * 32];
    __shared__ uint32_t s_new[kChunk];
    __shared__ uint32_t s_scan[kRbWaves], s_n[2][kRbWaves];
    __shared__ uint64_t s_base[2];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint64_t off = rb_uniform(a.off[rb_word(d + 1)]);
    const uint64_t room = a.cap - off;
    uint64_t *const next = a.all + off;
    const uint32_t *__restrict__ seen = a.seen;
    uint32_t parity = 0;
    for (uint32_t w0 = blockIdx.x * kChunk; w0 < kWords; w0 += gridDim.x * kChunk) {
        uint32_t v = ~0u;
        if (tid < kChunk) {
            v = seen[w0 + tid];
            s_new[tid] = 0;
        }
        uint32_t n;
        uint32_t at = block_excl_scan<kRbWaves>((uint32_t)__popc(~v), s_scan, &n);
        for (uint32_t x = ~v; x; x &= x - 1u) s_list[at++] = (uint16_t)(tid << 5 | (uint32_t)__builtin_ctz(x));
        __syncthreads();
        for (uint32_t i0 = 0; i0 < n; i0 += kRbBlock) {
            const uint32_t i = i0 + tid;
            bool hit = false;
            uint32_t bit = 0;
            uint64_t key = 0;
            if (i < n) {
                bit = s_list[i];
                key = perm_unrank_t<N>(RbBits<N>::to_rank((w0 << 5) + bit));
                const Nibbles s = split_nibbles(key);
                for (uint32_t g = 0; g < a.k && !hit; ++g) {
                    const uint32_t r = RbBits<N>::of_state(apply_gensel_nibbles(s, uniform_gensel(inv, g)));
                    hit = (seen[r >> 5] >> (r & 31u)) & 1u;
                }
                if (hit) atomicOr(&s_new[bit >> 5], 1u << (bit & 31u));
            }
            const uint64_t m = __ballot(hit);
            if (lane == 0) s_n[parity][wave] = (uint32_t)__popcll(m);
            __syncthreads();
            uint32_t before = 0, total = 0;
#pragma unroll
            for (uint32_t w = 0; w < kRbWaves; ++w) {
                const uint32_t c = s_n[parity][w];
                before += w < wave ? c : 0;
                total += c;
            }
            if (tid == 0 && total)
                s_base[parity] = atomicAdd((unsigned long long *)&a.cnt[rb_word(d + 1)], (unsigned long long)total);
            __syncthreads();
            if (hit) {
                const uint64_t x = s_base[parity] + before + mask_rank(m);
                if (x < room)
                    next[x] = key;
                else
                    atomicOr(a.flags, kRbFlagRoom);
            }
            parity ^= 1u;
        }
        __syncthreads();
        if (tid < kChunk) to[w0 + tid] = v | s_new[tid];
        __syncthreads();
    }
}

// Place and size of layer d (host values) and cleared counts of the next two.
__global__ void rb_next_kernel(RbArgs a, uint32_t d, uint64_t off, uint64_t F) {
    a.off[rb_word(d)] = off;
    a.cnt[rb_word(d)] = F;
    a.off[rb_word(d + 1)] = off + F;
    a.cnt[rb_word(d + 1)] = 0;
    a.cnt[rb_word(d + 2)] = 0;
}

template <class Fn>
void with_rb_large_n(int n, Fn &&fn) {
    switch (n) {
        case 10: fn(std::integral_constant<int, 10>{}); break;
        case 11: fn(std::integral_constant<int, 11>{}); break;
        default: fn(std::integral_constant<int, 12>{}); break;
    }
}

}  // namespace

void launch_rb_begin(int n, const RbArgs &a, uint32_t d, uint64_t off, uint64_t F, hipStream_t s) {
    hipLaunchKernelGGL(rb_set_kernel, dim3(1), dim3(kRbWindow), 0, s, a, d, off, F);
    CG_HIP(hipGetLastError());
    const uint64_t m = off + F;
    with_rank_n(n, [&](auto NN) {
        hipLaunchKernelGGL((rb_mark_kernel<decltype(NN)::value>), dim3((uint32_t)((m + 255) / 256)), dim3(256), 0, s,
                           a.all, m, a.seen);
    });
    CG_HIP(hipGetLastError());
}

void launch_rb_step(int n, const RbArgs &a, uint32_t d, uint64_t most, PipeWork &w) {
    const uint64_t items = (most + kRbBlock - 1) / kRbBlock * ((a.k + kRbRows - 1) / kRbRows);
    const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(items, 512));
    if (w.prof) w.prof->begin(K_STEP);
    with_rank_n(n, [&](auto NN) {
        hipLaunchKernelGGL((rb_step_kernel<decltype(NN)::value>), dim3(grid), dim3(kRbBlock), 0, w.stream, a, d);
    });
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->end(K_STEP, 0, 0);
}

uint64_t rb_bitmap_words(int n) {
    uint64_t w = 1;
    with_rank_n(n, [&](auto NN) { w = 1ull << (RbBits<decltype(NN)::value>::B - 5); });
    return w;
}

RbPlan rb_plan(uint64_t F, uint32_t k) {
    RbPlan p;
    const uint32_t pairs = (k + kRbPartGens - 1) / kRbPartGens;
    p.tiles = (uint32_t)((F + kRbPartTile - 1) / kRbPartTile);
    p.ranges = p.tiles >= 512 ? 1u : std::min(pairs, (512 + p.tiles - 1) / p.tiles);
    const uint64_t items = (uint64_t)p.tiles * p.ranges;
    p.blocks = (uint32_t)std::min<uint64_t>(items, 256);
    const double per_item = (double)std::min<uint64_t>(F, kRbPartTile) *
                            (double)std::min<uint32_t>(k, kRbPartGens * ((pairs + p.ranges - 1) / p.ranges));
    const double per_block = per_item * (double)((items + p.blocks - 1) / p.blocks);
    p.cap = part_cap(per_block / (double)(1u << kRbLgDigits), k);
    return p;
}

void launch_rb_large(int n, const RbArgs &a, uint32_t d, uint64_t off, uint64_t F, const RbPlan &p, uint32_t *part,
                     uint32_t *count, PipeWork &w) {
    hipLaunchKernelGGL(rb_next_kernel, dim3(1), dim3(1), 0, w.stream, a, d, off, F);
    CG_HIP(hipGetLastError());
    const double C = (double)F * (double)a.k;
    if (w.prof) w.prof->begin(K_EXPAND);
    PartOut<uint32_t> o{part, (uint64_t)p.blocks * p.cap, p.cap, count, p.blocks, a.flags, kRbFlagPart};
    with_rb_large_n(n, [&](auto NN) {
        hipLaunchKernelGGL((rb_part_kernel<decltype(NN)::value>), dim3(p.blocks), dim3(kPartBlock), 0, w.stream,
                           a.all + off, F, a.sel, a.k, p.tiles, p.ranges, o);
    });
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->end(K_EXPAND, 8.0 * (double)F + 4.0 * C, C);
    if (w.prof) w.prof->begin(K_BUCKET);
    with_rb_large_n(n, [&](auto NN) {
        hipLaunchKernelGGL((rb_segment_kernel<decltype(NN)::value>), dim3(1u << kRbLgDigits), dim3(kRbBlock), 0,
                           w.stream, a, d, (const uint32_t *)part, (const uint32_t *)count, p.blocks, p.cap,
                           p.cap < 512 ? 16u : (uint32_t)kWave);
    });
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->end(K_BUCKET, 4.0 * C, C);
}

void launch_rb_mark_unused(int n, uint32_t *seen, hipStream_t s) {
    with_rb_large_n(n, [&](auto NN) {
        hipLaunchKernelGGL((rb_mark_unused_kernel<decltype(NN)::value>), dim3(4096), dim3(256), 0, s, seen);
    });
    CG_HIP(hipGetLastError());
}

void launch_rb_pull(int n, const RbArgs &a, uint32_t d, uint64_t off, uint64_t F, const GenSel *inv, uint32_t *to,
                    PipeWork &w) {
    hipLaunchKernelGGL(rb_next_kernel, dim3(1), dim3(1), 0, w.stream, a, d, off, F);
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->begin(K_STEP);
    const uint32_t grid = (uint32_t)std::min<uint64_t>(512, rb_bitmap_words(n) / 256);
    with_rb_large_n(n, [&](auto NN) {
        hipLaunchKernelGGL((rb_pull_kernel<decltype(NN)::value>), dim3(grid), dim3(kRbBlock), 0, w.stream, a, d, inv,
                           to);
    });
    CG_HIP(hipGetLastError());
    if (w.prof) w.prof->end(K_STEP, 8.0 * (double)rb_bitmap_words(n), 0);  // both bitmaps once
}

}  // namespace cg
