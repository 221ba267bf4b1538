// Write-combining partition of one workgroup's keys, for gfx950.
//
// Every digit owns a ring of keys in LDS; whole lines (128 bytes, or 64 with
// 1024 digits of 8-byte keys) go to the digit's own part of the output, so
// no line of memory is written twice or in pieces, no position is shared
// with another workgroup and no order is kept. A round takes R keys per
// thread; a key whose ring is full waits for the round's flush and tries
// again.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_util.h"
#include "internal.h"

namespace cg {

constexpr int kPartBlock = 1024;             // threads of a partition workgroup (one per CU: LDS)
constexpr uint32_t kPartBytes = 128u << 10;  // rings
constexpr uint32_t kPartMaxLgDigits = 10;

template <class K>
struct PartLds {
    static constexpr uint32_t kLgBuf = sizeof(K) == 4 ? 15 : 14;  // keys of all rings
    static constexpr uint32_t kMaxLines = sizeof(K) == 4 ? 1024 : 2048;
    static constexpr uint32_t kMaxDigits = sizeof(K) == 4 ? 512 : 1024;
    static_assert((sizeof(K) << kLgBuf) == kPartBytes, "rings");
    // keys per line written to memory
    static __device__ __forceinline__ uint32_t lg_line(uint32_t lg) {
        return sizeof(K) == 4 ? 5u : (lg > 9 ? 3u : 4u);
    }
    K buf[1u << kLgBuf];
    // a ring: its first key's place (high half) and how many it holds (low
    // half; may overshoot within a round). One word, so that a key's atomic
    // brings both.
    uint32_t ring[kMaxDigits];
    uint32_t head[kMaxDigits];   // keys written out so far, this round's lines included
    // the lines to write this round: first key in buf, and where to: lines
    // from the output's start (all ones: past the part's end, dropped)
    uint16_t line[kMaxLines];
    uint32_t at[kMaxLines];
    uint32_t lines[2];           // how many (by round parity)
    uint32_t more[2];            // some key of the block waits (by round parity)
};

template <class K>
struct PartOut {
    K *base;            // digit d's part: base + d * stride, cap keys (a multiple of 32)
    uint64_t stride;
    uint32_t cap;
    uint32_t *count;    // count[d * count_stride] = keys of digit d
    uint32_t count_stride;
    uint32_t *flags;    // gets `flag` when a part overran
    uint32_t flag;
    // where `keys` more of digit d go, of which `head` were written so far
    __device__ __forceinline__ uint32_t place(uint32_t, uint32_t head, uint32_t) const { return head; }
};

// Parts that several workgroups fill, a line at a time: for keys that come
// in lumps (many of one digit to one workgroup), which even out over the
// workgroups only. Unused places of a workgroup's last line hold all ones.
template <class K>
struct PartShared {
    K *base;            // digit d's part: base + d * stride, cap keys (a multiple of 32)
    uint64_t stride;
    uint32_t cap;
    uint32_t *cursor;   // cursor[d * kStep]: places given away (past cap: overrun)
    static constexpr uint32_t kStep = 16;  // a line of memory each
    __device__ __forceinline__ uint32_t place(uint32_t d, uint32_t, uint32_t keys) const {
        return atomicAdd(&cursor[d * kStep], keys);
    }
};

template <class K>
__device__ __forceinline__ void part_begin(PartLds<K> &L, uint32_t digits) {
    for (uint32_t i = threadIdx.x; i < digits; i += kPartBlock) L.ring[i] = L.head[i] = 0;
    if (threadIdx.x < 2) L.more[threadIdx.x] = L.lines[threadIdx.x] = 0;
    __syncthreads();
}

// One round: key[r] of digit dig[r] (below 2^lg) for the set bits r of
// `pend`. Every thread of the block calls it the same number of times.
template <class K, int R, class Out>
__device__ __forceinline__ void part_round(PartLds<K> &L, const K (&key)[R], const uint32_t (&dig)[R], uint32_t pend,
                                           uint32_t lg, const Out &o, uint32_t &parity) {
    const uint32_t lg_depth = PartLds<K>::kLgBuf - lg, depth = 1u << lg_depth, lg_line = PartLds<K>::lg_line(lg);
    const uint32_t tid = threadIdx.x, sub = tid & ((1u << lg_line) - 1), grp = tid >> lg_line;
    for (;;) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if ((pend >> r) & 1u) {
                const uint32_t d = dig[r];
                const uint32_t w = atomicAdd(&L.ring[d], 1u), n = w & 0xFFFFu;
                if (n < depth) {
                    L.buf[(d << lg_depth) + (((w >> 16) + n) & (depth - 1))] = key[r];
                    pend &= ~(1u << r);
                }
            }
        }
        if (pend) L.more[parity] = 1;
        __syncthreads();
        for (uint32_t d = tid; d < (1u << lg); d += kPartBlock) {
            const uint32_t w = L.ring[d], pos = w >> 16;
            const uint32_t have = min(w & 0xFFFFu, depth);  // less the keys that wait
            const uint32_t n = have >> lg_line, keys = n << lg_line;
            if (n || have != (w & 0xFFFFu)) L.ring[d] = ((pos + keys) & (depth - 1)) << 16 | (have - keys);
            if (n) {
                const uint32_t head = L.head[d], first = atomicAdd(&L.lines[parity], n);
                const uint32_t to = o.place(d, head, keys);
                for (uint32_t l = 0; l < n; ++l) {
                    const uint32_t at = to + (l << lg_line);
                    L.line[first + l] = (uint16_t)((d << lg_depth) + ((pos + (l << lg_line)) & (depth - 1)));
                    L.at[first + l] = at < o.cap ? (uint32_t)(((uint64_t)d * o.stride + at) >> lg_line) : ~0u;
                }
                L.head[d] = head + keys;
            }
        }
        if (tid == 0) L.more[parity ^ 1u] = L.lines[parity ^ 1u] = 0;
        __syncthreads();
        const uint32_t nl = L.lines[parity];
        for (uint32_t i = grp; i < nl; i += kPartBlock >> lg_line) {
            const uint32_t at = L.at[i];
            if (at != ~0u) o.base[((uint64_t)at << lg_line) + sub] = L.buf[L.line[i] + sub];
        }
        const bool more = L.more[parity] != 0;
        parity ^= 1u;
        __syncthreads();
        if (!more) break;
    }
}

// The keys still in the rings, then the counts.
template <class K>
__device__ __forceinline__ void part_end(PartLds<K> &L, uint32_t lg, const PartOut<K> &o) {
    const uint32_t lg_depth = PartLds<K>::kLgBuf - lg, depth = 1u << lg_depth;
    const uint32_t lg_line = PartLds<K>::lg_line(lg);
    const uint32_t sub = threadIdx.x & ((1u << lg_line) - 1), grp = threadIdx.x >> lg_line;
    for (uint32_t d = grp; d < (1u << lg); d += kPartBlock >> lg_line) {
        const uint32_t w = L.ring[d], n = w & 0xFFFFu, at = L.head[d] + sub, t = L.head[d] + n;
        if (sub < n && at < o.cap)
            o.base[(uint64_t)d * o.stride + at] = L.buf[(d << lg_depth) + (((w >> 16) + sub) & (depth - 1))];
        if (sub == 0) {
            o.count[(uint64_t)d * o.count_stride] = t < o.cap ? t : o.cap;
            if (t > o.cap) atomicOr(o.flags, o.flag);
        }
    }
}

// Shared parts: the keys still in the rings, as a line each.
template <class K>
__device__ __forceinline__ void part_end(PartLds<K> &L, uint32_t lg, const PartShared<K> &o) {
    const uint32_t lg_depth = PartLds<K>::kLgBuf - lg, depth = 1u << lg_depth;
    const uint32_t lg_line = PartLds<K>::lg_line(lg), line = 1u << lg_line;
    for (uint32_t d = threadIdx.x; d < (1u << lg); d += kPartBlock)
        if (L.ring[d] & 0xFFFFu) L.at[d] = o.place(d, 0, line);
    __syncthreads();
    const uint32_t sub = threadIdx.x & (line - 1), grp = threadIdx.x >> lg_line;
    for (uint32_t d = grp; d < (1u << lg); d += kPartBlock >> lg_line) {
        const uint32_t w = L.ring[d], n = w & 0xFFFFu;
        if (!n) continue;
        const uint32_t to = L.at[d];
        if (to < o.cap)
            o.base[(uint64_t)d * o.stride + to + sub] =
                sub < n ? L.buf[(d << lg_depth) + (((w >> 16) + sub) & (depth - 1))] : (K)~(K)0;
    }
}

// Keys a part has to hold when `mean` are expected: every state may come up
// to k times, so the variance is up to k times that of a uniform draw; seven
// deviations, and a few whole states' copies for parts that expect next to
// nothing. (CG_PART_FACTOR: times that, for tests of parts that overrun.)
inline uint32_t part_cap(double mean, uint32_t k) {
    mean *= plan_factor("CG_PART_FACTOR");
    const double c = mean + 7.0 * __builtin_sqrt((double)k * mean) + 4.0 * (double)k + 48.0;
    return ((uint32_t)c + 32) / 32 * 32;
}

}  // namespace cg
