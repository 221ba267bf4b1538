// Device side of the permute-expand step (used by the stand-alone expand
// kernel and by the first sort pass, which regenerates candidates from the
// frontier instead of reading them back).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"
#include "perm_rank.h"

namespace cg {

// Split a key into its even nibbles (E, bytes = nibbles 0,2,..,14) and odd
// nibbles (O, bytes = nibbles 1,3,..,15), one entry per byte.
struct Nibbles {
    uint32_t e0, e1, o0, o1;
};

__device__ __forceinline__ Nibbles split_nibbles(uint64_t key) {
    const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
    Nibbles r;
    r.e0 = lo & 0x0F0F0F0Fu;
    r.o0 = (lo >> 4) & 0x0F0F0F0Fu;
    r.e1 = hi & 0x0F0F0F0Fu;
    r.o1 = (hi >> 4) & 0x0F0F0F0Fu;
    return r;
}

// Generator g of a table, the same for a whole wave, by scalar loads.
__device__ __forceinline__ GenSel uniform_gensel(const GenSel *table, uint32_t g) {
    const uint32_t __attribute__((address_space(4))) *p =
        (const uint32_t __attribute__((address_space(4))) *)(uintptr_t)&table[g].sel[0];
    GenSel v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v.sel[i] = p[i];
    return v;
}

// s.g for the generator whose selectors are `g` (make_gensel).
__device__ __forceinline__ Nibbles apply_gensel_nibbles(const Nibbles &s, const GenSel &g) {
    Nibbles y;
    y.e0 = __builtin_amdgcn_perm(s.e1, s.e0, g.sel[0]) | __builtin_amdgcn_perm(s.o1, s.o0, g.sel[1]);
    y.e1 = __builtin_amdgcn_perm(s.e1, s.e0, g.sel[2]) | __builtin_amdgcn_perm(s.o1, s.o0, g.sel[3]);
    y.o0 = __builtin_amdgcn_perm(s.e1, s.e0, g.sel[4]) | __builtin_amdgcn_perm(s.o1, s.o0, g.sel[5]);
    y.o1 = __builtin_amdgcn_perm(s.e1, s.e0, g.sel[6]) | __builtin_amdgcn_perm(s.o1, s.o0, g.sel[7]);
    return y;
}
__device__ __forceinline__ uint64_t join_nibbles(const Nibbles &y) {
    return (uint64_t)(y.e1 | (y.o1 << 4)) << 32 | (y.e0 | (y.o0 << 4));
}

// Key of s.g.
__device__ __forceinline__ uint64_t apply_gensel(const Nibbles &s, const GenSel &g) {
    return join_nibbles(apply_gensel_nibbles(s, g));
}

__device__ __forceinline__ uint64_t apply_gensel(uint64_t key, const GenSel &g) {
    return apply_gensel(split_nibbles(key), g);
}

// Rank of a split state: its entries are read from their bytes.
template <int N, class R = uint32_t>
__device__ __forceinline__ R nibbles_rank_t(const Nibbles &y) {
    return perm_rank_of<N, R>([&](int i) {
        const int q = N - 1 - i;  // nibble of the key
        const uint32_t w = q & 1 ? (q < 8 ? y.o0 : y.o1) : (q < 8 ? y.e0 : y.e1);
        return (w >> (8 * (q / 2 % 4))) & 255u;
    });
}

}  // namespace cg
