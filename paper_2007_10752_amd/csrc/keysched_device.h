// DES round keys on the device, one a lane (Sec. III-A): the key's halves from a
// bit-matrix transpose, rotated once by the summed shift table, and gathers that
// move runs of bits as fields.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "keysched_core.h"

namespace tdes {

// Bit i of the result is bit SRC::at(i) of src (64 bits), i < N <= 32; a run of
// consecutive source bits is moved as one field.
template <class SRC, int N, int I = 0>
__device__ __forceinline__ uint32_t pick_bits(uint64_t src) {
    if constexpr (I >= N) {
        return 0;
    } else {
        constexpr int len = [] {
            int n = 1;
            while (I + n < N && SRC::at(I + n) == SRC::at(I) + n &&
                   SRC::at(I) / 32 == (SRC::at(I) + n) / 32)
                n++;
            return n;
        }();
        const uint32_t w = SRC::at(I) < 32 ? (uint32_t)src : (uint32_t)(src >> 32);
        const uint32_t field = (w >> (SRC::at(I) % 32)) & (uint32_t)((1ull << len) - 1);
        return field << I | pick_bits<SRC, N, I + len>(src);
    }
}
// Bit of the halves d (bits 0..27) and c (32..59) that PC-2 makes round-key bit e
// (0..47).
constexpr int pc2_at(int e) { return kPC2[e] <= 28 ? 32 + 28 - kPC2[e] : 56 - kPC2[e]; }

// PC-1 of a key read as a little-endian word: the 8x8 bit matrix of its bytes, last
// byte first, transposed by exchanging index bits (the two-word method of Warren,
// Hacker's Delight, Sec. 7-3), has row j = bit j + 1 of bytes 8 .. 1.
__device__ __forceinline__ uint64_t pc1_halves(uint64_t key) {
    uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)key, t;
    t = (hi ^ (hi >> 7)) & 0x00AA00AAu, hi ^= t ^ (t << 7);
    t = (lo ^ (lo >> 7)) & 0x00AA00AAu, lo ^= t ^ (t << 7);
    t = (hi ^ (hi >> 14)) & 0x0000CCCCu, hi ^= t ^ (t << 14);
    t = (lo ^ (lo >> 14)) & 0x0000CCCCu, lo ^= t ^ (t << 14);
    t = (hi & 0xF0F0F0F0u) | ((lo >> 4) & 0x0F0F0F0Fu);
    lo = ((hi << 4) & 0xF0F0F0F0u) | (lo & 0x0F0F0F0Fu);
    hi = t;
    // C: rows 1-3 and half of row 4; D: rows 7, 6, 5 and the other half of row 4
    const uint32_t c = hi >> 4;
    const uint32_t d = ((lo >> 8) & 0xFFu) << 20 | ((lo >> 16) & 0xFFu) << 12 | (lo >> 24) << 4 | (hi & 15u);
    return (uint64_t)c << 32 | d;
}

// The halves of round i (0..15), in the same places.
__device__ __forceinline__ uint64_t round_halves(uint64_t key, int i) {
    const uint64_t cd = pc1_halves(key);
    int s = 0;
#pragma unroll
    for (int j = 0; j < 16; j++) s += j <= i ? (int)kShifts[j] : 0;
    s %= 28;
    return (uint64_t)ks_rotl28((uint32_t)(cd >> 32), s) << 32 | ks_rotl28((uint32_t)cd & 0x0FFFFFFFu, s);
}

// The 8 key bytes at p as a little-endian word; aligned: p is a multiple of 8.
__device__ __forceinline__ uint64_t load_key(const uint8_t *p, bool aligned) {
    if (aligned) return *reinterpret_cast<const uint64_t *>(p);
    uint64_t key = 0;
    for (int i = 0; i < 8; i++) key |= (uint64_t)p[i] << (8 * i);
    return key;
}

}  // namespace tdes
