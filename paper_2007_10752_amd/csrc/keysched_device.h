// DES round keys on the device, one a lane (Sec. III-A): the key's halves from a
// bit-matrix transpose, rotated once by the summed shift table, and gathers that
// move runs of bits as fields.  What a lane makes of its round key for the batched
// kernels' schedules and for the table kernel.  Plain C++, so that a host program
// can check it against keysched_core.h.
#pragma once
#include <stdint.h>

#include "keysched_core.h"

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define TDES_HD_INLINE __host__ __device__ __forceinline__
#else
#define TDES_HD_INLINE inline
#endif

namespace tdes {

// Bit i of the result is bit SRC::at(i) of src (64 bits), i < N <= 32; a run of
// consecutive source bits is moved as one field.
template <class SRC, int N, int I = 0>
TDES_HD_INLINE uint32_t pick_bits(uint64_t src) {
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
TDES_HD_INLINE uint64_t pc1_halves(uint64_t key) {
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
TDES_HD_INLINE uint64_t round_halves(uint64_t key, int i) {
    const uint64_t cd = pc1_halves(key);
    int s = 0;
#pragma unroll
    for (int j = 0; j < 16; j++) s += j <= i ? (int)kShifts[j] : 0;
    s %= 28;
    return (uint64_t)ks_rotl28((uint32_t)(cd >> 32), s) << 32 | ks_rotl28((uint32_t)cd & 0x0FFFFFFFu, s);
}

// The 8 key bytes at p as a little-endian word; aligned: p is a multiple of 8.
TDES_HD_INLINE uint64_t load_key(const uint8_t *p, bool aligned) {
    if (aligned) return *reinterpret_cast<const uint64_t *>(p);
    uint64_t key = 0;
    for (int i = 0; i < 8; i++) key |= (uint64_t)p[i] << (8 * i);
    return key;
}

struct Pc2Lo {  // round-key bit e (0..31, 32..47) at bit e % 32
    static constexpr int at(int i) { return pc2_at(i); }
};
struct Pc2Hi {
    static constexpr int at(int i) { return pc2_at(32 + i); }
};
struct PrimaryBits {  // of the expanded key: bit e at e
    static constexpr int at(int i) { return kBsPrimaryE[i]; }
};
struct DupKeyBits {
    static constexpr int at(int i) { return kBsDupE[i]; }
};
struct DupMaskBits {  // of the primary mask
    static constexpr int at(int i) { return kBsESrc[kBsDupE[i]]; }
};
struct OutBits {
    static constexpr int at(int i) { return kBsOutWord[i]; }
};

// What depends on round key i of a key alone: its primary mask, the same in the
// order of the S-box outputs, and its second-use word.
struct RoundMasks {
    uint32_t primary, out, dup;
};
TDES_HD_INLINE RoundMasks round_masks(uint64_t key, int i) {
    const uint64_t r = round_halves(key, i);
    const uint64_t rk = (uint64_t)pick_bits<Pc2Hi, 16>(r) << 32 | pick_bits<Pc2Lo, 32>(r);
    RoundMasks m;
    m.primary = pick_bits<PrimaryBits, 32>(rk);
    m.out = pick_bits<OutBits, 32>(m.primary);
    m.dup = pick_bits<DupKeyBits, 16>(rk) ^ pick_bits<DupMaskBits, 16>(m.primary);
    return m;
}

// Words 2t and 2t + 1 (bs_comp_word, bs_dup_word) of direction dir for t < 48, for
// t = 48 and 49 the extra words 96, 97 and 98, 99, from the round masks of the
// bundle's 48 round keys.
struct WordPair {
    uint32_t x, y;
};
TDES_HD_INLINE WordPair schedule_words(const uint32_t *primary, const uint32_t *out,
                                       const uint32_t *dup, int dir, int t) {
    WordPair w;
    if (t < 48) {
        const int before = bs_mask_before(t), after = bs_mask_after(t);
        w.x = (before < 0 ? 0u : out[round_key_slot(dir, before)]) ^
              (after < 0 ? 0u : out[round_key_slot(dir, after)]);
        w.y = dup[round_key_slot(dir, t)];
    } else {  // bs_extra_word
        auto P = [&](int r) { return primary[round_key_slot(dir, r)]; };
        w.x = t == 48 ? P(0) : P(31) ^ P(32);
        w.y = t == 48 ? P(15) ^ P(16) : P(47);
    }
    return w;
}

// The table kernel's keys of round key i of a key.
struct Pc2Low {  // round-key bit e at bit 47 - e, as host code has it
    static constexpr int at(int i) { return pc2_at(47 - i); }
};
struct Pc2High {
    static constexpr int at(int i) { return pc2_at(15 - i); }
};
TDES_HD_INLINE SpboxRound table_round_keys(uint64_t key, int i) {
    const uint64_t r = round_halves(key, i);
    return spbox_round_keys((uint64_t)pick_bits<Pc2High, 16>(r) << 32 | pick_bits<Pc2Low, 32>(r));
}

}  // namespace tdes
