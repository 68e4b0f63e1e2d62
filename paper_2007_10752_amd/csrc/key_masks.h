// Key masks of the bitsliced kernels: how an S-box's masks are read from a table
// in LDS (S-box j at kBsBoxMasks * j of a round's row: 4 output masks, up to 4
// second-use masks), or widened from a round's two key words, and the round
// runner whose masks stay in scalar registers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bitslice_core.h"
#include "generated/bitslice_keys_gen.h"

namespace tdes {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v3u __attribute__((ext_vector_type(3)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

constexpr bool box_ndup_fits() {
    for (int j = 0; j < 8; j++)
        if (BS_BOX_NDUP[j] < 0 || BS_BOX_NDUP[j] > 4) return false;
    return true;
}
static_assert(box_ndup_fits(), "an S-box has at most 4 second-use inputs");

#ifndef TDES_BS_PIPE
#define TDES_BS_PIPE 2  // S-boxes between a mask read from LDS and its use
#endif

// Masks of one S-box read from LDS.
struct LdsBoxLoad {
    // n (0..4, the box's second uses) is a compile-time constant after
    // inlining; only words that are used are read, so no read's destination
    // register is reused while the read is in flight
    template <class P>
    __device__ __forceinline__ void operator()(BsBoxMasks &m, P p, int n) const {
        // volatile keeps each read where it is issued (otherwise the reads
        // that cross the loop back edge are folded into reads at first use)
        typedef const volatile __attribute__((address_space(3))) v4u lds_v4u;
        typedef const volatile __attribute__((address_space(3))) v3u lds_v3u;
        typedef const volatile __attribute__((address_space(3))) v2u lds_v2u;
        typedef const volatile __attribute__((address_space(3))) uint32_t lds_u;
        const v4u a = *(lds_v4u *)p;
        m.o[0] = a[0]; m.o[1] = a[1]; m.o[2] = a[2]; m.o[3] = a[3];
        if (n == 4) {
            const v4u b = *(lds_v4u *)(p + 4);
            m.e[0] = b[0]; m.e[1] = b[1]; m.e[2] = b[2]; m.e[3] = b[3];
        } else if (n == 3) {
            const v3u b = *(lds_v3u *)(p + 4);
            m.e[0] = b[0]; m.e[1] = b[1]; m.e[2] = b[2];
        } else if (n == 2) {
            const v2u b = *(lds_v2u *)(p + 4);
            m.e[0] = b[0]; m.e[1] = b[1];
        } else if (n == 1) {
            m.e[0] = *(lds_u *)(p + 4);
        }
    }
};

// kBsBoxDup[4j + i] for a j known only at run time, without a memory
// lookup: column i packed into 5-bit fields of one constant (31: unused).
constexpr uint64_t dup_column(int i) {
    uint64_t c = 0;
    for (int j = 0; j < 8; j++) c |= (uint64_t)(kBsBoxDup[4 * j + i] & 31) << (5 * j);
    return c;
}
__device__ __forceinline__ int box_dup(int j, int i) {
    constexpr uint64_t kCol[4] = {dup_column(0), dup_column(1), dup_column(2), dup_column(3)};
    const int k = (int)((kCol[i] >> (5 * j)) & 31u);
    return k == 31 ? -1 : k;
}

// Masks widened from a round's key words (words 2t and 2t + 1 of a direction):
// output mask q of S-box j is bit 4j + q of the first, second use i bit
// kBsBoxDup[4j + i] of the second.
struct KeyWords {  // a round's key words and the place (8 a box) of the masks meant
    uint2 w;
    int at;
    __device__ __forceinline__ KeyWords operator+(int k) const { return KeyWords{w, at + k}; }
};
struct WidenedMasks {
    // (p.at and n are constants after inlining)
    __device__ __forceinline__ void operator()(BsBoxMasks &m, KeyWords p, int n) const {
        const int j = p.at / kBsBoxMasks;
#pragma unroll
        for (int q = 0; q < 4; q++)
            m.o[q] = (uint32_t)__builtin_amdgcn_sbfe((int)p.w.x, (uint32_t)(4 * j + q), 1);
#pragma unroll
        for (int i = 0; i < 4; i++)
            if (i < n)
                m.e[i] = (uint32_t)__builtin_amdgcn_sbfe((int)p.w.y, (uint32_t)kBsBoxDup[4 * j + i], 1);
    }
};

// Runs the rounds with masks widened one S-box ahead of their use.  Where the
// wave has one key, the words are uniform: the compiler widens them by scalar
// instructions and the masks enter the rounds as scalar operands, with no LDS and
// no vector registers for them.  Where every lane has its own, it is 48 v_bfe_i32 a
// round.
struct WordRounds {
    const uint32_t *words;  // the key's 100 words of one direction
    uint2 cur, next;        // key words of this round and the next
    BsBoxMasks pm[8];
    __device__ __forceinline__ uint2 load(int t) const { return make_uint2(words[2 * t], words[2 * t + 1]); }
    __device__ __forceinline__ void start() {
        cur = load(0);
        next = load(1);
        WidenedMasks{}(pm[0], KeyWords{cur, 0}, BS_BOX_NDUP[0]);
    }
    template <int PH>
    __device__ __forceinline__ void round(uint32_t (&d)[32], const uint32_t (&r)[32], int t) {
        const uint2 after = load(t + 2);  // past round 47: the extra words, not used
        bs_round_piped<1>(d, r, KeyWords{cur, 0}, KeyWords{next, 0}, pm, WidenedMasks{});
        cur = next;
        next = after;
    }
    __device__ __forceinline__ void extra(int g, uint32_t (&a)[32]) const {
        const uint32_t w = words[96 + g];
#pragma unroll
        for (int i = 0; i < 32; i++) a[i] ^= (uint32_t)__builtin_amdgcn_sbfe((int)w, (uint32_t)i, 1);
    }
};

}  // namespace tdes
