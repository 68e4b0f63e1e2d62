// The core of the table kernels (spbox.hip, batch_table.hip): the combined
// S-box + P tables in LDS and the 48 rounds on blocks held one per lane.  The
// method is described in spbox.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "generated/spbox_gen.h"
#include "internal.h"

namespace tdes {

constexpr int kTableThreads = 1024;  // threads of a workgroup
constexpr int kCopies = 32;
constexpr int kTableWords = 8 * 64 * kCopies;
constexpr int kTableBytes = 64 * kCopies * 4;  // one S-box's table
constexpr uint32_t kIndexMask = 63u << 7;      // entry index, scaled by 128 bytes

__device__ __forceinline__ uint32_t rotl(uint32_t x, int s) {
    return __builtin_amdgcn_alignbit(x, x, 32 - s);
}

// A constant held in a vector register: the asm hides the value, so it is
// not folded back into a scalar or literal operand.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t c) {
    uint32_t v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(c));
    return v;
}

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// One round: L ^ f(R, K).  `sp` is the LDS table base; `lane` is this
// lane's copy offset (4 (l % 32)); k = {odd chunks, even chunks, windows 0
// and 6 of the rotated half, window 7 of the rotated half}.
__device__ __forceinline__ uint32_t round_step(uint32_t L, uint32_t R, const uint8_t *sp,
                                               uint32_t lane, uint32_t mask, uint4 k) {
    const uint32_t ro = R ^ k.x, re = R ^ k.y, rr = rotl(R, 12);
    const uint32_t a06 = rr ^ k.z, a7 = rr ^ k.w;
    // (v >> sh) & mask | lane: 0xEA = (first & second) | third
    auto look = [&](int s, uint32_t v, int sh) {
        const uint32_t a = __builtin_amdgcn_bitop3_b32(v >> sh, mask, lane, 0xEA);
        return *reinterpret_cast<const uint32_t *>(sp + s * kTableBytes + a);
    };
    const uint32_t v0 = look(0, a06, 0), v1 = look(1, ro, 16), v2 = look(2, re, 12);
    const uint32_t v3 = look(3, ro, 8), v4 = look(4, re, 4), v5 = look(5, ro, 0);
    const uint32_t v6 = look(6, a06, 8), v7 = look(7, a7, 4);
    return xor3(xor3(v0, v1, v2), xor3(v3, v4, v5), xor3(v6, v7, L));
}

// IP, the 48 rounds and FP of N blocks at once, in place, interleaved so that
// one block's LDS reads wait while the others compute.  rk[i]: block i's keys.
template <int N>
__device__ __forceinline__ void cipher_blocks(uint2 (&w)[N], const uint8_t *sp, uint32_t lane,
                                              uint32_t mask, const uint4 *const (&rk)[N]) {
    uint32_t X[N], Y[N];
#pragma unroll
    for (int i = 0; i < N; i++) SP_IP(w[i].x, w[i].y, X[i], Y[i]);
    // Pass 1: L = X, R = Y.
#pragma unroll 2
    for (int r = 0; r < 16; r += 2) {
#pragma unroll
        for (int i = 0; i < N; i++) X[i] = round_step(X[i], Y[i], sp, lane, mask, rk[i][r]);
#pragma unroll
        for (int i = 0; i < N; i++) Y[i] = round_step(Y[i], X[i], sp, lane, mask, rk[i][r + 1]);
    }
    // Pass 2 from R16 || L16: L = Y, R = X.
#pragma unroll 2
    for (int r = 16; r < 32; r += 2) {
#pragma unroll
        for (int i = 0; i < N; i++) Y[i] = round_step(Y[i], X[i], sp, lane, mask, rk[i][r]);
#pragma unroll
        for (int i = 0; i < N; i++) X[i] = round_step(X[i], Y[i], sp, lane, mask, rk[i][r + 1]);
    }
    // Pass 3: L = X, R = Y.
#pragma unroll 2
    for (int r = 32; r < 48; r += 2) {
#pragma unroll
        for (int i = 0; i < N; i++) X[i] = round_step(X[i], Y[i], sp, lane, mask, rk[i][r]);
#pragma unroll
        for (int i = 0; i < N; i++) Y[i] = round_step(Y[i], X[i], sp, lane, mask, rk[i][r + 1]);
    }
#pragma unroll
    for (int i = 0; i < N; i++) {
        uint32_t o0, o1;
        SP_FP(X[i], Y[i], o0, o1);  // preoutput R16 || L16 = Y || X
        w[i] = make_uint2(o0, o1);
    }
}

// The same with one key.
template <int N>
__device__ __forceinline__ void cipher_blocks(uint2 (&w)[N], const uint8_t *sp, uint32_t lane,
                                              uint32_t mask, const uint4 *rk) {
    const uint4 *rks[N];
#pragma unroll
    for (int i = 0; i < N; i++) rks[i] = rk;
    cipher_blocks<N>(w, sp, lane, mask, rks);
}

// The workgroup's tables; no barrier.
__device__ __forceinline__ void fill_tables(uint32_t *table) {
    // the 512 entries x 32 copies as 16-byte chunks (8 per entry), lane i
    // writing chunks i, i + 1024, ...: each store of a wave covers 1 KiB in a
    // row, free of bank conflicts
    static_assert(kTableWords == 4 * 4 * kTableThreads && kCopies == 32, "table fill layout");
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int c = threadIdx.x + j * kTableThreads;
        const uint32_t v = SP_TABLE[c >> 3];
        reinterpret_cast<uint4 *>(table)[c] = make_uint4(v, v, v, v);
    }
}

}  // namespace tdes
