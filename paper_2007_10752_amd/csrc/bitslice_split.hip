// Bitsliced 3DES-EDE with the eight S-boxes of a chunk on eight waves, for
// inputs that leave the plain bitsliced kernel's SIMDs with a wave or two.
//
// A wave of the plain kernel (bitslice.hip) takes a chunk through 48 rounds of
// some 220 instructions each, ~28 us whatever the input's size, and a SIMD that
// holds one such wave has none to issue beside it.  Here a workgroup owns one
// 16 KiB chunk (2048 blocks, 32 per lane: lane l of every wave stands for the
// same 32 blocks) and wave w computes S-box w + 1 of every round, so it holds
// only what that box touches: the four words of each half that its outputs
// land in (P is fixed, so they are always the same four) and the six words of
// the other half that it reads.  After a round a wave writes its four new words
// to LDS ([word][lane]: 256 B a row, free of bank conflicts) and, behind one
// barrier, reads its six for the next round.  The halves have a buffer each, so
// a round's writes never meet the reads of the round before.  Rounds 15 | 16 and
// 31 | 32 need no exchange: the same half feeds both.
//
// The key masks are bits of the launch's key words, widened by scalar
// instructions: no mask table in LDS, and nothing to build before the rounds.
//
// With one chunk a CU a round takes ~540 clocks, most of it the exchange, which all
// waves make at once: 80 rows of LDS traffic (160 clocks at 128 B a clock), two LDS
// latencies and the barrier.  A second chunk fits beside it almost free; from the
// third on LDS traffic (8,320 clocks a chunk) and issue slots (6,400, the masks'
// operations do not pair) add up, neither of them full (0.54 of a CU's time each at
// 12 MiB), and the plain kernel is the faster one where its SIMDs hold two waves or
// more.  Measured (us a launch, plain -> split): 2 MiB 28.4 -> 14.2, 4 MiB 29.2 -> 14.7,
// 8 MiB 30.0 -> 16.3, 12 MiB 30.2 -> 21.0, 16 MiB 30.8 -> 26.0, 20 MiB
// 34.5 -> 31.9.  The round loop unrolled four times: 8 MiB 17.2 -> 16.5, 12 MiB 21.5
// -> 21.1.  Key words picked from vector registers by v_readlane in place of scalar
// loads: 18.3 and 22.8.  Two boxes a wave (four waves, fewer rows): 19.2 at 1 MiB,
// 27.9 at 16 MiB.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bitslice_core.h"
#include "generated/bitslice_boxes_gen.h"
#include "generated/bitslice_keys_gen.h"
#include "internal.h"

namespace tdes {

namespace {

typedef uint32_t v2u __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kWaves = 8;
constexpr size_t kChunk = 16384;
constexpr int kBufferFlags = 0x00020000;  // word 3 of a raw gfx9 buffer resource

// LDS words of one chunk: two halves of 32 words x 64 lanes.
typedef uint32_t Exchange[2][32][kWave];

// All earlier LDS accesses of the workgroup are done (no wait for global
// memory, unlike __syncthreads).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Bit b of w as 0 / ~0.
__device__ __forceinline__ uint32_t mask_bit(uint32_t w, int b) {
    return (uint32_t)__builtin_amdgcn_sbfe((int)w, (uint32_t)b, 1);
}

// The words S-box `box` reads (E) and updates (P).
constexpr int src_word(int box, int i) { return (4 * box + 31 + i) % 32; }
constexpr int own_word(int box, int i) { return kBsOutWord[4 * box + i]; }
constexpr bool sources_consecutive() {
    for (int e = 0; e < 48; e++)
        if (kBsESrc[e] != src_word(e / 6, e % 6)) return false;
    return true;
}
static_assert(sources_consecutive(), "E as index arithmetic");

// Plane 32 h + 8 k + j (bit j of byte k of word h) is word 8 (3 - j / 2) +
// 7 - 4 h - k of the left half (even j) or the right half (odd j); the
// preoutput's words land in planes by the mirrored rule.
constexpr bool planes_regular() {
    for (int h = 0; h < 2; h++)
        for (int k = 0; k < 4; k++)
            for (int j = 0; j < 8; j++) {
                const int in = 8 * (3 - j / 2) + 7 - 4 * h - k, plane = 32 * h + 8 * k + j;
                if ((j % 2 ? BS_IP_R : BS_IP_L)[in] != plane) return false;
                const int out = 31 - 8 * (j / 2) - 4 * h - k;
                if (BS_FP_SRC[plane] != out + (j % 2 ? 32 : 0)) return false;
            }
    return true;
}
static_assert(planes_regular(), "IP and FP as index arithmetic");

// The 48 rounds of the wave that runs S-box B.  ex holds the halves (left in
// ex[0]) before and R16, L16 after.
template <int B>
__device__ __forceinline__ void split_rounds(const BitsliceKeys &keys, Exchange &ex, uint32_t lane) {
    uint32_t D1[4], D2[4], S[6];
#pragma unroll
    for (int i = 0; i < 4; i++) D1[i] = ex[0][own_word(B, i)][lane];
#pragma unroll
    for (int i = 0; i < 4; i++) D2[i] = ex[1][own_word(B, i)][lane];
#pragma unroll
    for (int i = 0; i < 6; i++) S[i] = ex[1][src_word(B, i)][lane];
    lds_barrier();
    // one round: kw, kd its two key words
    auto box = [&](uint32_t (&D)[4], uint32_t kw, uint32_t kd) {
        BsBoxMasks m;
#pragma unroll
        for (int q = 0; q < 4; q++) m.o[q] = mask_bit(kw, 4 * B + q);
#pragma unroll
        for (int i = 0; i < 4; i++)
            m.e[i] = kBsBoxDup[4 * B + i] < 0 ? 0u : mask_bit(kd, kBsBoxDup[4 * B + i]);
        bs_box<B>(S, D, m);
    };
    auto exchange = [&](uint32_t (&D)[4], int half) {
#pragma unroll
        for (int i = 0; i < 4; i++) ex[half][own_word(B, i)][lane] = D[i];
        lds_barrier();
#pragma unroll
        for (int i = 0; i < 6; i++) S[i] = ex[half][src_word(B, i)][lane];
    };
    // the key words of two rounds, loaded two rounds ahead (past round 47:
    // the four extra words, not used as keys)
    uint32_t k0 = keys.w[0], k1 = keys.w[1], k2 = keys.w[2], k3 = keys.w[3];
    int t = 0;
#pragma unroll 1
    for (int pass = 0; pass < 3; pass++) {
        // the source half takes the mask of its next use (initial mask, re-masks)
        const uint32_t kx = keys.w[96 + pass];
#pragma unroll
        for (int i = 0; i < 4; i++) D2[i] ^= mask_bit(kx, own_word(B, i));
#pragma unroll
        for (int i = 0; i < 6; i++) S[i] ^= mask_bit(kx, src_word(B, i));
        const int left = pass & 1;
#pragma unroll 4
        for (int r = 0; r < 8; r++) {
            t += 2;
            const uint32_t n0 = keys.w[2 * t], n1 = keys.w[2 * t + 1];
            const uint32_t n2 = keys.w[2 * t + 2], n3 = keys.w[2 * t + 3];
            box(D1, k0, k1);
            exchange(D1, left);
            box(D2, k2, k3);
            k0 = n0, k1 = n1, k2 = n2, k3 = n3;
            if (r < 7) exchange(D2, left ^ 1);
        }
        // R16 || L16: the halves change places
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t u = D1[i];
            D1[i] = D2[i];
            D2[i] = u;
        }
    }
    const uint32_t kx = keys.w[99];
#pragma unroll
    for (int i = 0; i < 4; i++) D2[i] ^= mask_bit(kx, own_word(B, i));
    lds_barrier();  // the last round's source words have been read
#pragma unroll
    for (int i = 0; i < 4; i++) ex[0][own_word(B, i)][lane] = D1[i];
#pragma unroll
    for (int i = 0; i < 4; i++) ex[1][own_word(B, i)][lane] = D2[i];
    lds_barrier();
}

template <int B = 0>
__device__ __forceinline__ void split_wave(uint32_t wave, const BitsliceKeys &keys, Exchange &ex,
                                           uint32_t lane) {
    if (B == 7 || wave == B)
        split_rounds<B>(keys, ex, lane);
    else if constexpr (B < 7)
        split_wave<B + 1>(wave, keys, ex, lane);
}

// Byte transpose: byte k of word c to byte c of word k.
__device__ __forceinline__ void bytes4x4(uint32_t (&x)[4]) {
    const uint32_t lo = vconst(0x05040100u), hi = vconst(0x07060302u);
    const uint32_t ev = vconst(0x06020400u), od = vconst(0x07030501u);
    const uint32_t a = __builtin_amdgcn_perm(x[2], x[0], lo), c = __builtin_amdgcn_perm(x[2], x[0], hi);
    const uint32_t b = __builtin_amdgcn_perm(x[3], x[1], lo), d = __builtin_amdgcn_perm(x[3], x[1], hi);
    x[0] = __builtin_amdgcn_perm(b, a, ev);
    x[1] = __builtin_amdgcn_perm(b, a, od);
    x[2] = __builtin_amdgcn_perm(d, c, ev);
    x[3] = __builtin_amdgcn_perm(d, c, od);
}

// One stage of the 8x8 bit transposes in the four byte columns of 8 words.
template <int J>
__device__ __forceinline__ void bit_stage(uint32_t (&x)[8]) {
    const uint32_t k0 = vconst(J == 4 ? 0x0F0F0F0Fu : J == 2 ? 0x33333333u : 0x55555555u);
#pragma unroll
    for (int i = 0; i < 8; i++) {
        if (i & J) continue;
        const uint32_t a = x[i], b = x[i + J];
        x[i] = __builtin_amdgcn_bitop3_b32(a, shl_paired<J>(b), k0, 0xE4);
        x[i + J] = __builtin_amdgcn_bitop3_b32(a >> J, b, k0, 0xE4);
    }
}
__device__ __forceinline__ void bits8x8(uint32_t (&x)[8]) {
    bit_stage<4>(x);
    bit_stage<2>(x);
    bit_stage<1>(x);
}

template <int MODE>
__global__ __launch_bounds__(kWave * kWaves)
void tdes_bitslice_split_kernel(const uint8_t *in, uint8_t *out, size_t nbytes, BitsliceKeys keys,
                                ModeArgs mode) {
    __shared__ Exchange ex;
    uint32_t(*rows)[kWave] = reinterpret_cast<uint32_t(*)[kWave]>(&ex);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t lane = threadIdx.x % kWave;
    const size_t base = (size_t)blockIdx.x * kChunk;
    // buffer resources sized to the chunk: loads past the input's end read 0,
    // stores past it are dropped
    const uint32_t avail = (uint32_t)(nbytes - base < kChunk ? nbytes - base : kChunk);
    const __amdgpu_buffer_rsrc_t src =
        __builtin_amdgcn_make_buffer_rsrc((void *)(in + base), 0, (int)avail, kBufferFlags);
    const __amdgpu_buffer_rsrc_t dst =
        __builtin_amdgcn_make_buffer_rsrc((void *)(out + base), 0, (int)avail, kBufferFlags);

    // Wave w moves block w of the lane's four byte columns c: half w % 2 of
    // the 16-byte piece 4 (w / 2) + c (waves 2 m and 2 m + 1 share its lines).
    const uint32_t off = lane * 16u + (wave % 2) * 8u + (wave / 2) * 4096u;
    v2u p[4];
#pragma unroll
    for (int c = 0; c < 4; c++) {
        if (MODE == kModeCtr) {
            const uint64_t ctr = mode.ctr + (base + off) / 8 + (uint64_t)(c * 128);
            p[c] = v2u{__builtin_bswap32((uint32_t)(ctr >> 32)), __builtin_bswap32((uint32_t)ctr)};
        } else {
            p[c] = __builtin_amdgcn_raw_buffer_load_b64(src, off + c * 1024u, 0, 0);
        }
    }

    // Words to bytes: row 8 (4 h + k) + w holds byte k of word h of block w,
    // one byte per column c.
#pragma unroll
    for (int h = 0; h < 2; h++) {
        uint32_t x[4] = {p[0][h], p[1][h], p[2][h], p[3][h]};
        bytes4x4(x);
#pragma unroll
        for (int k = 0; k < 4; k++) rows[8 * (4 * h + k) + wave][lane] = x[k];
    }
    lds_barrier();
    // Bytes to planes: wave w takes byte place 4 h + k = w.
    uint32_t x[8];
#pragma unroll
    for (int i = 0; i < 8; i++) x[i] = rows[8 * wave + i][lane];
    lds_barrier();
    bits8x8(x);
#pragma unroll
    for (int j = 0; j < 8; j++) ex[j % 2][8 * (3 - j / 2) + 7 - wave][lane] = x[j];
    lds_barrier();

    split_wave(wave, keys, ex, lane);

    // What is XORed into the result: CTR's input, CBC's previous blocks.
    v2u q[4];
    if (MODE == kModeCtr) {
#pragma unroll
        for (int c = 0; c < 4; c++)
            q[c] = __builtin_amdgcn_raw_buffer_load_b64(src, off + c * 1024u, 0, 0);
    }
    if (MODE == kModeCbcDec) {
        // from a resource 8 bytes before the chunk, so that no offset is
        // negative; before the first chunk there is nothing, and its first
        // block (out of range there, read as 0) takes the IV
        const uint32_t shift = base > 0 ? 8u : 0u;
        const __amdgpu_buffer_rsrc_t prev = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(in + base - shift), 0, (int)(avail + shift), kBufferFlags);
        const bool first = base == 0 && off == 0;
#pragma unroll
        for (int c = 0; c < 4; c++)
            q[c] = __builtin_amdgcn_raw_buffer_load_b64(
                prev, c == 0 && first ? 0x40000000u : off + c * 1024u + shift - 8u, 0, 0);
        if (first) q[0] = v2u{mode.iv0, mode.iv1};
    }

    // Preoutput R16 || L16 (ex[0], ex[1]) to planes, then back to blocks.
#pragma unroll
    for (int j = 0; j < 8; j++) x[j] = ex[j % 2][31 - 8 * (j / 2) - wave][lane];
    lds_barrier();
    bits8x8(x);
#pragma unroll
    for (int i = 0; i < 8; i++) rows[8 * wave + i][lane] = x[i];
    lds_barrier();
#pragma unroll
    for (int h = 0; h < 2; h++) {
        uint32_t y[4];
#pragma unroll
        for (int k = 0; k < 4; k++) y[k] = rows[8 * (4 * h + k) + wave][lane];
        bytes4x4(y);
#pragma unroll
        for (int c = 0; c < 4; c++) p[c][h] = MODE == kModeEcb ? y[c] : y[c] ^ q[c][h];
    }
#pragma unroll
    for (int c = 0; c < 4; c++)
        __builtin_amdgcn_raw_buffer_store_b64(p[c], dst, off + c * 1024u, 0, 0);
}

}  // namespace

template <int MODE>
hipError_t launch_bitslice_split(const BitsliceKeys &k, const ModeArgs &m, const uint8_t *in,
                                 uint8_t *out, size_t nbytes, hipStream_t stream) {
    const size_t chunks = (nbytes + kChunk - 1) / kChunk;
    if (chunks == 0 || chunks > 0x7fffffffu) return hipErrorInvalidValue;
    hipLaunchKernelGGL(tdes_bitslice_split_kernel<MODE>, dim3((unsigned)chunks), dim3(kWave * kWaves),
                       0, stream, in, out, nbytes, k, m);
    return hipGetLastError();
}
template hipError_t launch_bitslice_split<kModeEcb>(const BitsliceKeys &, const ModeArgs &,
                                                    const uint8_t *, uint8_t *, size_t, hipStream_t);
template hipError_t launch_bitslice_split<kModeCtr>(const BitsliceKeys &, const ModeArgs &,
                                                    const uint8_t *, uint8_t *, size_t, hipStream_t);
template hipError_t launch_bitslice_split<kModeCbcDec>(const BitsliceKeys &, const ModeArgs &,
                                                       const uint8_t *, uint8_t *, size_t,
                                                       hipStream_t);

}  // namespace tdes
