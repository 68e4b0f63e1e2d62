// Bitsliced 3DES-EDE ECB kernel for gfx950.
//
// Data layout.  One wave owns a 16 KiB chunk (2048 blocks).  Lane l loads
// the 16-byte pieces at chunk offsets l*16 + k*1024, k = 0..15, so every
// load instruction of the wave reads 1 KiB of contiguous memory, and the
// lane ends up with 32 blocks (which 32 is irrelevant in ECB: each block is
// stored back where it came from).  Two in-register 32x32 bit transposes turn
// the 32 blocks x 2 words into 64 "plane" words: plane h*32 + p holds bit
// position p of word h of all 32 blocks, one block per bit.
//
// Arithmetic.  In plane form every DES permutation is a renaming of
// registers: IP picks which planes form L and R, E picks which R words feed
// each S-box, P picks which L word each S-box output is XORed into, FP picks
// which word goes to which output plane.  The S-boxes (Sec. III-B) are
// gate networks of v_bitop3_b32 (any boolean function of three inputs),
// found by search and verified exhaustively at build time.  Key mixing is an
// XOR with all-zeros / all-ones masks (the key is uniform over the launch),
// mostly folded into the XOR that adds an S-box output into the other half:
// each half is kept XORed with the key bits its next round needs (the mask
// bookkeeping is done on the host, see keysched.cpp).  The three DES passes of EDE run back
// to back in registers: FP followed by IP is the identity, so the inner
// permutations vanish and the R16 || L16 swap between passes is a change of
// roles between the two halves.
//
// Modes.  ECB processes the loaded blocks.  CTR (SP 800-38A) processes
// counter blocks made in registers (the block at byte offset o holds
// ctr + o / 8, big-endian) and XORs the data into the result on the way
// out; nothing is loaded before the rounds.  CBC decryption decrypts the
// loaded blocks, then XORs each with the ciphertext block before it (the
// IV before the first), re-read after the rounds.
//
// Bound by VALU issue: an instruction takes 2.35 clocks of its SIMD on 1 GiB, 2.0
// where every one pairs with another wave's.  1 GiB by the operations of a round,
// each pair on one machine: 242 (196 S-box gates) 1,083 us, 224 (176 gates) 1,028;
// 224 1,066 us, 211 (163 gates) 1,015; 211 919, 202 (159 gates, five of the sixteen
// second-use masks folded into them) 892; 202 910, 201 (six folded) 906.
//
// The key masks are scalars, widened from the key words by scalar instructions.
// Read from a table in LDS, 17 reads a round (vector operands, which were thought to
// pair where scalar ones do not), they cost issue slots: 1 GiB 986 -> 918 us, 64 MiB
// 69.2 -> 64.8, CTR of 256 MiB 255 -> 239, CBC decryption 264 -> 248.  Workgroups of
// one wave or two: the same at most sizes (48 MiB: 59 us with two, 50 with one or
// four); of eight: 36 MiB 58 to 48.  A 6-wave register budget: 64 MiB 68 to 66.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bitslice_core.h"
#include "key_masks.h"
#include "generated/bitslice_keys_gen.h"
#include "internal.h"

#ifndef TDES_BS_MIN_WAVES
#define TDES_BS_MIN_WAVES 4  // waves per SIMD the register budget must allow
#endif

namespace tdes {

namespace {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr size_t kChunk = 16384;  // bytes per wave
// Buffer-resource word 3 for gfx9-family raw (unstructured) buffers.
constexpr int kBufferFlags = 0x00020000;

// The 16-byte piece k of a lane (blocks 2k and 2k + 1), read after the
// rounds: one 16-byte load, or two 8-byte loads on the partial path.
template <bool WHOLE>
__device__ __forceinline__ v4u load_piece_late(__amdgpu_buffer_rsrc_t src, uint32_t lane_off, int k) {
    if (WHOLE) return __builtin_amdgcn_raw_buffer_load_b128(src, lane_off, k * 1024, 0);
    const v2u a = __builtin_amdgcn_raw_buffer_load_b64(src, lane_off, k * 1024, 0);
    const v2u b = __builtin_amdgcn_raw_buffer_load_b64(src, lane_off + 8u, k * 1024, 0);
    return v4u{a[0], a[1], b[0], b[1]};
}

// CBC decryption output: XOR each decrypted block with the ciphertext block
// before it.  Piece k's two previous blocks are the 16 bytes at 8 bytes
// before the piece: prev resource offset vbase + k * 1024.  The first block
// of the whole buffer takes the IV instead (the caller marks it with
// first_iv and gives it the out-of-range offset voff0, read as 0).
template <bool WHOLE>
__device__ __forceinline__ void cbc_store_blocks(const uint32_t (&h0)[32], const uint32_t (&h1)[32],
                                                 __amdgpu_buffer_rsrc_t prev,
                                                 __amdgpu_buffer_rsrc_t dst, uint32_t lane_off,
                                                 uint32_t voff0, uint32_t vbase, bool first_iv,
                                                 uint32_t iv0, uint32_t iv1) {
#pragma unroll
    for (int g = 0; g < 4; g++) {
        __builtin_amdgcn_sched_barrier(0);
        v4u pv[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int k = 4 * g + j;
            const uint32_t off = vbase + (uint32_t)(k * 1024);
            if (k == 0) {
                // two halves: block A's previous block (out of range where the
                // IV stands in), block B's (block A itself)
                const v2u a = __builtin_amdgcn_raw_buffer_load_b64(prev, voff0, 0, 0);
                const v2u b = __builtin_amdgcn_raw_buffer_load_b64(prev, off + 8u, 0, 0);
                pv[j] = v4u{a[0], a[1], b[0], b[1]};
            } else if (WHOLE) {
                pv[j] = __builtin_amdgcn_raw_buffer_load_b128(prev, off, 0, 0);
            } else {
                const v2u a = __builtin_amdgcn_raw_buffer_load_b64(prev, off, 0, 0);
                const v2u b = __builtin_amdgcn_raw_buffer_load_b64(prev, off + 8u, 0, 0);
                pv[j] = v4u{a[0], a[1], b[0], b[1]};
            }
        }
        if (g == 0 && first_iv) {
            pv[0][0] = iv0;
            pv[0][1] = iv1;
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int k = 4 * g + j;
            const v4u v = {h0[2 * k] ^ pv[j][0], h1[2 * k] ^ pv[j][1], h0[2 * k + 1] ^ pv[j][2],
                           h1[2 * k + 1] ^ pv[j][3]};
            if (WHOLE) {
                __builtin_amdgcn_raw_buffer_store_b128(v, dst, lane_off, k * 1024, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b64(v2u{v[0], v[1]}, dst, lane_off, k * 1024, 0);
                __builtin_amdgcn_raw_buffer_store_b64(v2u{v[2], v[3]}, dst, lane_off + 8u, k * 1024, 0);
            }
        }
    }
}

// CTR output: XOR the lane's 32 input blocks into its 32 keystream blocks
// and store each piece as soon as it is complete, four pieces at a time (16
// registers of input in flight; each result goes straight to its store).
template <bool WHOLE>
__device__ __forceinline__ void xor_store_blocks(const uint32_t (&h0)[32], const uint32_t (&h1)[32],
                                                 __amdgpu_buffer_rsrc_t src,
                                                 __amdgpu_buffer_rsrc_t dst, uint32_t lane_off) {
#pragma unroll
    for (int g = 0; g < 4; g++) {
        __builtin_amdgcn_sched_barrier(0);
        v4u dv[4];
#pragma unroll
        for (int j = 0; j < 4; j++) dv[j] = load_piece_late<WHOLE>(src, lane_off, 4 * g + j);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int k = 4 * g + j;
            const v4u v = {h0[2 * k] ^ dv[j][0], h1[2 * k] ^ dv[j][1], h0[2 * k + 1] ^ dv[j][2],
                           h1[2 * k + 1] ^ dv[j][3]};
            if (WHOLE) {
                __builtin_amdgcn_raw_buffer_store_b128(v, dst, lane_off, k * 1024, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b64(v2u{v[0], v[1]}, dst, lane_off, k * 1024, 0);
                __builtin_amdgcn_raw_buffer_store_b64(v2u{v[2], v[3]}, dst, lane_off + 8u, k * 1024, 0);
            }
        }
    }
}

// Every mode takes 84-89 registers (5 waves per SIMD).
template <bool VEC16, int MODE>
__global__ __launch_bounds__(kWave *kWavesPerBlock)
__attribute__((amdgpu_waves_per_eu(TDES_BS_MIN_WAVES, 8)))
void tdes_bitslice_kernel(const uint8_t *in, uint8_t *out, size_t nbytes, BitsliceKeys keys,
                          ModeArgs mode) {
    // Issue priority: a new wave's loads and transposes run at the highest
    // priority and its rounds at the lowest.  The SIMD's arbiter otherwise
    // favours the older waves, which are in their rounds, so a new wave
    // reaches its own rounds late and fewer waves are there to pair
    // instructions (1 GiB 872 us, 928 without).
    __builtin_amdgcn_s_setprio(3);
    // the wave index is uniform within the wave; say so, so the chunk base
    // and the buffer resources below live in scalar registers
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const size_t chunk = (size_t)blockIdx.x * kWavesPerBlock + wave;
    const size_t base = chunk * kChunk;
    const bool live = base < nbytes;  // wave-uniform
    const uint32_t lane_off = (threadIdx.x % kWave) * 16u;
    // Bytes of this chunk that exist: 16384 except in the last chunk.  The
    // chunk is addressed through buffer resources sized to it, so the
    // hardware range check zero-fills loads and drops stores past the end.
    // The partial path (last chunk, or 8-byte aligned buffers) is written
    // with 8-byte accesses; the compiler may merge a lane's two loads into
    // one 16-byte load, which is still exact because the range check
    // applies per dword (odd block counts in the parity tests cover a piece
    // that straddles the end).
    const uint32_t avail = live ? (uint32_t)(nbytes - base < kChunk ? nbytes - base : kChunk) : 0u;
    const bool whole = VEC16 && avail == (uint32_t)kChunk;
    const __amdgpu_buffer_rsrc_t src =
        __builtin_amdgcn_make_buffer_rsrc((void *)(in + base), 0, (int)avail, kBufferFlags);
    const __amdgpu_buffer_rsrc_t dst =
        __builtin_amdgcn_make_buffer_rsrc((void *)(out + base), 0, (int)avail, kBufferFlags);

    // the chunk
    uint32_t h0[32], h1[32];
    if (MODE == kModeCtr) {
        if (live) {
            // counter blocks: ctr + (byte offset) / 8, as big-endian bytes,
            // so each 32-bit word (loaded little-endian) is byte-swapped
            const uint64_t c0 = mode.ctr + (base + lane_off) / 8;
#pragma unroll
            for (int k = 0; k < 16; k++) {
                const uint64_t ca = c0 + (uint64_t)(k * 128), cb = ca + 1;
                h0[2 * k] = __builtin_bswap32((uint32_t)(ca >> 32));
                h1[2 * k] = __builtin_bswap32((uint32_t)ca);
                h0[2 * k + 1] = __builtin_bswap32((uint32_t)(cb >> 32));
                h1[2 * k + 1] = __builtin_bswap32((uint32_t)cb);
            }
        }
    } else if (whole) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const v4u v = __builtin_amdgcn_raw_buffer_load_b128(src, lane_off, k * 1024, 0);
            h0[2 * k] = v[0];
            h1[2 * k] = v[1];
            h0[2 * k + 1] = v[2];
            h1[2 * k + 1] = v[3];
        }
    } else if (live) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const v2u a = __builtin_amdgcn_raw_buffer_load_b64(src, lane_off, k * 1024, 0);
            const v2u b = __builtin_amdgcn_raw_buffer_load_b64(src, lane_off + 8u, k * 1024, 0);
            h0[2 * k] = a[0];
            h1[2 * k] = a[1];
            h0[2 * k + 1] = b[0];
            h1[2 * k + 1] = b[1];
        }
    }

    if (!live) return;

    // one transpose at a time: interleaved, they hold more words live than
    // the register budget allows
    transpose32(h0);
    __builtin_amdgcn_sched_barrier(0);
    transpose32(h1);
    __builtin_amdgcn_sched_barrier(0);

    __builtin_amdgcn_s_setprio(0);
    WordRounds rr;
    rr.words = keys.w;
    des3_planes(h0, h1, rr);
    __builtin_amdgcn_sched_barrier(0);
    transpose32(h0);
    __builtin_amdgcn_sched_barrier(0);
    transpose32(h1);

    if (MODE == kModeCtr) {
        if (whole)
            xor_store_blocks<true>(h0, h1, src, dst, lane_off);
        else
            xor_store_blocks<false>(h0, h1, src, dst, lane_off);
        return;
    }
    if (MODE == kModeCbcDec) {
        // previous blocks: a resource from 8 bytes before the chunk (none
        // before the first chunk, whose first block takes the IV), so every
        // offset is non-negative
        const uint32_t shift = base > 0 ? 8u : 0u;
        const __amdgpu_buffer_rsrc_t prev = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(in + base - shift), 0, (int)(avail + shift), kBufferFlags);
        const bool first_iv = base == 0 && lane_off == 0;
        // lane_off + shift - 8 wraps for lane 0 of the first chunk; adding
        // k * 1024 (k >= 1) brings it back to k * 1024 - 8, and piece 0 of
        // that lane reads from an out-of-range offset instead
        const uint32_t vbase = lane_off + shift - 8u;
        const uint32_t voff0 = first_iv ? 0x40000000u : vbase;
        if (whole)
            cbc_store_blocks<true>(h0, h1, prev, dst, lane_off, voff0, vbase, first_iv, mode.iv0,
                                   mode.iv1);
        else
            cbc_store_blocks<false>(h0, h1, prev, dst, lane_off, voff0, vbase, first_iv, mode.iv0,
                                    mode.iv1);
        return;
    }
    if (whole) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const v4u v = {h0[2 * k], h1[2 * k], h0[2 * k + 1], h1[2 * k + 1]};
            __builtin_amdgcn_raw_buffer_store_b128(v, dst, lane_off, k * 1024, 0);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const v2u a = {h0[2 * k], h1[2 * k]}, b = {h0[2 * k + 1], h1[2 * k + 1]};
            __builtin_amdgcn_raw_buffer_store_b64(a, dst, lane_off, k * 1024, 0);
            __builtin_amdgcn_raw_buffer_store_b64(b, dst, lane_off + 8u, k * 1024, 0);
        }
    }
}

}  // namespace

template <int MODE>
hipError_t launch_bitslice_mode(const BitsliceKeys &k, const ModeArgs &m, const uint8_t *in,
                                uint8_t *out, size_t nbytes, hipStream_t stream) {
    const size_t chunks = (nbytes + kChunk - 1) / kChunk;
    // Up to five chunks a CU every SIMD here would hold one wave, some two, and
    // the split kernel is the faster (us on 256 CUs, split against this: 8 MiB 16.3 to
    // 30.0, 12 MiB 21.0 to 30.2, 16 MiB 26.0 to 30.8, 20 MiB 31.9 to 34.5; CTR of 20
    // MiB 30.5 to 34.8, CBC decryption 31.1 to 35.1).  Each chunk a CU more costs it 5
    // us, this one 0.3 as long as the waves a SIMD are the same.  Of calls that overlap on several
    // streams this kernel does more, which a call cannot see: us a call on two and on
    // four streams, 8 MiB 10.7, 10.3 to 15.7, 10.3; 12 MiB 15.6, 16.0 to 16.2, 11.6; 16
    // MiB 20.5, 21.1 to 17.1, 13.5.
    if (chunks <= 5 * device_cus()) return launch_bitslice_split<MODE>(k, m, in, out, nbytes, stream);
    const size_t blocks = (chunks + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > 0x7fffffffu) return hipErrorInvalidValue;
    const bool vec16 = ((((uintptr_t)in) | ((uintptr_t)out)) & 15u) == 0;
    if (vec16)
        hipLaunchKernelGGL((tdes_bitslice_kernel<true, MODE>), dim3((unsigned)blocks),
                           dim3(kWave * kWavesPerBlock), 0, stream, in, out, nbytes, k, m);
    else
        hipLaunchKernelGGL((tdes_bitslice_kernel<false, MODE>), dim3((unsigned)blocks),
                           dim3(kWave * kWavesPerBlock), 0, stream, in, out, nbytes, k, m);
    return hipGetLastError();
}

template hipError_t launch_bitslice_mode<kModeCtr>(const BitsliceKeys &, const ModeArgs &,
                                                   const uint8_t *, uint8_t *, size_t, hipStream_t);
template hipError_t launch_bitslice_mode<kModeCbcDec>(const BitsliceKeys &, const ModeArgs &,
                                                      const uint8_t *, uint8_t *, size_t,
                                                      hipStream_t);

hipError_t launch_bitslice(const BitsliceKeys &k, const uint8_t *in, uint8_t *out,
                           size_t nbytes, hipStream_t stream) {
    return launch_bitslice_mode<kModeEcb>(k, ModeArgs{}, in, out, nbytes, stream);
}

}  // namespace tdes
