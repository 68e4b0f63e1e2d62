// Table-driven 3DES-EDE ECB kernel for gfx950: one 64-bit block per lane
// (up to four at a time, interleaved, in its grid-stride loop).
//
// Each round (Sec. III-B) computes f(R, K) as the XOR of eight lookups in
// combined S-box + straight-permutation tables SP_s[64] (32-bit words: the
// S-box output already moved to its P position), indexed by the six R bits
// the expansion feeds S-box s XORed with six round-key bits.  The tables
// live in LDS, replicated 32 times and interleaved so that entry e of copy c
// sits in bank c (byte 128 e + 4 c of the table): lane l reads copy l % 32,
// so a lookup is free of bank conflicts whatever the indices.  (8 tables x
// 64 entries x 32 copies x 4 B = 64 KiB per workgroup.)
//
// Key mixing: windows 1..6 of the expansion are contiguous in R (bit i of R
// at position 32 - i) and odd and even windows are disjoint, so XORing R
// once with the odd key chunks and once with the even ones keys windows
// 1..5.  Windows 0 and 7 wrap around; in R rotated left by 12 they sit at
// positions 7..12 and 11..16, and window 6 at 15..20, so one XOR of the
// rotated R keys windows 0 and 6 and another keys window 7.  Every window
// then lies at or above position 7: a right shift brings it to bits 7..12,
// and one three-input bitwise op masks it and adds the lane's copy offset,
// which makes the LDS byte address (the table's base goes into the
// instruction's offset field).  Shifts right, three-input bitwise ops and
// XORs of vector registers are the VALU instructions that issue together
// with another wave's; the mask and the copy offset are held in vector
// registers, and so are the round keys (read from LDS, where the workgroup
// copies them), so only the rotation issues alone.  The eight table words
// and the left half are folded by four three-input XORs.
//
// IP and FP run once per block as delta swaps; the three DES passes are
// fused as in the bitsliced kernel (FP then IP cancel between passes).
//
// The modes are those of bitslice.hip.  Inputs of a block per lane are bound by
// one lane's chain of rounds (203 clocks each; the table fill takes ~2,100),
// large ones by LDS and VALU issue together.  CTR and CBC decryption of 2 MiB
// run 11 us a launch here, 14 on the split bitsliced kernel, 28 on the plain
// one.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "internal.h"
#include "keysched_device.h"
#include "spbox_core.h"

namespace tdes {

namespace {

constexpr int kThreads = kTableThreads;

// What block b of a mode puts through the cipher (ECB and CBC: input block b;
// CTR: its counter), and what is XORed into the result (CTR: input block b;
// CBC: the block before, the IV for the first), as little-endian words.
__device__ __forceinline__ uint2 load_block(const uint8_t *in, size_t b) {
    return *reinterpret_cast<const uint2 *>(in + 8 * b);
}
template <int MODE>
__device__ __forceinline__ uint2 cipher_input(const uint8_t *in, const ModeArgs &m, size_t b) {
    if (MODE != kModeCtr) return load_block(in, b);
    const uint64_t c = m.ctr + b;
    return make_uint2(__builtin_bswap32((uint32_t)(c >> 32)), __builtin_bswap32((uint32_t)c));
}
template <int MODE>
__device__ __forceinline__ uint2 xor_input(const uint8_t *in, const ModeArgs &m, size_t b) {
    if (MODE == kModeCtr) return load_block(in, b);
    if (MODE == kModeCbcDec) {
        const uint2 w = load_block(in, b == 0 ? 0 : b - 1);
        return b == 0 ? make_uint2(m.iv0, m.iv1) : w;
    }
    return make_uint2(0, 0);
}

// N blocks, stride blocks apart.
template <int N, int MODE>
__device__ __forceinline__ void blocks(const uint8_t *in, uint8_t *out, const ModeArgs &m, size_t b,
                                       size_t stride, const uint8_t *sp, uint32_t lane,
                                       uint32_t mask, const uint4 *rk) {
    uint2 w[N];
#pragma unroll
    for (int i = 0; i < N; i++) w[i] = cipher_input<MODE>(in, m, b + i * stride);
    cipher_blocks<N>(w, sp, lane, mask, rk);
#pragma unroll
    for (int i = 0; i < N; i++) {
        const uint2 x = xor_input<MODE>(in, m, b + i * stride);
        *reinterpret_cast<uint2 *>(out + 8 * (b + i * stride)) = make_uint2(w[i].x ^ x.x, w[i].y ^ x.y);
    }
}

// The workgroup's tables and round keys; ends with a barrier.
__device__ __forceinline__ void fill_tables_and_keys(uint32_t *table, uint4 *rk,
                                                     const SpboxKeys &keys) {
    fill_tables(table);
    if (threadIdx.x < 48) {
        const int r = threadIdx.x;
        rk[r] = make_uint4(keys.w[r][0], keys.w[r][1], keys.w[r][2], keys.w[r][3]);
    }
    __syncthreads();
}

// `per`: lanes of each workgroup that take blocks (a multiple of 64, at most
// kThreads); all kThreads lanes fill the tables, then the others exit.
// (Requesting a lane's first block before the fill measured no faster:
// 6.1-6.6 us for 64 KiB either way.)
template <int MODE>
__global__ __launch_bounds__(kThreads) void tdes_spbox_kernel(const uint8_t *in, uint8_t *out,
                                                             size_t nblocks, uint32_t per,
                                                             SpboxKeys keys, ModeArgs mode) {
    __shared__ __align__(16) uint32_t table[kTableWords];
    __shared__ uint4 rk[48];
    fill_tables_and_keys(table, rk, keys);
    if (threadIdx.x >= per) return;  // whole waves: per is a multiple of 64
    const uint8_t *sp = reinterpret_cast<const uint8_t *>(table);
    const uint32_t lane = (threadIdx.x % kCopies) * 4u;
    const uint32_t mask = in_vgpr(kIndexMask);

    // Grid-stride over blocks: four at a time while this thread has four,
    // then two, then one.
    const size_t stride = (size_t)gridDim.x * per;
    size_t b = (size_t)blockIdx.x * per + threadIdx.x;
    for (; b + 3 * stride < nblocks; b += 4 * stride)
        blocks<4, MODE>(in, out, mode, b, stride, sp, lane, mask, rk);
    for (; b + stride < nblocks; b += 2 * stride)
        blocks<2, MODE>(in, out, mode, b, stride, sp, lane, mask, rk);
    if (b < nblocks) blocks<1, MODE>(in, out, mode, b, stride, sp, lane, mask, rk);
}

// Small inputs: eight lanes to a block, lane s of them S-box s + 1.  A lane looks
// one word up in a round and three DPP XORs add the eight, so every lane of the
// group has both halves.  A round is a rotate that brings the box's window to bits
// 7..12, one three-input op that keys it and adds the lane's place in the table,
// the read and the XORs; with one block per lane it is 23 operations and eight
// reads, which a lone wave issues one after the other (203 clocks a round).
// Entry v of the table is a row of 32 words, word b SP of S-box b % 8: lane l reads
// word l % 32, free of bank conflicts, and the whole table is 8 KiB.
// Measured (us a launch, back to back, one block per lane -> this): 1 KB 6.4 -> 4.4,
// 64 KiB 6.4 -> 4.5, 256 KiB 7.1 -> 5.4, 384 KiB 6.9 -> 6.8, 512 KiB 7.0 -> 8.1.
// Four lanes to a block: 5.4 at 64 KiB, 6.6 at 384, 7.5 at 512.
constexpr int kGroupThreads = 256;
constexpr int kGroupBlocks = kGroupThreads / 8;  // blocks per workgroup

template <int MODE>
__global__ __launch_bounds__(kGroupThreads) void tdes_spbox_group_kernel(const uint8_t *in,
                                                                        uint8_t *out,
                                                                        size_t nblocks,
                                                                        SpboxKeys keys,
                                                                        ModeArgs mode) {
    __shared__ __align__(16) uint32_t table[64 * kCopies];
    __shared__ uint32_t rk[48 * kCopies];
    const uint32_t tid = threadIdx.x, place = tid % kCopies, box = tid % 8;
    const size_t b = (size_t)blockIdx.x * kGroupBlocks + tid / 8;
    const size_t from = b < nblocks ? b : nblocks - 1;  // (lanes past the end repeat the last block)
    const uint2 w = cipher_input<MODE>(in, mode, from);
    const uint2 x = xor_input<MODE>(in, mode, from);
#pragma unroll
    for (int j = 0; j < 64 * kCopies / 4 / kGroupThreads; j++) {
        const uint32_t c = tid + j * kGroupThreads;  // row c / 8, words 4 (c % 8) ..
        reinterpret_cast<uint4 *>(table)[c] =
            reinterpret_cast<const uint4 *>(SP_BY_CHUNK)[2 * (c / 8) + c % 2];
    }
    // round keys: chunk `box` of round r at bits 7..12, with the lane's place in
    // the table below
    const uint32_t word = box == 7 ? 3u : box == 0 || box == 6 ? 2u : box % 2 ? 0u : 1u;
    const uint32_t sh = box == 7 ? 11u : box == 0 ? 7u : box == 6 ? 15u : 27u - 4u * box;
#pragma unroll
    for (int j = 0; j < 48 * kCopies / kGroupThreads; j++) {
        const uint32_t r = tid / kCopies + j * (kGroupThreads / kCopies);
        rk[r * kCopies + place] = ((keys.w[r][word] >> sh) & 63u) << 7 | 4u * place;
    }
    __syncthreads();
    const uint8_t *sp = reinterpret_cast<const uint8_t *>(table);
    const uint32_t rot = (20u - 4u * box) & 31u;  // window `box` of R down to bits 7..12
    const uint32_t mask = in_vgpr(kIndexMask);
    auto round = [&](uint32_t L, uint32_t R, uint32_t k) {
        // 0x6A: (first & second) ^ third
        const uint32_t a =
            __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_alignbit(R, R, rot), mask, k, 0x6A);
        uint32_t v = *reinterpret_cast<const uint32_t *>(sp + a);
        v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);   // lanes 1 0 3 2
        v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // lanes 2 3 0 1
        return L ^ v ^ (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);  // 7 - l
    };
    uint32_t X, Y;
    SP_IP(w.x, w.y, X, Y);
    const uint32_t *kp = rk + place;
#pragma unroll 1
    for (int pass = 0; pass < 3; pass++, kp += 16 * kCopies) {
        uint32_t k[16];
#pragma unroll
        for (int r = 0; r < 16; r++) k[r] = kp[r * kCopies];
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            X = round(X, Y, k[r]);
            Y = round(Y, X, k[r + 1]);
        }
        const uint32_t t = X;  // R16 || L16
        X = Y;
        Y = t;
    }
    uint32_t o0, o1;
    SP_FP(Y, X, o0, o1);  // (the halves have changed places once more)
    if (box == 0 && b < nblocks)
        *reinterpret_cast<uint2 *>(out + 8 * b) = make_uint2(o0 ^ x.x, o1 ^ x.y);
}

// ECB over device-mapped host memory.  Bound by the PCIe link, which carries
// both directions at once as long as reads and writes are spread evenly over
// the launch: one block per lane and step, one workgroup a CU, and stores that
// do not linger in L2 until the kernel ends (non-temporal).  16 MB in and out:
// 377 us, 450 with plain stores, 549 on the bitsliced kernel, whose waves all
// read, then all write (the copy engines take 337, both directions at once);
// 256 MiB: 48.4 GB/s against 42.7.  Other shapes (256-1024 lanes, 128-512
// workgroups, two adjacent blocks a lane, the next block requested early):
// 368-430 us for 16 MB, none the faster at 256 MiB too.
__global__ __launch_bounds__(kThreads) void tdes_spbox_host_kernel(const uint8_t *in, uint8_t *out,
                                                                  size_t nblocks, uint32_t per,
                                                                  SpboxKeys keys) {
    __shared__ __align__(16) uint32_t table[kTableWords];
    __shared__ uint4 rk[48];
    fill_tables_and_keys(table, rk, keys);
    if (threadIdx.x >= per) return;
    const uint32_t mask = in_vgpr(kIndexMask);
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    for (size_t b = (size_t)blockIdx.x * per + threadIdx.x; b < nblocks; b += (size_t)gridDim.x * per) {
        uint2 w[1] = {load_block(in, b)};
        cipher_blocks<1>(w, reinterpret_cast<const uint8_t *>(table), (threadIdx.x % kCopies) * 4u,
                         mask, rk);
        __builtin_nontemporal_store(v2u{w[0].x, w[0].y}, reinterpret_cast<v2u *>(out + 8 * b));
    }
}

// Several messages, each with its own keys: workgroup g takes up to `per`
// blocks of the message whose workgroup range holds g (one block per
// working lane), after filling its tables and copying that message's round
// keys.  n <= 64, so one ballot over the messages' first workgroups finds
// the message: they do not decrease and the first is 0, so the lanes whose
// entry is at or before g are a prefix, and the last of them is the message
// (an empty message shares its first workgroup with the next one).
__global__ __launch_bounds__(kThreads) void tdes_spbox_multi_kernel(const SpboxMsg *msgs,
                                                                   uint32_t n,
                                                                   const SpboxKeys *keys,
                                                                   uint32_t per) {
    static_assert(kSpboxMultiMax <= 64, "one ballot covers the messages");
    __shared__ __align__(16) uint32_t table[kTableWords];
    __shared__ uint4 rk[48];
    const uint32_t g = blockIdx.x;
    const uint32_t l64 = threadIdx.x % 64;
    const bool le = l64 < n && msgs[l64].first_wg <= g;
    const uint32_t k = (uint32_t)__popcll(__ballot(le));
    const uint32_t m = k > 0 ? k - 1 : 0;  // (k is at least 1 when message 0 starts at 0)
    fill_tables_and_keys(table, rk, keys[m]);
    if (threadIdx.x >= per) return;  // whole waves: per is a multiple of 64
    const SpboxMsg d = msgs[m];
    const uint64_t b = (uint64_t)(g - d.first_wg) * per + threadIdx.x;
    if (g >= d.first_wg && b < d.nblocks)
        blocks<1, kModeEcb>(d.in, d.out, ModeArgs{}, b, 0, reinterpret_cast<const uint8_t *>(table),
                            (threadIdx.x % kCopies) * 4u, in_vgpr(kIndexMask), rk);
}

// What a multi-message launch needs in device memory, from the messages' descriptors
// and raw bundles in host memory, a wave to a message: lane t < 48 makes the table
// kernel's keys of round t, four more copy the descriptor.  (A copy of host-built
// keys took 8 us, and the host 1 us a message to build them.)
constexpr int kPrepareWaves = 4;

__global__ __launch_bounds__(64 * kPrepareWaves) void tdes_spbox_prepare_kernel(
    const SpboxMsg *h_msgs, const uint8_t *h_keys24, uint32_t n, SpboxMsg *msgs, SpboxKeys *keys) {
    const uint32_t lane = threadIdx.x % 64;
    const uint32_t m = blockIdx.x * kPrepareWaves + threadIdx.x / 64;
    if (m >= n) return;
    const uint32_t dir = h_msgs[m].dir & 1u;
    if (lane >= 48) {
        static_assert(sizeof(SpboxMsg) == 32, "four 8-byte words");
        if (lane < 52)
            reinterpret_cast<uint64_t *>(&msgs[m])[lane - 48] =
                reinterpret_cast<const uint64_t *>(&h_msgs[m])[lane - 48];
        return;
    }
    const int slot = round_key_slot((int)dir, (int)lane);
    const SpboxRound k = table_round_keys(load_key(h_keys24 + 24 * m + 8 * (slot / 16), true), slot % 16);
    *reinterpret_cast<uint4 *>(keys[m].w[lane]) = make_uint4(k.w[0], k.w[1], k.w[2], k.w[3]);
}

// Workgroups that fit on the current device at once: 64 KiB of tables per
// workgroup, two in a CU's 160 KiB of LDS.
size_t resident_workgroups() { return 2 * device_cus(); }

}  // namespace

// Cached per device (atomics: first calls from several threads may race;
// they all store the same value).
size_t device_cus() {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cache[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
    int n = cache[dev].load();
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cache[dev].store(n);
    }
    return (size_t)n;
}

size_t spbox_one_pass_bytes() { return resident_workgroups() * kThreads * 8; }

// Few blocks: fewer working lanes per workgroup and more workgroups, so that
// the blocks spread over as many CUs as there are (one workgroup each) rather
// than crowding a few CUs' LDS: the fewest whole waves whose workgroups fit the
// CUs once, at most 1,024 lanes.  (Powers of two before: 1.02 MiB 10.6 -> 8.2 us,
// 1.5 MiB 10.7 -> 8.7, 0.75 MiB 7.2 -> 7.0.)
static uint32_t working_lanes(size_t nblocks) {
    const size_t per_cu = (nblocks + device_cus() - 1) / device_cus();
    return per_cu >= (size_t)kThreads ? (uint32_t)kThreads : (uint32_t)((per_cu + 63) / 64 * 64);
}

hipError_t launch_spbox_host(const SpboxKeys &k, const uint8_t *in, uint8_t *out, size_t nbytes,
                             hipStream_t stream) {
    const size_t nblocks = nbytes / 8;
    const uint32_t per = working_lanes(nblocks);
    size_t grid = (nblocks + per - 1) / per;
    if (grid > device_cus()) grid = device_cus();
    hipLaunchKernelGGL(tdes_spbox_host_kernel, dim3((unsigned)grid), dim3(kThreads), 0, stream, in,
                       out, nblocks, per, k);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_spbox(const SpboxKeys &k, const ModeArgs &m, const uint8_t *in, uint8_t *out,
                        size_t nbytes, hipStream_t stream) {
    const size_t nblocks = nbytes / 8;
    // up to four waves of groups a SIMD (256 KiB on 256 CUs)
    if (nblocks <= 128 * device_cus()) {
        hipLaunchKernelGGL(tdes_spbox_group_kernel<MODE>,
                           dim3((unsigned)((nblocks + kGroupBlocks - 1) / kGroupBlocks)),
                           dim3(kGroupThreads), 0, stream, in, out, nblocks, k, m);
        return hipGetLastError();
    }
    const uint32_t per = working_lanes(nblocks);
    size_t grid = (nblocks + per - 1) / per;
    // Two workgroups per resident slot: the second wave of workgroups fills
    // the slots of those that finish early.
    const size_t cap = 2 * resident_workgroups();
    if (grid > cap) grid = cap;
    hipLaunchKernelGGL(tdes_spbox_kernel<MODE>, dim3((unsigned)grid), dim3(kThreads), 0, stream, in,
                       out, nblocks, per, k, m);
    return hipGetLastError();
}
template hipError_t launch_spbox<kModeEcb>(const SpboxKeys &, const ModeArgs &, const uint8_t *,
                                           uint8_t *, size_t, hipStream_t);
template hipError_t launch_spbox<kModeCtr>(const SpboxKeys &, const ModeArgs &, const uint8_t *,
                                           uint8_t *, size_t, hipStream_t);
template hipError_t launch_spbox<kModeCbcDec>(const SpboxKeys &, const ModeArgs &, const uint8_t *,
                                              uint8_t *, size_t, hipStream_t);

uint32_t spbox_multi_lanes(const uint64_t *nblocks, size_t n) {
    const uint64_t cus = device_cus();
    uint32_t per = 64;
    for (; per < (uint32_t)kThreads; per += 64) {
        uint64_t wgs = 0;
        for (size_t i = 0; i < n; i++) wgs += (nblocks[i] + per - 1) / per;
        if (wgs <= cus) break;
    }
    return per;
}

hipError_t launch_spbox_multi(const SpboxMsg *h_msgs, const uint8_t *h_keys24, SpboxMsg *d_msgs,
                              SpboxKeys *d_keys, uint32_t n, uint32_t per, uint32_t n_wg,
                              hipStream_t stream) {
    if (n == 0 || n > kSpboxMultiMax || n_wg == 0 || per == 0 || per % 64 != 0 ||
        per > (uint32_t)kThreads)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(tdes_spbox_prepare_kernel, dim3((n + kPrepareWaves - 1) / kPrepareWaves),
                       dim3(64 * kPrepareWaves), 0, stream, h_msgs, h_keys24, n, d_msgs, d_keys);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tdes_spbox_multi_kernel, dim3(n_wg), dim3(kThreads), 0, stream, d_msgs, n,
                       d_keys, per);
    return hipGetLastError();
}

}  // namespace tdes
