// Batched 3DES-EDE ECB on the table kernel, for small batches.
//
// One block per lane (spbox.hip), or two or three, interleaved; the blocks of all
// messages in a row, `per` of them to a workgroup and step.  The lanes of the
// bitsliced batch kernel (batch.hip) take 32 blocks each through the rounds, ~36 us
// for the smallest batch.
//
// A workgroup has a CU to itself: 64 KiB of tables, the round keys of up to
// kRows messages (a row each, 784 bytes, padded so that the rows of different
// messages start on different banks) and the messages' first blocks.  Up to
// kTableScanMax messages every workgroup scans the descriptors itself, so a
// batch is one launch (one workgroup more leaves the scan in the workspace);
// beyond, the scan launches of batch.hip come first and the lanes go by its
// slices, 32 to a slice.  The round keys are recovered from the device schedule's mask words by one wave per
// message: lane t the row's entry of round t (make_row).
//
// Bound by the latency of its steps (descriptors, schedules, tables, one block's
// 48 rounds), which a workgroup goes through one after the other: ~10 us for the
// smallest batch, 180 GB/s on large ones.  Measured (us a submit, bitsliced ->
// table): 16 messages of 4 KiB 40 -> 9.4, 300 of 7 KB 36 -> 19.4, 2,000 of 72
// bytes 41 -> 11.7.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "batch_core.h"
#include "generated/bitslice_keys_gen.h"
#include "keysched_core.h"
#include "spbox_core.h"

namespace tdes {

namespace {

constexpr int kThreads = kTableThreads;
constexpr int kWaves = kThreads / kWave;
constexpr uint32_t kRows = 64;      // messages whose round keys are in LDS at once
constexpr uint32_t kRowStride = 49;  // entries (16 bytes) from row to row: 48 rounds and a pad
constexpr int kRowsPerWave = kRows / kWaves;

// What lane t needs of a message's device schedule: round t's two words and the
// extra words 96..98.
struct RowWords {
    uint2 w;
    uint32_t e0, e1, e2;
};

__device__ __forceinline__ RowWords load_row(const tdes_msg &m, const uint32_t *sched,
                                             uint32_t n_sched, uint32_t lane) {
    const uint32_t *p = sched + (size_t)(m.sched_idx < n_sched ? m.sched_idx : 0u) * kDeviceScheduleWords +
                        (m.dir & 1u) * kDirWords;
    RowWords r;
    r.w = reinterpret_cast<const uint2 *>(p)[lane < 48 ? lane : 47];
    r.e0 = p[96];
    r.e1 = p[97];
    r.e2 = p[98];
    return r;
}

// The table kernel's keys of round t = lane.  The schedule's words are masks the
// halves carry (keysched_core.h).  Word 2t holds the change of the mask of the
// half that round t updates, so the mask a half has when round t reads it is the
// XOR of its changes so far, and of the extra words.  In the order of the right
// half's bits that mask is the key at every word's primary expansion position;
// word 2t + 1 holds what its second uses differ by.
__device__ __forceinline__ uint4 make_row(const RowWords &r, uint32_t lane) {
    const bool dx = bs_dest_is_x((int)lane);
    uint32_t x = lane < 48 && dx ? r.w.x : 0u, y = lane < 48 && !dx ? r.w.x : 0u;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t ux = __shfl_up(x, d, kWave), uy = __shfl_up(y, d, kWave);
        if ((int)lane >= d) {
            x ^= ux;
            y ^= uy;
        }
    }
    // (round t's own change is in the half it updates, not the one it reads)
    const uint32_t c = dx ? y : x;
    uint32_t p = __builtin_bitreverse32(dx ? r.e0 ^ (lane >= 32 ? r.e2 : 0u) : lane >= 16 ? r.e1 : 0u);
#pragma unroll
    for (int o = 0; o < 32; o++) p ^= ((c >> o) & 1u) << (31 - kBsOutWord[o]);
    uint32_t odd = p, even = p, w06 = p, w7 = p;
#pragma unroll
    for (int k = 0; k < 16; k++) {
        const int s = kBsDupE[k] / 6;
        const uint32_t b = ((r.w.y >> k) & 1u) << (31 - kBsESrc[kBsDupE[k]]);
        if (s == 7) w7 ^= b;
        else if (s == 0 || s == 6) w06 ^= b;
        else if (s & 1) odd ^= b;
        else even ^= b;
    }
    return make_uint4(odd, even, rotl(w06, 12), rotl(w7, 12));
}

// Exclusive prefix of v over the workgroup's threads; *sum its total.  A barrier
// comes before sums (one word per wave) may be used again.
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t *sums, uint32_t *sum) {
    const uint32_t lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const uint32_t incl = (uint32_t)wave_scan(v, (int)lane);
    if (lane == kWave - 1) sums[wave] = incl;
    __syncthreads();
    uint32_t before = 0, s = 0;
    for (uint32_t w = 0; w < kWaves; w++) {
        before += w < wave ? sums[w] : 0u;
        s += sums[w];
    }
    *sum = s;
    return before + incl - v;
}

// SCAN: the workgroup scans the descriptors itself (n <= kTableScanMax);
// otherwise ws holds their scan.
// NB: blocks a lane takes in a step.
// per: lanes of a step, with SCAN the most of them; least: see below.
template <bool SCAN, int NB>
__global__ __launch_bounds__(kThreads) void batch_table_kernel(const tdes_msg *__restrict__ msgs,
                                                              uint32_t n,
                                                              const uint32_t *__restrict__ sched,
                                                              uint32_t n_sched, const uint8_t *in,
                                                              uint8_t *out, BatchBounds bb,
                                                              uint64_t *ws, uint64_t *skipped_out,
                                                              uint32_t per, uint32_t least) {
    __shared__ __align__(16) uint32_t table[kTableWords];
    __shared__ uint4 rows[kRows * kRowStride];
    // SCAN: first lane of every message (entries past the last: the total).
    // Else first slices of the 1,024 messages after the step's first one, from
    // the step's first slice on.
    __shared__ uint32_t start[SCAN ? kTableScanMax : kThreads];
    __shared__ uint32_t sums[2][kWaves], span[2];
    const uint32_t tid = threadIdx.x, lane = tid % kWave;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint64_t *first = ws + kWsHeader;
    uint32_t grid = gridDim.x;
    uint64_t total;  // lanes of all messages, or of all slices
    if (SCAN) {
        static_assert(kTableScanMax == 2 * kThreads, "two descriptors a thread");
        // A message takes a lane per block, and no fewer than `least`, so that a
        // step's lanes hold kRows messages at most (empty ones aside), one pass of the
        // loop below, however unlike the messages are: a step whose first and last
        // messages are cut has 1 + ceil((per - 1) / least) of them.
        // (batch_is_table bounds the work of so few messages, and a message is no
        // longer than that where outputs overlap: the sums fit 32 bits)
        uint32_t v[2], u[2], bad = 0;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const uint32_t i = 2 * tid + k;
            bool b = false;
            v[k] = (uint32_t)units_of(msgs[i < n ? i : n - 1], n_sched, bb, 8, &b);
            v[k] = i < n ? v[k] : 0u;
            u[k] = (v[k] + kSlice / 8 - 1) / (kSlice / 8);
            v[k] = v[k] == 0 ? 0u : max(v[k], least);
            bad += i < n && b;
        }
        uint32_t sum;
        if (blockIdx.x == --grid) {
            // the last workgroup: the workspace's table, as the scan launches
            // leave it, and the skipped count
            uint32_t skipped;
            block_prefix(bad, sums[0], &skipped);
            const uint32_t f = block_prefix(u[0] + u[1], sums[1], &sum);
            if (2 * tid < n) first[2 * tid] = f;
            if (2 * tid + 1 < n) first[2 * tid + 1] = f + u[0];
            if (tid == 0) {
                ws[0] = first[n] = sum;
                ws[1] = skipped;
                if (skipped_out != nullptr) *skipped_out = skipped;
            }
            return;
        }
        fill_tables(table);
        const uint32_t f = block_prefix(v[0] + v[1], sums[0], &sum);
        start[2 * tid] = f;
        start[2 * tid + 1] = f + v[0];
        total = sum;
        // what there is, evenly over the workgroups: the first multiple of the lanes
        // that NB waves' blocks fill which takes it in one step (the lanes try one each)
        const uint32_t unit = NB * kWave;
        const uint64_t enough = __ballot((lane + 1) * unit * grid >= sum);
        if (enough != 0) per = min(per, (uint32_t)__builtin_ctzll(enough) * unit + unit);
        __syncthreads();
    } else {
        fill_tables(table);
        total = ws[0] * (kSlice / 8);
    }

    const uint8_t *sp = reinterpret_cast<const uint8_t *>(table);
    const uint32_t mask = in_vgpr(kIndexMask);
    for (uint64_t base = (uint64_t)blockIdx.x * per; base < total; base += (uint64_t)grid * per) {
        const uint32_t here = (uint32_t)min((uint64_t)per, total - base);  // lanes of this step
        // this lane's blocks (tid, tid + lanes, ...): their messages, and their
        // places there
        const uint32_t lanes = NB == 1 ? kThreads : per / NB;
        uint32_t m[NB];
        uint64_t at[NB];
        bool active[NB];
#pragma unroll
        for (int k = 0; k < NB; k++) {
            m[k] = 0;
            at[k] = 0;
            active[k] = tid < lanes && tid + k * lanes < here;
        }
        if (SCAN) {
#pragma unroll
            for (uint32_t step = kTableScanMax / 2; step >= 1; step /= 2)
#pragma unroll
                for (int k = 0; k < NB; k++)
                    if (m[k] + step < n && start[m[k] + step] <= (uint32_t)base + tid + k * lanes)
                        m[k] += step;
#pragma unroll
            for (int k = 0; k < NB; k++) at[k] = (uint32_t)base + tid + k * lanes - start[m[k]];
        } else {
            static_assert(SCAN || NB == 1, "lanes by slices take one block");
            const uint64_t s0 = base / (kSlice / 8);
            const uint32_t s = tid / (kSlice / 8);
            const uint32_t m0 = find_message(first, n, s0, lane);
            const uint64_t i = (uint64_t)m0 + 1 + tid;
            const uint64_t rel = i <= n ? first[i] - s0 : ~0ull;
            start[tid] = rel < ~0u ? (uint32_t)rel : ~0u;
            __syncthreads();
            uint32_t r = 0;  // messages that start at or before this lane's slice
#pragma unroll
            for (uint32_t step = kThreads / 2; step >= 1; step /= 2)
                if (start[r + step - 1] <= s) r += step;
            if (start[r] <= s) r++;
            m[0] = m0 + (active[0] ? r : 0u);
            if (active[0]) {
                while (first[m[0] + 1] <= s0 + s) m[0]++;  // past 1,024 messages: many empty ones
                at[0] = (s0 + s - first[m[0]]) * (kSlice / 8) + tid % (kSlice / 8);
            }
        }
#pragma unroll
        for (int k = 0; k < NB; k++) {
            if (k == 0 && tid == 0) span[0] = m[0];
            if (active[k] && tid + k * lanes == here - 1) span[1] = m[k];
        }
        uint2 w[NB] = {};
        uint8_t *dst[NB];
#pragma unroll
        for (int k = 0; k < NB; k++) {
            dst[k] = nullptr;
            if (active[k]) {
                const tdes_msg d = msgs[m[k]];
                // (a message shorter than `least`, or its last slice, leaves lanes idle:
                // they load its last block, so that no load waits for a branch)
                const uint64_t nblk = d.nbytes / 8;
                w[k] = *reinterpret_cast<const uint2 *>(in + d.in_off + 8 * min(at[k], nblk - 1));
                dst[k] = out + d.out_off + 8 * at[k];
                active[k] = at[k] < nblk;
            }
        }
        __syncthreads();
        const uint32_t m_lo = __builtin_amdgcn_readfirstlane(span[0]);
        const uint32_t m_hi = __builtin_amdgcn_readfirstlane(span[1]);
        // kRows messages at a time: their rows, then their lanes' blocks
        for (uint32_t g = m_lo; g <= m_hi; g += kRows) {
            RowWords rw[kRowsPerWave];
#pragma unroll
            for (int k = 0; k < kRowsPerWave; k++)
                rw[k] = load_row(msgs[min(g + wave + k * kWaves, m_hi)], sched, n_sched, lane);
#pragma unroll
            for (int k = 0; k < kRowsPerWave; k++) {
                const uint32_t j = wave + k * kWaves;
                if (g + j > m_hi) break;
                const uint4 row = make_row(rw[k], lane);
                if (lane < 48) rows[j * kRowStride + lane] = row;
            }
            __syncthreads();
            const uint4 *rk[NB];
            bool now[NB];
            bool any = false;
#pragma unroll
            for (int k = 0; k < NB; k++) {
                now[k] = active[k] && m[k] - g < kRows;
                any |= now[k];
                // (a block of another pass runs along, on row 0, and is not stored)
                rk[k] = rows + (now[k] ? m[k] - g : 0u) * kRowStride;
            }
            if (any) {
                uint2 v[NB];
#pragma unroll
                for (int k = 0; k < NB; k++) v[k] = w[k];
                cipher_blocks<NB>(v, sp, (lane % kCopies) * 4u, mask, rk);
#pragma unroll
                for (int k = 0; k < NB; k++)
                    if (now[k]) *reinterpret_cast<uint2 *>(dst[k]) = v[k];
            }
            __syncthreads();
        }
    }
}

}  // namespace

bool batch_is_table(size_t n_msgs, uint64_t work_bytes) {
    // us a submit, this kernel against the bitsliced one (256 CUs, one launch up
    // to kTableScanMax messages): 300 messages in 2.1 MB 20 to 36, in 6 MB 35 to 36,
    // in 7 MiB 52 to 38; 1,000 in 6 MB 36 to 37; 2,000 in 6 MB 37 to 41.  With the scan
    // before it, lanes by slices: 4,000 in 1 MB 22 to 38, in 3 MB 34 to 37; 16,000 of
    // a block 37 to 37.
    if (n_msgs <= kTableScanMax) return work_bytes <= spbox_one_pass_bytes() / 2 * 3;
    return work_bytes + kSlice * (uint64_t)n_msgs <= spbox_one_pass_bytes();
}

hipError_t launch_batch_table(const tdes_msg *msgs, size_t n_msgs, const uint32_t *schedules,
                              size_t n_schedules, const uint8_t *in, uint8_t *out, BatchBounds bb,
                              uint64_t work_bytes, uint64_t *ws, uint64_t *skipped_out,
                              hipStream_t stream) {
    // Blocks per workgroup and step: the work evenly over the CUs, one workgroup
    // each, in as few steps as lanes of up to three blocks allow.  The lookups of a
    // step take LDS time by the block, a step itself ~6 us of dependent loads, so
    // more blocks a lane beat more steps (300 messages: 2.1 MB 21.2 -> 20.1 us, 4
    // MiB 28.4 -> 27.1, 6 MiB 39.8 -> 37.3), and even steps beat full ones with a
    // small last one (2.1 MB 25.5 -> 21.4).  work_bytes only bounds the work, so a
    // kernel that scans divides what it finds.  (Steps sized here, by the mean message
    // and work_bytes, against these: one of 5 MB beside 2,000 of a block, all in one
    // workgroup's step of 32 passes, 482 -> 43 us; 2,048 of a block in a buffer of 6
    // MiB 479 -> 27, 300 of 1,000 bytes there 34 -> 18; even ones up to 2 % slower.)
    // Where lanes go by slices, one block a lane.  Any grid is correct.
    const bool scan = n_msgs <= kTableScanMax;
    // (a scanning kernel's extra workgroup has a CU too: as one more than fit it would
    // start when another ends, 1-1.8 us later)
    const uint64_t cus = scan && device_cus() > 1 ? device_cus() - 1 : device_cus();
    const uint64_t work = work_bytes / 8 + (scan ? 0 : n_msgs * (kSlice / 8));
    const uint64_t cu_work = (work + cus - 1) / cus;
    const uint32_t nb = !scan || cu_work <= kThreads ? 1 : cu_work <= 2 * kThreads ? 2 : 3;
    const uint64_t steps = (cu_work + nb * kThreads - 1) / (nb * kThreads);
    uint64_t per = steps == 0 ? 1 : (cu_work + steps - 1) / steps;
    const uint32_t unit = nb * kWave;
    auto whole = [&](uint64_t v) { return (v + unit - 1) / unit * unit; };
    per = whole(per);
    // (no more workgroups than whole shares fill: one with nothing to do still holds a
    // CU's LDS while it scans, 8-11 % of the rate of two streams)
    uint64_t grid = (work + per - 1) / per;
    grid = grid < 1 ? 1 : grid > cus ? cus : grid;
    // room for the lanes that short messages leave idle, n_msgs x per / (kRows - 1) at
    // most; a step of kRows lanes needs none
    if (scan && per > kRows) {
        const uint64_t room = (kRows - 1) * grid;
        per = whole(per + (room > 2 * n_msgs ? per * n_msgs / (room - n_msgs) : per));
    }
    if (per > (uint64_t)nb * kThreads) per = (uint64_t)nb * kThreads;
    const uint32_t least = per <= kRows ? 1 : (uint32_t)(per + kRows - 2) / (kRows - 1);
    auto launch = [&](auto kernel, uint64_t g) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)g), dim3(kThreads), 0, stream, msgs, (uint32_t)n_msgs,
                           schedules, (uint32_t)n_schedules, in, out, bb, ws, skipped_out, (uint32_t)per, least);
    };
    if (!scan) launch(batch_table_kernel<false, 1>, grid);
    else if (nb == 1) launch(batch_table_kernel<true, 1>, grid + 1);
    else if (nb == 2) launch(batch_table_kernel<true, 2>, grid + 1);
    else launch(batch_table_kernel<true, 3>, grid + 1);
    return hipGetLastError();
}

}  // namespace tdes
