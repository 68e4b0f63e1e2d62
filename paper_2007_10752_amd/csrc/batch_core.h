// What the batched kernels share: the descriptor checks, the workspace layout
// and the choice between them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace tdes {

constexpr int kWave = 64;

// Work unit of the bitsliced kernel: a lane's 32 blocks.
constexpr uint32_t kSlice = 256;
// Workspace words: [0] total slices, [1] skipped messages, [2 + i] first slice of
// message i (i = 0..n; entry n = total).
constexpr int kWsHeader = 2;

// Buffer sizes a batch's message ranges are checked against.
struct BatchBounds {
    uint64_t in_bytes, out_bytes;
};

// Units (slices or blocks) of a message, 0 if it is invalid.
__device__ __forceinline__ uint64_t units_of(const tdes_msg &m, size_t n_sched, BatchBounds bb,
                                             uint32_t unit, bool *bad) {
    // bitwise, not short-circuit, so that no field is read under a branch;
    // in_bytes - nbytes may wrap, but only where nbytes <= in_bytes fails
    const bool ok = (((m.nbytes | m.in_off | m.out_off) % 8) == 0) & (m.sched_idx < n_sched) &
                    (m.dir <= 1) & (m.nbytes <= bb.in_bytes) &
                    (m.in_off <= bb.in_bytes - m.nbytes) & (m.nbytes <= bb.out_bytes) &
                    (m.out_off <= bb.out_bytes - m.nbytes);
    *bad = !ok;
    return ok ? (m.nbytes + unit - 1) / unit : 0;
}

// Inclusive scan of v over the 64 lanes of a wave.
__device__ __forceinline__ uint64_t wave_scan(uint64_t v, int lane) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint64_t u = __shfl_up(v, d, kWave);
        if (lane >= d) v += u;
    }
    return v;
}

// Message holding slice `base`: the largest m with first[m] <= base, for a wave
// (first[] is non-decreasing, first[n] > base).  A 64-way search: each step
// every lane tests one evenly spaced entry and a ballot keeps the sub-range, so
// 16k messages take 3 steps.
__device__ __forceinline__ uint32_t find_message(const uint64_t *first, uint32_t n, uint64_t base,
                                                 uint32_t lane) {
    uint32_t lo = 0, hi = n;  // first[lo] <= base < first[hi]
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint64_t idx = lo + (uint64_t)(lane + 1) * step;
        const bool le = idx < hi && first[idx] <= base;
        const uint32_t k = (uint32_t)__popcll(__ballot(le));  // a prefix of lanes
        const uint64_t nhi = lo + (uint64_t)(k + 1) * step;
        lo = lo + k * step;
        hi = nhi < hi ? (uint32_t)nhi : hi;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// Most messages the batched table kernel scans by itself.
constexpr uint32_t kTableScanMax = 2048;
// Whether a batch of n_msgs messages with at most work_bytes in all runs on the
// table kernel.
bool batch_is_table(size_t n_msgs, uint64_t work_bytes);
// The batched table kernel.  For more than kTableScanMax messages ws holds the
// descriptor scan; for fewer the kernel makes it.  work_bytes sizes the grid.
hipError_t launch_batch_table(const tdes_msg *msgs, size_t n_msgs, const uint32_t *schedules,
                              size_t n_schedules, const uint8_t *in, uint8_t *out, BatchBounds bb,
                              uint64_t work_bytes, uint64_t *ws, uint64_t *skipped_out,
                              hipStream_t stream);

}  // namespace tdes
