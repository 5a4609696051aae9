// Parts shared by the on-chip kernels that keep one byte per site in LDS
// (batch.hip: k_sweep_site, quad.hip: k_sweep_quad): site bytes, the schedule
// words made ahead, and the records of a launch over several observation
// intervals.  Included by the .hip sources only.
#pragma once

#include "device_common.h"

namespace lat {
namespace {

constexpr uint32_t site_byte(int code) { return (kSiteBytes >> (8 * code)) & 0xFFu; }

// Four site bytes to four codes (one a byte).
__device__ __forceinline__ uint32_t codes_from_site(uint32_t e)
{
    const uint32_t one = 0x01010101u;
    return ((e >> 3) & (one << 1)) | (~((e >> 5) | (e >> 1)) & one);  // charged; sigma = -1 or S = -1
}

// Schedules of up to kSchedSweeps sweeps from s on, one Philox call (4 of a
// sweep's 12 words) a thread: r, then m_p and k_p of the four phases.
constexpr uint32_t kSchedSweeps = 16;
__device__ __forceinline__ void make_schedules(uint32_t *sched, uint64_t s, uint32_t sweeps, uint32_t key0,
                                               uint32_t key1, uint32_t L)
{
    const uint32_t t = threadIdx.x;
    if (t >= 3u * min(kSchedSweeps, sweeps)) return;
    const uint64_t q = s + t / 3u;
    const u32x4 w = philox4x32_10((uint32_t)q, kDomSchedule, t % 3u, (uint32_t)(q >> 32), key0, key1);
    sched[4u * t] = t % 3u == 0u ? 1u + (((w.x >> 8) * 3u) >> 24) : mulhi_u32(w.x, L >> 1);
    sched[4u * t + 1u] = mulhi_u32(w.y, L >> 2);
    sched[4u * t + 2u] = mulhi_u32(w.z, L >> 1);
    sched[4u * t + 3u] = mulhi_u32(w.w, L >> 2);
}
// A sweep's schedule on its way to scalar registers: loaded a phase before it is
// needed.
struct SweepLoads {
    uint32_t w[9];
};
__device__ __forceinline__ SweepLoads sweep_loads(const uint32_t *sched)
{
    SweepLoads v;
#pragma unroll
    for (int i = 0; i < 9; ++i) v.w[i] = sched[i];
    return v;
}
struct SweepWords {
    uint32_t r, m[4], k[4];
};
__device__ __forceinline__ SweepWords sweep_words(const SweepLoads &v)
{
    uint32_t w[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) w[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)v.w[i]);
    return SweepWords{w[0], {w[1], w[3], w[5], w[7]}, {w[2], w[4], w[6], w[8]}};
}

// This thread's share of a lattice's tracker slots (phase kernels) and, for
// thread 0, its tracker base (single-block kernels).
__device__ __forceinline__ void tracker_partial(const uint8_t *scr, long long (&t3)[3])
{
    const long long *slots = (const long long *)(scr + kScrSlots);
    for (int i = threadIdx.x; i < kMaxSlots; i += blockDim.x) {
        t3[0] += slots[3 * i];
        t3[1] += slots[3 * i + 1];
        t3[2] += slots[3 * i + 2];
    }
    if (threadIdx.x == 0) {
        const long long *base = (const long long *)(scr + kScrTrackBase);
        t3[0] += base[0];
        t3[1] += base[1];
        t3[2] += base[2];
    }
}

// Records written by a sweep kernel itself: the tracker total before the
// launch, and the waves' sums.
struct ObsStage {
    long long base[3];
    int part[16][10];
};
__device__ __forceinline__ void tracker_before(const uint8_t *scr, ObsStage &o)
{
    long long t3[3] = {0, 0, 0};
    tracker_partial(scr, t3);
    block_reduce_store<3>(t3, o.base);
}
// Record k of this block's lattice from the threads' tracker moves since the
// launch began and shares of the seven sums.  Every wave has read the lattice
// before the barrier in here, and there are four more before the next record.
__device__ __forceinline__ void write_record(const BatchArgs &args, ObsStage &o, const int (&tr)[3], const int (&sums)[7],
                                             uint32_t k, uint64_t next_sweep)
{
    int v[10] = {tr[0], tr[1], tr[2], sums[0], sums[1], sums[2], sums[3], sums[4], sums[5], sums[6]};
    wave_partials<10, int>(v, o.part);
    __syncthreads();
    unsigned long long *rec = args.obs_out + (size_t)args.obs_stride * k + (size_t)args.obs_words * blockIdx.x;
    if (threadIdx.x < 10) {
        long long sum = threadIdx.x < 3 ? o.base[threadIdx.x] : 0ll;
        for (uint32_t w = 0; w < blockDim.x >> 6; ++w) sum += (long long)o.part[w][threadIdx.x];
        rec[threadIdx.x] = (unsigned long long)sum;
    }
    if (args.obs_words > 10 && threadIdx.x == 0) rec[10] = next_sweep;
}

}  // namespace
}  // namespace lat
