// gfx950 observable reduction of one lattice (sum S, sum S^2, bond sums,
// magnetisations; arXiv:2301.11735 section 2.1 energy terms) and the fold of
// the per-block partial sums into the totals.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_common.h"
#include "onchip.h"
#include "word_task.h"

namespace lat {
namespace {

__global__ void k_zero_i64(unsigned long long *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// Bound by the reads (16 bytes a load in the NW = 4 form, for sides that are
// a multiple of 16 on an aligned state).  L = 4096: 9.5 us
// (37 us with three byte loads a site).
template <int NW>
__global__ void __launch_bounds__(1024) k_obs_int8(const uint8_t *__restrict__ st, int L, long long *slots)
{
    SiteSums sums;
    const uint32_t n = (uint32_t)L * (uint32_t)L / (4u * NW);
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x)
        obs_group_int8<NW>(st, (uint32_t)L, t, sums);
    long long v[7];
    sums.get(v);
    block_reduce_store<7>(v, slots + 7 * (size_t)blockIdx.x);
}

__global__ void __launch_bounds__(1024) k_obs_2bit(const uint32_t *__restrict__ st, int L, long long *slots)
{
    long long v[7] = {0, 0, 0, 0, 0, 0, 0};
    const uint32_t nwords = (uint32_t)L * (uint32_t)L / 16u;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += gridDim.x * blockDim.x)
        obs_word_2bit(st, (uint32_t)L, i, v);
    block_reduce_store<7>(v, slots + 7 * (size_t)blockIdx.x);
}

// Totals of one lattice: tracker = base triple + every tracker slot;
// observables = the first n_obs observable slots.  Written to dst (tracker,
// then the 7 sums) and, with stamp, dst[10] = the lattice's next sweep index.  Four
// waves: sixteen have more partial sums to wait for (4.7 us against 3.2).
constexpr int kFoldThreads = 256;
__global__ void __launch_bounds__(kFoldThreads) k_fold_sums(uint8_t *scr, int n_obs, long long *dst, int stamp)
{
    long long t[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    long long t3[3] = {0, 0, 0};
    tracker_partial(scr, t3);
#pragma unroll
    for (int k = 0; k < 3; ++k) t[k] = t3[k];
    const long long *os = (const long long *)(scr + kScrObsSlots);
    for (int i = threadIdx.x; i < n_obs; i += blockDim.x)
#pragma unroll
        for (int k = 0; k < 7; ++k) t[3 + k] += os[7 * i + k];
    block_reduce_store<10>(t, dst);
    if (stamp && threadIdx.x == 0) dst[10] = (long long)((const LatDesc *)(scr + kScrDesc))->next_sweep;
}

// Observables and tracker of a small lattice in one launch of one block
// (k_obs_* and k_fold_sums together): a launch and the gap before it cost more
// than the block's few passes over at most kOneBlockUnits groups of 16 sites (or
// 4).  One sweep and its observables, with the two launches and one: L = 32
// 48.6 -> 37.8 us (ten sweeps), L = 256 2-bit 51.8 -> 43.4 us.
constexpr uint32_t kOneBlockUnits = 8192;
__global__ void __launch_bounds__(1024) k_obs_one(uint8_t *scr, const uint8_t *st, int L, int enc, int wide,
                                                  long long *dst, int stamp)
{
    long long t[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    long long v[7] = {0, 0, 0, 0, 0, 0, 0};
    const uint32_t N = (uint32_t)L * (uint32_t)L;
    long long t3[3] = {0, 0, 0};
    tracker_partial(scr, t3);
#pragma unroll
    for (int k = 0; k < 3; ++k) t[k] = t3[k];
    if (enc != 0) {
        for (uint32_t i = threadIdx.x; i < N / 16u; i += blockDim.x) obs_word_2bit((const uint32_t *)st, (uint32_t)L, i, v);
    } else {
        SiteSums sums;
        if (wide)
            for (uint32_t i = threadIdx.x; i < N / 16u; i += blockDim.x) obs_group_int8<4>(st, (uint32_t)L, i, sums);
        else
            for (uint32_t i = threadIdx.x; i < N / 4u; i += blockDim.x) obs_group_int8<1>(st, (uint32_t)L, i, sums);
        sums.get(v);
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) t[3 + k] = v[k];
    block_reduce_store<10>(t, dst);
    if (stamp && threadIdx.x == 0) dst[10] = (long long)((const LatDesc *)(scr + kScrDesc))->next_sweep;
}

// The error flags of a batch's lattices (one thread each) in one word.
static_assert(kMaxBatch <= 256, "a thread a lattice");
__global__ void __launch_bounds__(256) k_gather_flags(BatchArgs a, uint32_t *out)
{
    __shared__ uint32_t all;
    if (threadIdx.x == 0) all = 0u;
    __syncthreads();
    if ((int)threadIdx.x < a.count) {
        const uint32_t flags = *(const uint32_t *)(a.scratch[threadIdx.x] + kScrErr);
        if (flags) atomicOr(&all, flags);
    }
    __syncthreads();
    if (threadIdx.x == 0) *out = all;
}

}  // namespace

hipError_t launch_zero_i64(unsigned long long *p, int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_i64, dim3((n + 63) / 64), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_gather_flags(const BatchArgs &a, uint32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_gather_flags, dim3(1), dim3(256), 0, s, a, out);
    return hipGetLastError();
}

hipError_t launch_observables(uint8_t *scratch, const void *state, int L, int encoding, hipStream_t s,
                              long long *record)
{
    const bool wide = encoding == 0 && L % 16 == 0 && ((uintptr_t)state & 15u) == 0;
    const uint32_t units = (uint32_t)L * L / (encoding == 0 && !wide ? 4u : 16u);
    long long *dst = record ? record : (long long *)(scratch + kScrTrack);
    if (units <= kOneBlockUnits) {
        hipLaunchKernelGGL(k_obs_one, dim3(1), dim3(1024), 0, s, scratch, (const uint8_t *)state, L, encoding, wide ? 1 : 0,
                           dst, record ? 1 : 0);
        return hipGetLastError();
    }
    uint32_t grid = (units + 1023u) / 1024u;
    if (grid > (uint32_t)kMaxObsSlots) grid = (uint32_t)kMaxObsSlots;
    long long *slots = (long long *)(scratch + kScrObsSlots);
    if (encoding == 0 && wide)
        hipLaunchKernelGGL(k_obs_int8<4>, dim3(grid), dim3(1024), 0, s, (const uint8_t *)state, L, slots);
    else if (encoding == 0)
        hipLaunchKernelGGL(k_obs_int8<1>, dim3(grid), dim3(1024), 0, s, (const uint8_t *)state, L, slots);
    else
        hipLaunchKernelGGL(k_obs_2bit, dim3(grid), dim3(1024), 0, s, (const uint32_t *)state, L, slots);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fold_sums, dim3(1), dim3(kFoldThreads), 0, s, scratch, (int)grid, dst, record ? 1 : 0);
    return hipGetLastError();
}

}  // namespace lat
