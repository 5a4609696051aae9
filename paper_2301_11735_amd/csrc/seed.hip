// gfx950 seeded initial state (arXiv:2301.11735 section 3.1, stage 1): site i
// gets the key (w0 << 32 | w1) of Philox counter (0, 0x200, i, 0); the N+ sites
// with the smallest (key, i) become +1, the next N- become -1, the others are
// spins with sigma from bit 0 of w2.
//
// The two sets are fixed by the elements of rank N+ and N+ + N- in the order of
// (key, i).  They are found without storing or sorting the keys, which are
// drawn again in every pass: a histogram of the keys' upper 11 bits, one of
// the next 11 bits within each rank's bin, and the few elements of the bins
// that are then left (N / 2^22 on average, 256 for the largest lattice), whose
// ranks the last pass counts before it writes the codes.  Should a bin hold more
// than kSeedCap elements, the caller is told, and seeds on the host.
//
// What bounds it: the launches for small lattices, four Philox calls a site
// for large ones.  A lattice made, tables and copies included, with the host's
// keys and selection and with these passes (ms): L = 16 0.15 and 0.10, L = 128
// 0.40 and 0.09, L = 512 2.8 and 0.09, L = 2048 50 and 0.12, L = 8192 825 and 0.46; a
// served burst of 40 requests 126 and 89 in one run.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_common.h"

namespace lat {
namespace {

constexpr uint32_t kSeedBins = 2048, kSeedThreads = 256;
static_assert(kSeedBins == 8 * kSeedThreads, "find_bin's share of a thread");

struct SeedCand {
    uint32_t hi, lo, i;
};
// Where it all is in the lattice's scratch, in regions that hold nothing yet.
struct SeedSpace {
    uint32_t *hist[3];  // the upper 11 bits; the next 11 in the bin of rank 0 and of rank 1
    SeedCand *cand[2];
    uint32_t *found;  // [2]
};
static_assert(kScrSlots + 3 * kSeedBins * 4 <= kScrFullTab, "the histograms fit the tracker slots");
static_assert(kScrObsSlots + 2 * kSeedCap * sizeof(SeedCand) + 8 <= kScrSlots, "the candidates fit the observable slots");
__device__ __forceinline__ SeedSpace seed_space(uint8_t *scr)
{
    SeedSpace s;
    for (int k = 0; k < 3; ++k) s.hist[k] = (uint32_t *)(scr + kScrSlots) + k * kSeedBins;
    for (int k = 0; k < 2; ++k) s.cand[k] = (SeedCand *)(scr + kScrObsSlots) + k * kSeedCap;
    s.found = (uint32_t *)(s.cand[0] + 2 * kSeedCap);
    return s;
}

__device__ __forceinline__ u32x4 seed_draw(const SeedArgs &a, uint32_t i)
{
    return philox4x32_10(0u, kDomInit, i, 0u, a.key0, a.key1);
}

// The bin that holds the element of rank r (the block's threads together), and
// its rank within the bin; kNoBin if there are not that many elements.
constexpr uint32_t kNoBin = 0xFFFFFFFFu;
struct SeedBin {
    uint32_t bin, rest;
};
__device__ SeedBin find_bin(const uint32_t *hist, uint32_t r)
{
    __shared__ uint32_t part[kSeedThreads];
    __shared__ SeedBin found;
    const uint32_t t = threadIdx.x;
    uint32_t n[8], sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) sum += n[k] = hist[8 * t + k];
    if (t == 0) found = {kNoBin, 0u};
    part[t] = sum;
    __syncthreads();
    for (uint32_t d = 1; d < kSeedThreads; d *= 2) {
        const uint32_t v = t >= d ? part[t - d] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    uint32_t before = part[t] - sum;
    if (r >= before && r - before < sum) {
        uint32_t bin = 8 * t;
#pragma unroll
        for (int k = 0; k < 7; ++k)
            if (bin == 8 * t + k && r - before >= n[k]) before += n[k], ++bin;
        found = {bin, r - before};
    }
    __syncthreads();
    const SeedBin out = found;
    __syncthreads();
    return out;
}

__global__ void __launch_bounds__(kSeedThreads) k_seed_clear(SeedArgs a)
{
    const SeedSpace s = seed_space(a.scratch);
    const uint32_t i = blockIdx.x * kSeedThreads + threadIdx.x;
    if (i < 3 * kSeedBins) s.hist[0][i] = 0u;
    if (i < 2) s.found[i] = 0u;
}

__global__ void __launch_bounds__(kSeedThreads) k_seed_upper(SeedArgs a)
{
    __shared__ uint32_t h[kSeedBins];
    const SeedSpace s = seed_space(a.scratch);
    for (uint32_t i = threadIdx.x; i < kSeedBins; i += kSeedThreads) h[i] = 0u;
    __syncthreads();
    for (uint32_t i = blockIdx.x * kSeedThreads + threadIdx.x; i < a.sites; i += gridDim.x * kSeedThreads)
        atomicAdd(&h[seed_draw(a, i).x >> 21], 1u);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kSeedBins; i += kSeedThreads)
        if (h[i]) atomicAdd(&s.hist[0][i], h[i]);
}

__global__ void __launch_bounds__(kSeedThreads) k_seed_next(SeedArgs a)
{
    const SeedSpace s = seed_space(a.scratch);
    const uint32_t b0 = find_bin(s.hist[0], a.rank[0]).bin, b1 = find_bin(s.hist[0], a.rank[1]).bin;
    for (uint32_t i = blockIdx.x * kSeedThreads + threadIdx.x; i < a.sites; i += gridDim.x * kSeedThreads) {
        const uint32_t hi = seed_draw(a, i).x;
        if (hi >> 21 == b0) atomicAdd(&s.hist[1][hi >> 10 & 2047u], 1u);
        if (hi >> 21 == b1) atomicAdd(&s.hist[2][hi >> 10 & 2047u], 1u);
    }
}

// The upper 22 bits at each rank (kNoBin: no such element), and the rank among
// the elements that share them.
__device__ __forceinline__ void find_prefixes(const SeedArgs &a, const SeedSpace &s, SeedBin (&p)[2])
{
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const SeedBin u = find_bin(s.hist[0], a.rank[k]);
        const SeedBin v = find_bin(s.hist[1 + k], u.rest);
        p[k] = u.bin == kNoBin ? u : SeedBin{u.bin << 11 | v.bin, v.rest};
    }
}

__global__ void __launch_bounds__(kSeedThreads) k_seed_gather(SeedArgs a)
{
    const SeedSpace s = seed_space(a.scratch);
    SeedBin p[2];
    find_prefixes(a, s, p);
    for (uint32_t i = blockIdx.x * kSeedThreads + threadIdx.x; i < a.sites; i += gridDim.x * kSeedThreads) {
        const u32x4 w = seed_draw(a, i);
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (w.x >> 10 == p[k].bin) {
                const uint32_t at = atomicAdd(&s.found[k], 1u);
                if (at < a.cap) s.cand[k][at] = {w.x, w.y, i};
            }
    }
}

__device__ __forceinline__ bool seed_less(uint32_t hi, uint32_t lo, uint32_t i, const SeedCand &b)
{
    const uint64_t x = (uint64_t)hi << 32 | lo, y = (uint64_t)b.hi << 32 | b.lo;
    return x < y || (x == y && i < b.i);
}

__global__ void __launch_bounds__(kSeedThreads) k_seed_write(SeedArgs a)
{
    __shared__ SeedCand s_at[2];  // the elements of the two ranks
    const SeedSpace s = seed_space(a.scratch);
    SeedBin p[2];
    find_prefixes(a, s, p);
    if (threadIdx.x < 2) s_at[threadIdx.x] = {~0u, ~0u, ~0u};  // every element is before it
    __syncthreads();
    bool over = false;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (p[k].bin == kNoBin) continue;
        const uint32_t all = s.found[k], n = min(all, a.cap);
        over = over || all > a.cap;
        for (uint32_t j = threadIdx.x; j < n; j += kSeedThreads) {
            const SeedCand c = s.cand[k][j];
            uint32_t rank = 0;
            for (uint32_t m = 0; m < n; ++m) {
                const SeedCand o = s.cand[k][m];
                rank += seed_less(o.hi, o.lo, o.i, c) ? 1u : 0u;
            }
            if (rank == p[k].rest) s_at[k] = c;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.overflow = over ? 1u : 0u;
    __syncthreads();
    const SeedCand plus = s_at[0], charged = s_at[1];
    auto code = [&](uint32_t i) -> uint32_t {
        const u32x4 w = seed_draw(a, i);
        return seed_less(w.x, w.y, i, plus) ? 2u : seed_less(w.x, w.y, i, charged) ? 3u : w.z & 1u;
    };
    const uint32_t first = blockIdx.x * kSeedThreads + threadIdx.x, step = gridDim.x * kSeedThreads, L = a.L;
    if (a.enc == 0) {
        for (uint32_t t = first; t < a.sites / 4u; t += step) {
            uint32_t w = 0;
#pragma unroll
            for (uint32_t x = 0; x < 4u; ++x) w |= code(4u * t + x) << (8u * x);
            ((word_any *)a.state)[t] = w;
        }
    } else {
        const uint32_t W = L >> 6, H = L >> 1;
        for (uint32_t t = first; t < a.sites / 16u; t += step) {
            const uint32_t row = t / W, j = t - row * W, c = row / H, Y = row - c * H;
            const uint32_t i0 = (2u * Y + (c >> 2)) * L + 64u * j + (c & 3u);
            uint32_t w = 0;
            for (uint32_t X = 0; X < 16u; ++X) w |= code(i0 + 4u * X) << (2u * X);
            ((uint32_t *)a.state)[t] = w;
        }
    }
}

uint32_t seed_blocks(uint32_t sites, uint32_t per_block)
{
    return std::min(1024u, std::max(1u, sites / per_block));
}

}  // namespace

hipError_t launch_seed(const SeedArgs &a, hipStream_t s)
{
    const dim3 block(kSeedThreads), clear(3 * kSeedBins / kSeedThreads);
    const dim3 upper(seed_blocks(a.sites, 8192)), pass(seed_blocks(a.sites, 1024));
    hipLaunchKernelGGL(k_seed_clear, clear, block, 0, s, a);
    hipLaunchKernelGGL(k_seed_upper, upper, block, 0, s, a);
    hipLaunchKernelGGL(k_seed_next, pass, block, 0, s, a);
    hipLaunchKernelGGL(k_seed_gather, pass, block, 0, s, a);
    hipLaunchKernelGGL(k_seed_write, pass, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace lat
