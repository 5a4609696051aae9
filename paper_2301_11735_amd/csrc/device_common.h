// Device helpers shared by the gfx950 kernels of the coupled-pair Metropolis
// sweep (arXiv:2301.11735, section 3.1 update, section 3.2 parallel form):
// table staging, the per-pair step, neighbour sums 16 sites at a time, the
// on-device schedule and block reductions.  Included by the .hip sources only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "philox.h"

namespace lat {
namespace {

constexpr uint32_t kM5 = 0x55555555u;  // bit 0 of every 2-bit field
constexpr uint32_t kM3 = 0x33333333u;  // low 2 bits of every nibble
constexpr uint32_t kM0F = 0x0F0F0F0Fu; // low nibble of every byte

constexpr int charge_c(int c) { return (c & 2) ? 1 - 2 * (c & 1) : 0; }

// Pair states of 8 pairs: nibble u of the result is code_a | code_b << 2 of
// pair 8*half + u, for the aligned (a-word, b-word) couple (A, B).  One byte
// permute gathers (A byte, B byte) pairs, then two swap stages interleave
// their nibbles and 2-bit fields.
__device__ __forceinline__ uint32_t pair_states8(uint32_t A, uint32_t B, int half)
{
    uint32_t x = __builtin_amdgcn_perm(B, A, half ? 0x07030602u : 0x05010400u);
    uint32_t t = (x ^ (x >> 4)) & 0x00F000F0u;
    x ^= t ^ (t << 4);
    t = (x ^ (x >> 2)) & 0x0C0C0C0Cu;
    return x ^ t ^ (t << 2);
}

// Transition table of section 3.1's coupled-pair move with 12 choice slots a
// state, so that the slot depends on the draw alone: slot floor(12 u) holds
// configuration floor(12 u) / 2 = floor(6 u) where k_q = 6, floor(12 u) / 3 =
// floor(4 u) where k_q = 4, and the null move where the pair is frozen.
// Entry 16 x + slot of state x is {coef, C | codes << 16}: coef and C as in
// the host's transition table (dot4(coef, sums) + C is the device-table
// index, at most 932, so a dot4 that accumulates onto the whole word leaves the
// high half alone).
struct TransSlots {
    uint32_t v[2 * 256];
};
constexpr uint32_t trans_i8(int v) { return (uint32_t)(uint8_t)(int8_t)v; }
constexpr void trans_slot(int st, int slot, uint32_t &coef, uint32_t &C, int &a1, int &b1)
{
    constexpr int S[4] = {0, 0, 1, -1}, G[4] = {1, -1, 0, 0};
    constexpr int plus[4] = {2 | 0 << 2, 2 | 1 << 2, 0 | 2 << 2, 1 | 2 << 2};
    constexpr int zero[6] = {2 | 3 << 2, 3 | 2 << 2, 0 | 0 << 2, 1 | 1 << 2, 0 | 1 << 2, 1 | 0 << 2};
    constexpr int minus[4] = {3 | 0 << 2, 3 | 1 << 2, 0 | 3 << 2, 1 | 3 << 2};
    const int ca = st & 3, cb = st >> 2, q = S[ca] + S[cb];
    const int to = q == 0 ? zero[slot / 2] : q == 1 ? plus[slot / 3] : q == -1 ? minus[slot / 3] : st;
    a1 = to & 3;
    b1 = to >> 2;
    const int dSa = S[a1] - S[ca], dSb = S[b1] - S[cb], dGa = G[a1] - G[ca], dGb = G[b1] - G[cb];
    const int nD = S[a1] * S[a1] + S[b1] * S[b1] - S[ca] * S[ca] - S[cb] * S[cb];
    if (dSa == 2 || dSa == -2) {  // charge swap: V line
        coef = trans_i8(dSa) | trans_i8(dSb) << 8;
        C = (uint32_t)(kDevVLine + 16);
    } else if (dGa == 2 || dGa == -2 || dGb == 2 || dGb == -2) {  // spin change: J line
        coef = trans_i8(dGa) << 16 | trans_i8(dGb) << 24;
        C = (uint32_t)(kDevJLine + 16 - 4 * (dGa + dGb));
    } else {
        coef = trans_i8(17 * dSa) | trans_i8(17 * dSb) << 8 | trans_i8(dGa) << 16 | trans_i8(dGb) << 24;
        C = (uint32_t)((nD / 2 + 1) * kDevSlice + 8 * 17 + 8 - 4 * (dGa + dGb));
    }
}
// Byte offset 8 floor(12 (uc >> 8) / 2^24) of the draw's slot.
__device__ __forceinline__ uint32_t slot8_of(uint32_t uc) { return __umulhi(uc & ~255u, 96u) & 0x78u; }

// Word form: x = code_a | code_b << 2, and in the place of the codes the code
// changes d_a * 0x55 | d_b * 0x5500 (d: the XOR of new and old code): each
// 2-bit field of the high half's low byte holds site a's change and of its high
// byte site b's, so that one AND with a field mask places them at any of four
// pair positions.  8 bytes an entry, one ds_read_b64 a pair: the 16-byte
// entries that hold eight positions took twice the LDS cycles.
constexpr TransSlots make_word_slots()
{
    TransSlots t{};
    for (int st = 0; st < 16; ++st)
        for (int slot = 0; slot < 12; ++slot) {
            uint32_t coef = 0, C = 0;
            int a1 = 0, b1 = 0;
            trans_slot(st, slot, coef, C, a1, b1);
            const uint32_t at = 2u * (16u * (uint32_t)st + (uint32_t)slot);
            t.v[at] = coef;
            t.v[at + 1] = C | ((uint32_t)(a1 ^ (st & 3)) * 0x55u | (uint32_t)(b1 ^ (st >> 2)) * 0x5500u) << 16;
        }
    return t;
}
__device__ const TransSlots kWordSlots = make_word_slots();
constexpr int kSlotEntries = 256;

// The tables of the per-phase kernels in two steps: load() issues the loads of
// all that a block of kWordsThreads needs, store() puts them into LDS (and loads
// what smaller blocks still lack), so that a phase's other loads are issued
// in between.
constexpr int kTabAhead = 4;
static_assert(kTabAhead * kWordsThreads >= kDevTabEntries, "the whole table in blocks of kWordsThreads");
struct TableLoads {
    const uint2 *g_tab;
    uint2 tab[kTabAhead], slot;
    __device__ __forceinline__ void load(const uint2 *g, uint32_t threads)
    {
        g_tab = g;
#pragma unroll
        for (int k = 0; k < kTabAhead; ++k) tab[k] = g[min((int)(threadIdx.x + k * threads), kDevTabEntries - 1)];
        slot = ((const uint2 *)kWordSlots.v)[min((int)threadIdx.x, kSlotEntries - 1)];
    }
    __device__ __forceinline__ void store(uint2 *s_tab, uint2 *s_slots, uint32_t threads) const
    {
#pragma unroll
        for (int k = 0; k < kTabAhead; ++k)
            if (threadIdx.x + k * threads < kDevTabEntries) s_tab[threadIdx.x + k * threads] = tab[k];
        if (threadIdx.x < kSlotEntries) s_slots[threadIdx.x] = slot;
        for (int i = threadIdx.x + kTabAhead * threads; i < kDevTabEntries; i += threads) s_tab[i] = g_tab[i];
        for (int i = threadIdx.x + threads; i < kSlotEntries; i += threads) s_slots[i] = ((const uint2 *)kWordSlots.v)[i];
    }
};

// A Philox call as the two pairs' {slot offset, acceptance draw}: the draw is
// compared as min(u, 2^32 - 2) < threshold, so that the reserved "always"
// threshold 2^32 - 1 accepts every draw.
__device__ __forceinline__ u32x4 pair_draws(const u32x4 &w)
{
    return u32x4{slot8_of(w.x), min(w.y, 0xFFFFFFFEu), slot8_of(w.z), min(w.w, 0xFFFFFFFEu)};
}

// One coupled-pair Metropolis step (section 3.1) from the byte offset of its
// transition entry, the packed neighbour sums (sumS_a+4, sumS_b+4, sumsig_a+4,
// sumsig_b+4) and the acceptance draw.  An accepted move adds its packed triple to `packed`
// and ORs its code changes into dacc at `fields` (0x03030000 << 2 (t mod 4) for
// pair t of its word: bytes 2 and 3 collect the changes of the a-sites and the
// b-sites of four pairs).
__device__ __forceinline__ void pair_step_slot(uint32_t entry, uint32_t bpack, uint32_t ua, const uint8_t *s_slots,
                                               const uint2 *s_tab, uint32_t fields, uint32_t &packed, uint32_t &dacc)
{
    const uint2 tr = *(const uint2 *)(s_slots + entry);
    const uint32_t idx = (uint32_t)__builtin_amdgcn_sdot4((int)tr.x, (int)bpack, (int)tr.y, false);
    const uint2 e = *(const uint2 *)((const uint8_t *)s_tab + (uint32_t)(uint16_t)(idx << 3));
    const bool acc = ua < e.x;
    packed += acc ? e.y : 0u;
    dacc |= tr.y & (acc ? fields : 0u);
}

// Per-thread tracker: counts and biased sums of the accepted triples.
__device__ __forceinline__ void unpack_tracker(uint32_t packed, int (&tr)[3])
{
    const int cnt = (int)(packed >> 27);
    tr[0] += (int)((packed >> 20) & 127u) - 2 * cnt;
    tr[1] += (int)((packed >> 10) & 1023u) - 16 * cnt;
    tr[2] += (int)(packed & 1023u) - 16 * cnt;
}

// Wave-wide sum by DPP (row reductions, then row broadcasts 15 and 31): the
// total ends in lane 63 and is returned to every lane.  Every lane of the
// wave must be active.
template <int Ctrl, int RowMask>
__device__ __forceinline__ int dpp_i32(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, Ctrl, RowMask, 0xF, false);
}
template <int Ctrl, int RowMask>
__device__ __forceinline__ long long dpp_i64(long long v)
{
    const int lo = dpp_i32<Ctrl, RowMask>((int)(uint32_t)v), hi = dpp_i32<Ctrl, RowMask>((int)((uint64_t)v >> 32));
    return (long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ int dpp_step_sum(int v)
{
    v += dpp_i32<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
    v += dpp_i32<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
    v += dpp_i32<0x141, 0xF>(v);  // row_half_mirror
    v += dpp_i32<0x140, 0xF>(v);  // row_mirror
    v += dpp_i32<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_i32<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ long long dpp_step_sum(long long v)
{
    v += dpp_i64<0xB1, 0xF>(v);
    v += dpp_i64<0x4E, 0xF>(v);
    v += dpp_i64<0x141, 0xF>(v);
    v += dpp_i64<0x140, 0xF>(v);
    v += dpp_i64<0x142, 0xA>(v);
    v += dpp_i64<0x143, 0xC>(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)((uint64_t)v >> 32), 63);
    return (long long)(((uint64_t)hi << 32) | lo);
}

// Per-wave sums of K values, written to part[wave][*] by lane 0.  Full
// waves (blockDim a multiple of 64, the launch shapes of the sweep kernels)
// reduce by DPP; a partial wave falls back to shuffles.
template <int K, typename T>
__device__ __forceinline__ void wave_partials(T (&v)[K], T (*part)[K])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((blockDim.x & 63u) == 0) {
#pragma unroll
        for (int i = 0; i < K; ++i) v[i] = dpp_step_sum(v[i]);
    } else {
#pragma unroll
        for (int i = 0; i < K; ++i)
            for (int off = 32; off > 0; off >>= 1) v[i] += __shfl_xor(v[i], off, 64);
    }
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < K; ++i) part[wave][i] = v[i];
}

// Block-level sum of K values added to dst[0..K): thread i < K sums value i
// over the block's waves and adds it with one atomic.
template <int K, typename T>
__device__ __forceinline__ void block_reduce_add(T (&v)[K], unsigned long long *dst)
{
    __shared__ T part[16][K];
    wave_partials<K, T>(v, part);
    __syncthreads();
    if (threadIdx.x < K) {
        const int nw = (blockDim.x + 63) >> 6;
        long long s = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w)
            if (w < nw) s += (long long)part[w][threadIdx.x];
        if (s != 0) atomicAdd(&dst[threadIdx.x], (unsigned long long)s);
    }
}

// A wave's sums of the three tracker values, added with one atomic each (no
// block barrier).  Every lane of the wave must be active.
__device__ __forceinline__ void wave_reduce_add3(const int (&v)[3], unsigned long long *dst)
{
    const int v0 = dpp_step_sum(v[0]), v1 = dpp_step_sum(v[1]), v2 = dpp_step_sum(v[2]);
    const int lane = (int)(threadIdx.x & 63u), sum = lane == 0 ? v0 : lane == 1 ? v1 : v2;
    if (lane < 3 && sum != 0) atomicAdd(&dst[lane], (unsigned long long)(long long)sum);
}

// Neighbour contribution of a code c to the packed sums: byte 0 (a side) or
// byte 1 (b side) gets 1+S(c), byte 2 or byte 3 gets 1+sigma(c); the values
// per code are the bytes of kVS = {1,1,2,0} and kVG = {2,0,1,1}.
constexpr uint32_t kVS = 0x00020101u;
constexpr uint32_t kVG = 0x01010002u;
__device__ __forceinline__ uint32_t contrib_a(uint32_t c) { return __builtin_amdgcn_perm(kVG, kVS, 0x0C040C00u + c * 0x00010001u); }
__device__ __forceinline__ uint32_t contrib_b(uint32_t c) { return __builtin_amdgcn_perm(kVG, kVS, 0x040C000Cu + c * 0x01000100u); }

// Schedule of sweep s (same definition as the host's): r in {1,2,3};
// phase p has D_p = (r + 4 m_p, 1 + 2 k_p).  Whole (every lane of every wave is
// active): lanes 0 to 2 draw one of the three calls each (one after another, in
// scalar registers, they are most of a microsecond).  Blocks whose last wave may
// have fewer lanes draw all three in every lane.
template <bool Whole = true>
__device__ __forceinline__ void device_schedule(int L, uint32_t k0, uint32_t k1, uint64_t s, int &r, int (&m)[4],
                                                int (&k)[4])
{
    uint32_t Wd[12];
    if constexpr (Whole) {
        const u32x4 w = philox4x32_10((uint32_t)s, kDomSchedule, threadIdx.x & 3u, (uint32_t)(s >> 32), k0, k1);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            Wd[4 * t] = (uint32_t)__builtin_amdgcn_readlane((int)w.x, t);
            Wd[4 * t + 1] = (uint32_t)__builtin_amdgcn_readlane((int)w.y, t);
            Wd[4 * t + 2] = (uint32_t)__builtin_amdgcn_readlane((int)w.z, t);
            Wd[4 * t + 3] = (uint32_t)__builtin_amdgcn_readlane((int)w.w, t);
        }
    } else {
#pragma unroll
        for (uint32_t t = 0; t < 3u; ++t) {
            const u32x4 w = philox4x32_10((uint32_t)s, kDomSchedule, t, (uint32_t)(s >> 32), k0, k1);
            Wd[4 * t] = w.x;
            Wd[4 * t + 1] = w.y;
            Wd[4 * t + 2] = w.z;
            Wd[4 * t + 3] = w.w;
        }
    }
    r = 1 + (int)(((Wd[0] >> 8) * 3u) >> 24);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        m[p] = (int)mulhi_u32(Wd[1 + 2 * p], (uint32_t)(L / 4));
        k[p] = (int)mulhi_u32(Wd[2 + 2 * p], (uint32_t)(L / 2));
    }
}

// Device-wide barrier between phases of the persistent kernels: every block
// arrives once per phase on a monotonic counter.  Release: every wave fences
// (a wave's fence waits only for its own stores and atomics), so the block's
// results are past the compute unit's caches before its arrival; acquire:
// the fence after the wait invalidates the caches the block reads through.
// The wait is bounded in time (kBarrierTimeoutTicks of the device's
// constant-rate wall clock, 0.2 s at its 100 MHz): then the block raises the
// error flag and goes on (results are then invalid and reported as an
// error), so no wave can spin for long.
__device__ __forceinline__ void grid_barrier(unsigned *counter, unsigned target, unsigned *err)
{
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(counter, 1u);
        const long long t0 = wall_clock64();
        while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(1);
            if (wall_clock64() - t0 > kBarrierTimeoutTicks) {
                atomicOr(err, 1u);
                break;
            }
        }
        __threadfence();
    }
    __syncthreads();
}

// Global memory, said in the type: a pointer that was read from memory (a
// descriptor's state) gets flat accesses otherwise, with 64-bit addresses in
// vector registers and LDS counters to wait for.
#define LAT_GLOBAL __attribute__((address_space(1)))

// Word i of an array below 4 GiB (every lattice state is): a 32-bit byte
// offset from the base, so that a uniform base stays in scalar registers and
// no 64-bit address is formed per access.
__device__ __forceinline__ uint32_t word_at(const uint32_t *base, uint32_t i)
{
    return *(const uint32_t *)((const uint8_t *)base + (i << 2));
}
__device__ __forceinline__ void word_put(uint32_t *base, uint32_t i, uint32_t v)
{
    *(uint32_t *)((uint8_t *)base + (i << 2)) = v;
}

// The two words of the class row at word offset `row` that hold the 16 sites
// starting at class position xs (periodic); alignbit(hi, lo, 2 (xs mod 16))
// then gives the 16 sites (a shift of 0 gives lo).
__device__ __forceinline__ void load_pair(const uint32_t *__restrict__ st, uint32_t row, int W, int xs, uint32_t &lo,
                                          uint32_t &hi)
{
    const int jw = xs >> 4;
    lo = word_at(st, row + (uint32_t)jw);
    hi = word_at(st, row + (uint32_t)(jw + 1 == W ? 0 : jw + 1));
}

// 16 sites of the class row at word offset `row` of `st`, starting at class
// position xs (periodic).  32-bit offsets keep the base pointer uniform.
__device__ __forceinline__ uint32_t load16(const uint32_t *__restrict__ st, uint32_t row, int W, int xs)
{
    const int jw = xs >> 4, sh = xs & 15;
    const uint32_t w0 = word_at(st, row + (uint32_t)jw);
    const uint32_t w1 = word_at(st, row + (uint32_t)(jw + 1 == W ? 0 : jw + 1));
    return sh ? __builtin_amdgcn_alignbit(w1, w0, 2u * (uint32_t)sh) : w0;
}

// Neighbour sums of 16 sites from their 4 neighbour words, SWAR: per code
// the values 1+S in {0,1,2} and 1+sigma in {0,1,2} as 2-bit fields, split
// into even and odd sites so that the 4-term sums (at most 8) fit nibbles.
struct SideSums {
    uint32_t ES, OS, EG, OG;  // nibble u: sum over neighbours of site 2u (E) or 2u+1 (O)
};

// Adds one neighbour word's 16 values to the sums.
__device__ __forceinline__ void side_add(SideSums &s, uint32_t w)
{
    const uint32_t h = (w >> 1) & kM5, l = w & kM5;
    const uint32_t vS = ((h & ~l) << 1) | (h ^ kM5);        // code 2 -> 2, 3 -> 0, spins -> 1
    const uint32_t vG = (((h | l) ^ kM5) << 1) | h;          // code 0 -> 2, 1 -> 0, charges -> 1
    s.ES += vS & kM3;
    s.OS += (vS >> 2) & kM3;
    s.EG += vG & kM3;
    s.OG += (vG >> 2) & kM3;
}

// The sums over all four neighbour words at once, from three indicator
// planes per word (one bit per site, at the low bit of its field): h (a
// charge), P (charge +1) and U (spin +1).  Per site 1+S = 2P + 1 - h and
// 1+sigma = 2U + h, so over the four neighbours
//   4 + sum S = 4 + 2 sum P - sum h,   4 + sum sigma = 2 sum U + sum h.
// Two words' planes add without carry in 2-bit fields (at most 2); the two
// pair sums are then split into even and odd sites and added in nibbles (at
// most 4), and the nibble combinations stay within 0..8.
__device__ __forceinline__ SideSums side_sums(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    uint32_t h[4], P[4], U[4];
    const uint32_t w[4] = {w0, w1, w2, w3};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[i] = (w[i] >> 1) & kM5;
        P[i] = h[i] & ~w[i];
        U[i] = ~(h[i] | w[i]) & kM5;
    }
    const uint32_t h01 = h[0] + h[1], h23 = h[2] + h[3];
    const uint32_t P01 = P[0] + P[1], P23 = P[2] + P[3];
    const uint32_t U01 = U[0] + U[1], U23 = U[2] + U[3];
    const uint32_t hE = (h01 & kM3) + (h23 & kM3), hO = ((h01 >> 2) & kM3) + ((h23 >> 2) & kM3);
    const uint32_t PE = (P01 & kM3) + (P23 & kM3), PO = ((P01 >> 2) & kM3) + ((P23 >> 2) & kM3);
    const uint32_t UE = (U01 & kM3) + (U23 & kM3), UO = ((U01 >> 2) & kM3) + ((U23 >> 2) & kM3);
    constexpr uint32_t kFour = 0x44444444u;  // 4 in every nibble
    return SideSums{kFour + 2u * PE - hE, kFour + 2u * PO - hO, 2u * UE + hE, 2u * UO + hO};
}

// 4x4 byte transpose: out[k] = (r0.byte k, r1.byte k, r2.byte k, r3.byte k).
__device__ __forceinline__ void transpose4(uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3, uint32_t &c0,
                                           uint32_t &c1, uint32_t &c2, uint32_t &c3)
{
    const uint32_t p01lo = __builtin_amdgcn_perm(r1, r0, 0x05010400u);
    const uint32_t p01hi = __builtin_amdgcn_perm(r1, r0, 0x07030602u);
    const uint32_t p23lo = __builtin_amdgcn_perm(r3, r2, 0x05010400u);
    const uint32_t p23hi = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
    c0 = __builtin_amdgcn_perm(p23lo, p01lo, 0x05040100u);
    c1 = __builtin_amdgcn_perm(p23lo, p01lo, 0x07060302u);
    c2 = __builtin_amdgcn_perm(p23hi, p01hi, 0x05040100u);
    c3 = __builtin_amdgcn_perm(p23hi, p01hi, 0x07060302u);
}

// (r0.byte k, r1.byte k, r2.byte k, r3.byte k) with sel = k | (4 + k) << 8 | 0x0C0C0000.
__device__ __forceinline__ uint32_t gather_byte(uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3, uint32_t sel)
{
    const uint32_t lo = __builtin_amdgcn_perm(r1, r0, sel);
    const uint32_t hi = __builtin_amdgcn_perm(r3, r2, sel);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// Observable sums: sum S, sum S^2, bonds S S, bonds sigma sigma, sum sigma,
// staggered sigma, staggered S.  Bonds (x,y)-(x+1,y) and (x,y)-(x,y+1).
__device__ __forceinline__ int spin_of(uint32_t c) { return (c & 2u) ? 0 : 1 - 2 * (int)(c & 1u); }
__device__ __forceinline__ int charge_of(uint32_t c) { return (c & 2u) ? 1 - 2 * (int)(c & 1u) : 0; }

// Observable sums of int8 lattices, four sites (one word) at a time, from
// bytes (1 + S) | (1 + sigma) << 4.  With u = 1 + S and g = 1 + sigma:
// sum S S' over the 2N bonds is sum u u' - 4 sum u + 2N (every site is in
// four bonds), sum S^2 is sum u^2 - 2 sum u + N, and the offsets cancel in the
// staggered sums.
constexpr uint32_t kSiteBytes = 0x21u | 0x01u << 8 | 0x12u << 16 | 0x10u << 24;  // per code
__device__ __forceinline__ uint32_t site_from_codes(uint32_t c) { return __builtin_amdgcn_perm(0u, kSiteBytes, c); }

// Staggered signs of four sites x = 4X .. 4X + 3 of row y.
__device__ __forceinline__ int row_signs(uint32_t y) { return (int)((y & 1u) ? 0x01FF01FFu : 0xFF01FF01u); }

struct SiteSums {
    uint32_t su = 0, sg = 0, suu = 0, bu = 0, bg = 0, cnt = 0;
    int stu = 0, stg = 0;

    // w: four sites; wr, wd: their right and lower neighbours; sign: the
    // sites' staggered signs, a byte each.
    __device__ __forceinline__ void add(uint32_t w, uint32_t wr, uint32_t wd, int sign)
    {
        const uint32_t m4 = 0x0F0F0F0Fu, ones = 0x01010101u;
        const uint32_t u = w & m4, g = (w >> 4) & m4;
        su = __builtin_amdgcn_udot4(u, ones, su, false);
        sg = __builtin_amdgcn_udot4(g, ones, sg, false);
        suu = __builtin_amdgcn_udot4(u, u, suu, false);
        bu = __builtin_amdgcn_udot4(u, wr & m4, bu, false);
        bu = __builtin_amdgcn_udot4(u, wd & m4, bu, false);
        bg = __builtin_amdgcn_udot4(g, (wr >> 4) & m4, bg, false);
        bg = __builtin_amdgcn_udot4(g, (wd >> 4) & m4, bg, false);
        stu = __builtin_amdgcn_sdot4((int)u, sign, stu, false);
        stg = __builtin_amdgcn_sdot4((int)g, sign, stg, false);
        cnt += 4u;
    }
    // the seven sums of what was added (below 2^28 sites a thread)
    template <typename T>
    __device__ __forceinline__ void get(T (&v)[7]) const
    {
        v[0] = (T)((int)su - (int)cnt);
        v[1] = (T)((int)suu - 2 * (int)su + (int)cnt);
        v[2] = (T)((int)bu - 4 * (int)su + 2 * (int)cnt);
        v[3] = (T)((int)bg - 4 * (int)sg + 2 * (int)cnt);
        v[4] = (T)((int)sg - (int)cnt);
        v[5] = (T)stg;
        v[6] = (T)stu;
    }
};

// A word of codes at any byte address (a caller may place an int8 state
// anywhere), and NW of them (NW = 4: 16-byte aligned).
typedef uint32_t word_any __attribute__((aligned(1)));
template <int NW>
__device__ __forceinline__ void load_codes(const uint8_t *p, uint32_t (&w)[NW])
{
    if constexpr (NW == 4) {
        const uint4 v = *(const uint4 *)p;
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
    } else {
        w[0] = *(const word_any *)p;
    }
}

// Adds group t (NW words of a row) of an int8 lattice.
template <int NW>
__device__ __forceinline__ void obs_group_int8(const uint8_t *st, uint32_t L, uint32_t t, SiteSums &s)
{
    const uint32_t Lq = L >> 2, per_row = Lq / NW, y = t / per_row, X = (t - y * per_row) * NW;
    const uint32_t row = y * L;  // N <= 2^30
    uint32_t c[NW], d[NW];
    load_codes<NW>(st + row + 4u * X, c);
    load_codes<NW>(st + (y + 1 == L ? 0u : row + L) + 4u * X, d);
    const uint32_t after = *(const word_any *)(st + row + (X + NW == Lq ? 0u : 4u * (X + NW)));
    uint32_t e[NW + 1];
#pragma unroll
    for (int i = 0; i < NW; ++i) e[i] = site_from_codes(c[i]);
    e[NW] = site_from_codes(after);
#pragma unroll
    for (int i = 0; i < NW; ++i)
        s.add(e[i], __builtin_amdgcn_alignbit(e[i + 1], e[i], 8u), site_from_codes(d[i]), row_signs(y));
}

// Block-level sum of K values written (not added) to dst[0..K): no atomics.
template <int K, typename T>
__device__ __forceinline__ void block_reduce_store(T (&v)[K], long long *dst)
{
    __shared__ T part[16][K];
    wave_partials<K, T>(v, part);
    __syncthreads();
    if (threadIdx.x < K) {
        const int nw = (blockDim.x + 63) >> 6;
        long long s = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w)
            if (w < nw) s += (long long)part[w][threadIdx.x];
        dst[threadIdx.x] = s;
    }
}

// Bond sums of 16 sites (h, l bit planes) with 16 partner sites (hp, lp):
// S S = +1 for equal charges, -1 for opposite; sigma sigma likewise for spins.
__device__ __forceinline__ void bond_sums(uint32_t h, uint32_t l, uint32_t hp, uint32_t lp, int &bSS, int &bss)
{
    const uint32_t diff = l ^ lp;
    const uint32_t cc = h & hp, mm = (h | hp) ^ kM5;  // both charged / both spins
    bSS += __popc(cc & ~diff) - __popc(cc & diff);
    bss += __popc(mm & ~diff) - __popc(mm & diff);
}

}  // namespace
}  // namespace lat
