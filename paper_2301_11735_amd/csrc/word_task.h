// One a-word of a phase of the coupled-pair sweep (arXiv:2301.11735, section
// 3.1 update, section 3.2 parallel form), 16 pairs computed by Q cooperating
// lanes, on a lattice in the 2-bit class layout in global memory, for the
// multi-block kernels; their device-wide barrier; and the observable sums of a
// class word.  Included by the .hip sources only.
#pragma once

#include "device_common.h"

namespace lat {
namespace {

// Word-parallel form, for lattices with L % 64 == 0 in the 2-bit class
// layout (W = L/64 words per class row): a phase is computed 16 sites at a
// time as in the single-lattice phase kernel.  The 16 pairs of an a-word are
// split among Q threads (Q = 1, 2, 4 or 8, chosen per launch by its lattices):
// thread q of a word takes the Philox calls that call_of_task lists, i.e. sites
// 2c and 2c+1 of each.
//
// Within a phase no updated site neighbours another updated site, so every
// neighbour word read is constant during the phase.  The a-word belongs to the
// lanes of one word, whose first lane stores it; the two b-words are shared with
// another word's lanes in bit fields that each of them neither reads nor writes
// of the other, and their changes are applied as xor atomics.

struct WordPhase {
    uint32_t oA0, oAL, oAR, oAV, oB0, oBL, oBR, oBV;  // class offsets (words)
    int W, H, Lq, dX, k, p, pb;
    uint32_t magicW;                                 // ceil(2^32 / W)
    uint32_t s_lo, s_hi, key0, key1;
};

// Lattice word accessors.  Coh = false: ordinary loads and stores (the
// lattice in LDS, or in global memory within one launch, whose end makes the
// writes visible).  Coh = true: loads and stores at device coherence, which
// no compute unit's or die's cache keeps stale, for the persistent kernels
// whose blocks exchange lattice words across device-wide barriers without
// cache write-back or invalidation.  Read-modify-writes are device-scope
// atomics in both cases.
template <bool Coh>
__device__ __forceinline__ uint32_t ldw(const uint32_t *p, uint32_t i)
{
    if constexpr (Coh)
        // a 32-bit byte offset from the uniform base: no 64-bit address per access
        return __hip_atomic_load((const LAT_GLOBAL uint32_t *)((const LAT_GLOBAL uint8_t *)p + (i << 2)), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
    else
        return p[i];
}
template <bool Coh>
__device__ __forceinline__ void stw(uint32_t *p, uint32_t i, uint32_t v)
{
    if constexpr (Coh)
        __hip_atomic_store((LAT_GLOBAL uint32_t *)((LAT_GLOBAL uint8_t *)p + (i << 2)), v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    else
        p[i] = v;
}
// XOR into a word of a lattice in global memory.
__device__ __forceinline__ void xorw(uint32_t *p, uint32_t i, uint32_t v)
{
    (void)__hip_atomic_fetch_xor((LAT_GLOBAL uint32_t *)((LAT_GLOBAL uint8_t *)p + (i << 2)), v, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
}
// Device-wide barrier for kernels whose lattice words are all accessed at
// device coherence (ldw/stw<true> and device-scope atomics), in two halves.
// Arrive: every wave waits for its own memory operations to complete, the
// block meets, and one thread arrives on the monotonic counter.  Wait: that
// thread waits for the others, and the block meets again.  No cache
// write-back or invalidation is needed.  Between the halves a block may do
// work that touches no lattice word.  The wait is bounded as in grid_barrier
// (time-out flag, then go on), by `limit` ticks of the device wall clock; a block
// that has given up waits no more.
//
// The first meeting of a launch (arrive, then assemble in the place of wait)
// comes before any block touches the lattice.  Nothing guarantees that all blocks
// get a place while kernels of other streams hold compute units: blocks that have
// waited for the others longer than their limit call the launch off, all of its
// blocks end without having changed anything, and a second launch, a block a
// lattice, then does the work (alone()).  Either all blocks of a lattice go on or
// none does: the common counter holds kCalledOff or reaches its full count, never
// both.
//
// Up to kFlatBarrierBlocks blocks meet on one counter.  More meet in two
// levels: block b arrives on the counter of group b % 8 (blocks go to the
// eight XCDs in turn, so a group shares an L2), the last of a group on the
// common counter, and the last of all releases every group by its own flag.
// Every block's increments at one address cost 15 ns each; measured per
// barrier with 32 / 64 / 128 / 256 blocks: one counter 1.1 / 1.4 / 2.1 / 3.8
// us, two levels 1.6 / 1.65 / 1.75 / 1.95 us.
constexpr unsigned kFlatBarrierBlocks = 64, kBarrierGroups = 8, kBarrierLine = 32;  // words apart: 128 bytes
constexpr unsigned kBarrierWords = (1 + 3 * kBarrierGroups) * kBarrierLine;
constexpr unsigned kCalledOff = 0x80000000u;  // counts stay below it
struct GridBarrier {
    unsigned *words;  // the common counter, the group counters, the group flags, the group sums, a line each
    unsigned block, blocks;  // this block's number among those that meet
    unsigned rounds;         // barriers arrived at so far
    bool gave_up;
    __device__ __forceinline__ static unsigned load(const unsigned *p)
    {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ static void store(unsigned *p, unsigned v)
    {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ unsigned *group() const { return words + kBarrierLine * (1u + block % kBarrierGroups); }
    __device__ __forceinline__ unsigned *flag(unsigned g) const { return words + kBarrierLine * (1u + kBarrierGroups + g); }
    // six running sums of the group's blocks (series records)
    __device__ __forceinline__ unsigned long long *sums() const
    {
        return (unsigned long long *)(words + kBarrierLine * (1u + 2u * kBarrierGroups + block % kBarrierGroups));
    }
    __device__ __forceinline__ bool flat() const { return blocks <= kFlatBarrierBlocks; }

    // True in the thread that completed its group (two levels only): until its
    // block arrives again, no other block of the group passes the barrier
    // after this one.
    __device__ __forceinline__ bool arrive()
    {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        ++rounds;
        bool last = false;
        if (threadIdx.x == 0) {
            if (flat()) {
                __hip_atomic_fetch_add(words, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const unsigned g = block % kBarrierGroups;
                const unsigned mates = (blocks + kBarrierGroups - 1u - g) / kBarrierGroups;
                last = __hip_atomic_fetch_add(group(), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == mates * rounds;
                if (last && __hip_atomic_fetch_add(words, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
                                kBarrierGroups * rounds)
                    for (unsigned k = 0; k < kBarrierGroups; ++k) store(flag(k), rounds);
            }
        }
        return last;
    }
    __device__ __forceinline__ void wait(unsigned *err, long long limit)
    {
        if (threadIdx.x == 0 && !gave_up) {
            const unsigned *at = flat() ? words : flag(block % kBarrierGroups);
            const unsigned target = flat() ? blocks * rounds : rounds;
            const long long t0 = wall_clock64();
            // (no time at all is up at once, also where everyone has arrived)
            while (limit <= 0 || load(at) < target) {
                __builtin_amdgcn_s_sleep(1);
                if (wall_clock64() - t0 > limit || limit <= 0) {
                    atomicOr(err, 1u);
                    gave_up = true;
                    break;
                }
            }
        }
        __syncthreads();
    }

    // One thread: calls the launch off unless all have arrived at its first
    // meeting.  True if it is called off.
    __device__ bool call_off()
    {
        const unsigned all = flat() ? blocks : kBarrierGroups;
        unsigned n = load(words);
        while (n < all) {
            if (__hip_atomic_compare_exchange_strong(words, &n, n | kCalledOff, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT)) {
                for (unsigned k = 0; k < kBarrierGroups && !flat(); ++k) store(flag(k), kCalledOff);
                return true;
            }
        }
        return (n & kCalledOff) != 0;
    }
    // The first meeting's arrival (limit: assemble's); true.
    __device__ __forceinline__ bool first_arrive(long long limit)
    {
        // (no time at all: before block 0 has arrived, so that it is certain)
        if (limit <= 0 && block == 0 && threadIdx.x == 0) call_off();
        arrive();
        return true;
    }
    // False, for the whole block, if the launch is called off.
    __device__ __forceinline__ bool assemble(bool is_alone, long long limit)
    {
        __shared__ unsigned s_off;
        if (threadIdx.x == 0) {
            const unsigned *at = flat() ? words : flag(block % kBarrierGroups);
            const unsigned target = flat() ? blocks : 1u;
            const long long t0 = wall_clock64();
            unsigned n = 0u;
            while (!is_alone && (n = load(at)) < target) {  // kCalledOff is above any target
                __builtin_amdgcn_s_sleep(1);
                if (wall_clock64() - t0 > limit) {
                    n = call_off() ? kCalledOff : 0u;
                    break;
                }
            }
            s_off = n & kCalledOff;
        }
        __syncthreads();
        return s_off == 0u;
    }
    // A launch of one block a lattice behind the one that may have been called
    // off: true if it was, and the counter then stands as after this block's
    // arrival at the first meeting.
    __device__ __forceinline__ bool alone()
    {
        const bool off = (load(words) & kCalledOff) != 0;
        __syncthreads();
        if (threadIdx.x == 0 && off) store(words, 1u);
        return off;
    }
};

// The fields of WordPhase for phase p of a sweep with schedule (r, m, k), on
// a lattice of side L with key (key0, key1); s is the sweep index.
__device__ __forceinline__ void word_phase_setup(WordPhase &f, int L, uint32_t key0, uint32_t key1, uint64_t s,
                                                 int p, int r, const int (&mm)[4], const int (&kk)[4])
{
    f.W = L >> 6;
    f.H = L >> 1;
    f.Lq = L >> 2;
    f.magicW = f.W == 1 ? 0u : (uint32_t)((0x100000000ull + (uint64_t)f.W - 1u) / (uint64_t)f.W);
    f.key0 = key0;
    f.key1 = key1;
    f.s_lo = (uint32_t)s;
    f.s_hi = (uint32_t)(s >> 32);
    const uint32_t csz = (uint32_t)f.H * (uint32_t)f.W;
    f.k = kk[p];
    f.p = p;
    f.pb = (p + r) & 3;
    const int carry = (p + r) >> 2;
    f.dX = mm[p] + carry >= f.Lq ? mm[p] + carry - f.Lq : mm[p] + carry;
    f.oA0 = (uint32_t)p * csz;
    f.oAL = (uint32_t)(p > 0 ? p - 1 : 3) * csz;
    f.oAR = (uint32_t)(p < 3 ? p + 1 : 0) * csz;
    f.oAV = (uint32_t)(4 + p) * csz;
    f.oB0 = (uint32_t)(4 + f.pb) * csz;
    f.oBL = (uint32_t)(f.pb > 0 ? 4 + f.pb - 1 : 7) * csz;
    f.oBR = (uint32_t)(f.pb < 3 ? 4 + f.pb + 1 : 4) * csz;
    f.oBV = (uint32_t)f.pb * csz;
}

// Sum of the charges S and of the spins sigma of the 16 sites of a class
// word (2-bit codes: 0 sigma = +1, 1 sigma = -1, 2 S = +1, 3 S = -1).
__device__ __forceinline__ int charge_sum16(uint32_t w)
{
    const uint32_t h = (w >> 1) & kM5, l = w & kM5;
    return __popc(h & ~l) - __popc(h & l);
}
__device__ __forceinline__ int spin_sum16(uint32_t w)
{
    const uint32_t h = (w >> 1) & kM5, l = w & kM5;
    return __popc((h | l) ^ kM5) - __popc(l & ~h);
}

// Observable sums of class word i (16 sites) of a lattice of side L in the
// 2-bit class layout: sum S, sum S^2, the S S and sigma sigma bonds to the
// right and lower neighbours, sum sigma, and the staggered sums.  The right
// neighbours are the same word of the next class (or class 0 of the row,
// one site on), the lower ones the same word of the paired row class.
__device__ __forceinline__ void obs_word_2bit(const uint32_t *__restrict__ st, uint32_t L, uint32_t i, long long (&v)[7])
{
    const uint32_t W = L >> 6, H = L >> 1, Lq = L >> 2, csz = H * W;
    const uint32_t c = i / csz, rem = i - c * csz;
    const uint32_t Y = rem / W, j = rem - Y * W;
    const uint32_t cx = c & 3u, cy = c >> 2;
    const uint32_t w = st[i];
    const uint32_t wr = cx < 3 ? st[i + csz] : load16(st, 4u * cy * csz + Y * W, (int)W, 16 * j + 1 == Lq ? 0 : (int)(16 * j + 1));
    const uint32_t wd = cy == 0 ? st[i + 4 * csz] : st[cx * csz + (Y + 1 == H ? 0 : Y + 1) * W + j];
    const uint32_t h = (w >> 1) & kM5, l = w & kM5;
    const int sumS = charge_sum16(w);
    const int sumG = spin_sum16(w);
    int bSS = 0, bss = 0;
    bond_sums(h, l, (wr >> 1) & kM5, wr & kM5, bSS, bss);
    bond_sums(h, l, (wd >> 1) & kM5, wd & kM5, bSS, bss);
    const int sg = ((cx + cy) & 1) ? -1 : 1;
    v[0] += sumS;
    v[1] += __popc(h);
    v[2] += bSS;
    v[3] += bss;
    v[4] += sumG;
    v[5] += sg * sumG;
    v[6] += sg * sumS;
}

// Value of the lane XOR lanes away (quad permutes), or, with XOR = 4, of the
// other quad of eight lanes, for values that are the same in a whole quad
// (the half-row mirror: no LDS permute).
template <int XOR>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    constexpr int ctrl = XOR == 1 ? 0xB1 : XOR == 2 ? 0x4E : 0x141;  // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xF, 0xF, false);
}

// Philox calls a task makes: all 8 of its word (Q = 1) or 8/Q of them.  The
// i-th is call_of_task(q, i), in the order word_task uses them.
template <int Q>
constexpr int kTaskCalls = Q == 1 ? 8 : 8 / Q;
template <int Q>
__device__ __forceinline__ int call_of_task(int q, int i)
{
    if constexpr (Q == 1) return i < 4 ? 2 * i : 2 * (i - 4) + 1;
    else if constexpr (Q == 2) return 2 * i + q;
    else return 2 * ((q >> 1) + 2 * i) + (q & 1);
}

// First counter word of a task's word (its a-word's first Philox call): the
// same in every phase, since each phase's a-class has the same shape.
template <int Q>
__device__ __forceinline__ uint32_t task_call0(const WordPhase &f, uint32_t task)
{
    constexpr int LOGQ = Q == 1 ? 0 : Q == 2 ? 1 : Q == 4 ? 2 : 3;
    const uint32_t wi = task >> LOGQ;
    const int Y = f.W == 1 ? (int)wi : (int)__umulhi(wi, f.magicW), j = (int)wi - Y * f.W;
    return (uint32_t)Y * (uint32_t)(f.Lq >> 1) + 8u * (uint32_t)j;
}

// Changes of 16 pairs' codes from a task's accumulators, as words of 2-bit
// fields of the a-sites and of the b-sites.
template <int Q>
__device__ __forceinline__ void task_changes(const uint32_t (&dacc)[Q <= 2 ? 4 : 8 / Q], int q, uint32_t &dA,
                                             uint32_t &dB)
{
    if constexpr (Q <= 2) {
        dA = __builtin_amdgcn_perm(__builtin_amdgcn_perm(dacc[3], dacc[2], 0x0C0C0602u),
                                   __builtin_amdgcn_perm(dacc[1], dacc[0], 0x0C0C0602u), 0x05040100u);
        dB = __builtin_amdgcn_perm(__builtin_amdgcn_perm(dacc[3], dacc[2], 0x0C0C0703u),
                                   __builtin_amdgcn_perm(dacc[1], dacc[0], 0x0C0C0703u), 0x05040100u);
    } else {
        const uint32_t last = Q == 4 ? dacc[8 / Q - 1] : 0u;
        dA = __builtin_amdgcn_perm(last, dacc[0], 0x0C060C02u) << (8 * (q >> 1));
        dB = __builtin_amdgcn_perm(last, dacc[0], 0x0C070C03u) << (8 * (q >> 1));
    }
}

// The neighbour sums of a word's a-sites (sa) and b-sites (sb) from the
// words its Q lanes hold: lane q has words q (8 / Q) .. of (left, right, up,
// down of the a-word, the same of the b-word).  The lanes' partial sums are
// additive and fit nibbles; the two sides are then exchanged.
template <int Q>
__device__ __forceinline__ void combine_sides(const uint32_t (&n)[8 / Q], int q, SideSums &sa, SideSums &sb)
{
    if constexpr (Q == 1) {
        sa = side_sums(n[0], n[1], n[2], n[3]);
        sb = side_sums(n[4], n[5], n[6], n[7]);
    } else {
        SideSums full{0u, 0u, 0u, 0u}, other;
        if constexpr (Q == 2) {
            full = side_sums(n[0], n[1], n[2], n[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 8 / Q; ++i) side_add(full, n[i]);
            full.ES += lane_xor<1>(full.ES);
            full.OS += lane_xor<1>(full.OS);
            full.EG += lane_xor<1>(full.EG);
            full.OG += lane_xor<1>(full.OG);
        }
        if constexpr (Q == 8) {
            full.ES += lane_xor<2>(full.ES);
            full.OS += lane_xor<2>(full.OS);
            full.EG += lane_xor<2>(full.EG);
            full.OG += lane_xor<2>(full.OG);
        }
        other.ES = lane_xor<Q / 2>(full.ES);
        other.OS = lane_xor<Q / 2>(full.OS);
        other.EG = lane_xor<Q / 2>(full.EG);
        other.OG = lane_xor<Q / 2>(full.OG);
        const bool side = q >= Q / 2;
        sa = side ? other : full;
        sb = side ? full : other;
    }
}

// The pair steps of a task on its words A0 and B0 (aligned) and their
// neighbour sums: draw(i, c) gives Philox call c of the word, the task's i-th,
// as pair_draws.
template <int Q, typename F>
__device__ __forceinline__ void task_steps(uint32_t A0, uint32_t B0, const SideSums &sa, const SideSums &sb, int q,
                                           const uint2 *s_tab, const uint8_t *s_slots, uint32_t &packed,
                                           uint32_t (&dacc)[Q <= 2 ? 4 : 8 / Q], F draw)
{
    auto do_call = [&](int i, int c, uint32_t be, uint32_t bo, uint32_t &d) {
        const u32x4 w = draw(i, c);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int t = 2 * c + h;
            const uint32_t entry =
                (((A0 >> (2 * t)) & 3u) << 7) | (((B0 >> (2 * t)) & 3u) << 9) | (h ? w.z : w.x);
            pair_step_slot(entry, h ? bo : be, h ? w.w : w.y, s_slots, s_tab, 0x03030000u << (2 * (t & 3)), packed, d);
        }
    };
    if constexpr (Q <= 2) {
#pragma unroll
        for (int hh = 0; hh < (Q == 1 ? 2 : 1); ++hh) {
            const int half = Q == 1 ? hh : q;
            const int sh = 4 * half;
            uint32_t ge[4], go[4];
            transpose4((sa.ES >> sh) & kM0F, (sb.ES >> sh) & kM0F, (sa.EG >> sh) & kM0F, (sb.EG >> sh) & kM0F,
                       ge[0], ge[1], ge[2], ge[3]);
            transpose4((sa.OS >> sh) & kM0F, (sb.OS >> sh) & kM0F, (sa.OG >> sh) & kM0F, (sb.OG >> sh) & kM0F,
                       go[0], go[1], go[2], go[3]);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {  // pairs 4kk .. 4kk+3
                const int slot = Q == 1 ? 4 * hh + kk : kk;
                do_call(slot, 2 * kk + half, ge[kk], go[kk], dacc[kk]);
            }
        }
    } else {
        const int half = q & 1, sh = 4 * half;
        const uint32_t rES0 = (sa.ES >> sh) & kM0F, rES1 = (sb.ES >> sh) & kM0F;
        const uint32_t rEG0 = (sa.EG >> sh) & kM0F, rEG1 = (sb.EG >> sh) & kM0F;
        const uint32_t rOS0 = (sa.OS >> sh) & kM0F, rOS1 = (sb.OS >> sh) & kM0F;
        const uint32_t rOG0 = (sa.OG >> sh) & kM0F, rOG1 = (sb.OG >> sh) & kM0F;
#pragma unroll
        for (int i = 0; i < 8 / Q; ++i) {  // pairs of group kk
            const uint32_t kk = (uint32_t)(q >> 1) + 2u * (uint32_t)i;
            const uint32_t sel = kk | ((4u + kk) << 8) | 0x0C0C0000u;
            do_call(i, 2 * (int)kk + half, gather_byte(rES0, rES1, rEG0, rEG1, sel),
                    gather_byte(rOS0, rOS1, rOG0, rOG1, sel), dacc[i]);
        }
    }
}

// A task, in three parts, so that a
// persistent kernel can do the first before its device-wide barrier and issue
// all loads at once after it:
//   word_refs   where its words are (nothing of the lattice is read),
//   word_fetch  the loads,
//   word_apply  the pair steps and the stores.
// The Q lanes of a word OR their code changes together (their fields are
// disjoint), then the word's first lane stores the a-word, which no other
// word reads or writes in the phase, and applies the two b-word changes as
// atomics.  Every lane of a word must be active.
// Coh: the words are read and written at device coherence (ldw/stw<true>).
// Both words that cover 16 sites are always loaded: skipping the second where
// the run starts on a word boundary put a branch and a wait before the next
// load, and at L = 1024 a phase is a chain of latencies.
template <int Q>
struct WordRefs {
    uint32_t a0, blo, bhi;                       // word indices of the a-word and of the two b-words
    uint32_t lo[8 / Q], hi[8 / Q], sh[8 / Q];    // of this lane's neighbour words, and their shifts (bits)
};
template <int Q>
struct WordVals {
    uint32_t a0, blo, bhi, lo[8 / Q], hi[8 / Q];
};

template <int Q>
__device__ __forceinline__ WordRefs<Q> word_refs(const WordPhase &f, uint32_t task)
{
    constexpr int LOGQ = Q == 1 ? 0 : Q == 2 ? 1 : Q == 4 ? 2 : 3;
    const uint32_t wi = task >> LOGQ;
    const int q = (int)(task & (uint32_t)(Q - 1));
    const int W = f.W, H = f.H, Lq = f.Lq;
    const int Y = W == 1 ? (int)wi : (int)__umulhi(wi, f.magicW), j = (int)wi - Y * W;
    int Xb = 16 * j + f.dX;
    if (Xb >= Lq) Xb -= Lq;
    const int Yb = Y + f.k >= H ? Y + f.k - H : Y + f.k;
    const uint32_t ro = (uint32_t)Y * W, rob = (uint32_t)Yb * W;
    const uint32_t roU = (uint32_t)(Y == 0 ? H - 1 : Y - 1) * W;
    const uint32_t robD = (uint32_t)(Yb + 1 == H ? 0 : Yb + 1) * W;
    const int xAL = f.p > 0 ? 16 * j : (j == 0 ? Lq - 1 : 16 * j - 1);
    const int xAR = f.p < 3 ? 16 * j : 16 * j + 1;
    const int xBL = f.pb > 0 ? Xb : (Xb == 0 ? Lq - 1 : Xb - 1);
    const int xBR = f.pb < 3 ? Xb : (Xb + 1 == Lq ? 0 : Xb + 1);
    const uint32_t row[8] = {f.oAL + ro,  f.oAR + ro,  f.oAV + roU, f.oAV + ro,
                             f.oBL + rob, f.oBR + rob, f.oBV + rob, f.oBV + robD};
    const int x[8] = {xAL, xAR, 16 * j, 16 * j, xBL, xBR, Xb, Xb};
    WordRefs<Q> r;
    const int jb = Xb >> 4;
    r.a0 = f.oA0 + ro + (uint32_t)j;
    r.blo = f.oB0 + rob + (uint32_t)jb;
    r.bhi = f.oB0 + rob + (uint32_t)(jb + 1 == W ? 0 : jb + 1);
#pragma unroll
    for (int i = 0; i < 8 / Q; ++i) {
        // neighbour word q (8 / Q) + i, picked by the bits of q
        uint32_t rw = 0;
        int xw = 0;
#pragma unroll
        for (int n = i; n < 8; n += 8 / Q)
            if (Q == 1 || n / (8 / Q) == 0 || q == n / (8 / Q)) {
                rw = row[n];
                xw = x[n];
            }
        const int jw = xw >> 4;
        r.lo[i] = rw + (uint32_t)jw;
        r.hi[i] = rw + (uint32_t)(jw + 1 == W ? 0 : jw + 1);
        r.sh[i] = 2u * (uint32_t)(xw & 15);
    }
    return r;
}

template <int Q, bool Coh>
__device__ __forceinline__ WordVals<Q> word_fetch(const uint32_t *lat, const WordRefs<Q> &r)
{
    WordVals<Q> v;
    v.a0 = ldw<Coh>(lat, r.a0);
    v.blo = ldw<Coh>(lat, r.blo);
    v.bhi = ldw<Coh>(lat, r.bhi);
#pragma unroll
    for (int i = 0; i < 8 / Q; ++i) {
        v.lo[i] = ldw<Coh>(lat, r.lo[i]);
        v.hi[i] = ldw<Coh>(lat, r.hi[i]);
    }
    return v;
}

// Returns the packed triples of the accepted moves (for unpack_tracker).
// Obs: the word's first lane also adds the changes of the spin sum, the
// staggered spin sum and the staggered charge sum over the word's a-sites and
// b-sites to dv[0..2] (the other observable sums are the tracker's: the
// charged-site count and the two bond sums change by exactly the accepted
// energy-change triples, and the charge sum does not change).
template <int Q, bool Coh, bool Obs>
__device__ __forceinline__ uint32_t word_apply(uint32_t *lat, const WordPhase &f, const WordRefs<Q> &r,
                                               const WordVals<Q> &v, int q, const u32x4 *draws, const uint2 *s_tab,
                                               const uint8_t *s_slots, int *dv)
{
    const uint32_t shb = 2u * (uint32_t)(f.dX & 15);  // Xb mod 16 is the same for every word
    const uint32_t A0 = v.a0, B0 = __builtin_amdgcn_alignbit(v.bhi, v.blo, shb);
    uint32_t n[8 / Q];
#pragma unroll
    for (int i = 0; i < 8 / Q; ++i) n[i] = __builtin_amdgcn_alignbit(v.hi[i], v.lo[i], r.sh[i]);
    SideSums sa, sb;
    combine_sides<Q>(n, q, sa, sb);
    uint32_t dacc[Q <= 2 ? 4 : 8 / Q] = {}, packed = 0u, cA, cB;
    task_steps<Q>(A0, B0, sa, sb, q, s_tab, s_slots, packed, dacc, [&](int i, int) { return draws[i]; });
    task_changes<Q>(dacc, q, cA, cB);
    if constexpr (Q >= 2) {
        cA |= lane_xor<1>(cA);
        cB |= lane_xor<1>(cB);
    }
    if constexpr (Q >= 4) {
        cA |= lane_xor<2>(cA);
        cB |= lane_xor<2>(cB);
    }
    if constexpr (Q >= 8) {
        cA |= lane_xor<4>(cA);
        cB |= lane_xor<4>(cB);
    }
    if (q == 0) {
        stw<Coh>(lat, r.a0, A0 ^ cA);
        xorw(lat, r.blo, cB << shb);
        xorw(lat, r.bhi, shb ? cB >> (32u - shb) : 0u);
        if constexpr (Obs) {
            // staggered sign of a class (cx, cy): (-1)^(cx + cy); the
            // a-class is (p, 0), the b-class (pb, 1)
            const int gA = spin_sum16(A0 ^ cA) - spin_sum16(A0), gB = spin_sum16(B0 ^ cB) - spin_sum16(B0);
            const int sA = charge_sum16(A0 ^ cA) - charge_sum16(A0);
            const int sB = charge_sum16(B0 ^ cB) - charge_sum16(B0);
            const bool nA = f.p & 1, nB = !(f.pb & 1);
            dv[0] += gA + gB;
            dv[1] += (nA ? -gA : gA) + (nB ? -gB : gB);
            dv[2] += (nA ? -sA : sA) + (nB ? -sB : sB);
        }
    }
    return packed;
}

// The Philox draws of a task (phase p of sweep s), from its word's first call.
template <int Q>
__device__ __forceinline__ void word_draws(uint32_t call0, int q, uint64_t s, int p, uint32_t key0, uint32_t key1,
                                           u32x4 (&draws)[kTaskCalls<Q>])
{
#pragma unroll
    for (int i = 0; i < kTaskCalls<Q>; ++i)
        draws[i] = pair_draws(philox4x32_10((uint32_t)s, (uint32_t)p, call0 + (uint32_t)call_of_task<Q>(q, i),
                                            (uint32_t)(s >> 32), key0, key1));
}

}  // namespace
}  // namespace lat
