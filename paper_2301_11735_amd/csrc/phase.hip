// gfx950 phase kernels of the coupled-pair Metropolis sweep on one lattice
// (arXiv:2301.11735, section 3.1 update, section 3.2 parallel form): one launch
// per phase, or all phases of a call in one launch with device-wide barriers.
// Integer-only: no floating point, no matrix cores.
//
// One phase updates the N/8 pairs a = (x, y), x = p (mod 4), y even, with
// partners b = a + D.  No updated site neighbours another updated site, so
// every pair reads only sites nobody writes in the phase and the pairs are
// independent; the phase equals their sequential composition.
//
// Per pair the work is table driven (both tables staged in LDS once per
// block): the pair state st = code_a | code_b<<2 and the choice j select a
// transition entry (section 3.1's same-charge sets); one v_dot4 of that
// entry with the packed neighbour sums gives the index of the move's
// energy-change triple in the threshold table; the acceptance test is one
// unsigned compare.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_common.h"
#include "word_task.h"

namespace lat {
namespace {

// ---------------------------------------------------------------------------
// int8 layout: one code per byte, row-major, any side.  Rows of the grid update
// the lattices; a thread owns Philox calls t, i.e. pairs 2t and 2t+1 (words 0,1
// and 2,3 of the call).  As in k_phase_words, what bounds a launch at medium
// sides is its chain: the arguments, the descriptor with the tables behind
// it, and the sites of both pairs, all loaded at once (L = 1000 5.8 -> 5.5 us a
// phase, L = 4000 20.7 -> 18.6; before, tables and sites one after another).  A site and its left and
// right neighbours are mostly bytes of the aligned group of four that holds it:
// one 32-bit load, and a byte more in the phases whose column is the group's
// first or last.
// Offsets of what a pair reads: the groups of its two sites, their neighbours
// beyond the groups (loaded in every phase: a condition would wait for all
// the loads before it), the upper and lower neighbours, and the sites.
struct ByteRefs {
    uint32_t A, B, ae, be, au, ad, bu, bd, oa, ob;
};
struct ByteVals {
    uint32_t A, B, ae, be, au, ad, bu, bd;
};
// The phase on a lattice of side L: columns p and pb of the groups, the
// partners' shift (dX groups, k double rows).
struct BytePhase {
    uint32_t L, Lq, p, pb, dX, k;
};
__device__ __forceinline__ BytePhase byte_phase(int L, uint32_t p, int r, int m, int k)
{
    BytePhase f;
    f.L = (uint32_t)L;
    f.Lq = f.L >> 2;
    f.p = p;
    f.pb = (p + (uint32_t)r) & 3u;
    f.dX = (uint32_t)m + ((p + (uint32_t)r) >> 2);
    f.dX = min(f.dX, f.dX - f.Lq);  // x mod n for x < 2n
    f.k = (uint32_t)k;
    return f;
}

__device__ __forceinline__ ByteRefs byte_refs(const BytePhase &f, uint32_t X, uint32_t Y)
{
    ByteRefs v;
    const uint32_t L = f.L, ra = 2u * Y * L, rau = Y == 0 ? (L - 1u) * L : ra - L;
    uint32_t Xb = X + f.dX, Yb = Y + f.k;
    Xb = min(Xb, Xb - f.Lq);
    Yb = min(Yb, Yb - (L >> 1));
    const uint32_t rb = (2u * Yb + 1u) * L, rbd = 2u * Yb + 2u == L ? 0u : rb + L;
    const uint32_t xa = 4u * X, xb = 4u * Xb;
    auto beyond = [&](uint32_t row, uint32_t x, uint32_t X4, uint32_t c) {
        const uint32_t left = (X4 == 0 ? L : X4) - 1u, right = X4 + 4u == L ? 0u : X4 + 4u;
        return row + (c == 0u ? left : c == 3u ? right : x);
    };
    v.A = ra + xa;
    v.B = rb + xb;
    v.oa = v.A + f.p;
    v.ob = v.B + f.pb;
    v.ae = beyond(ra, xa + f.p, xa, f.p);
    v.be = beyond(rb, xb + f.pb, xb, f.pb);
    v.au = rau + xa + f.p;
    v.ad = v.oa + L;
    v.bu = v.ob - L;
    v.bd = rbd + xb + f.pb;
    return v;
}
// The two pairs of Philox call t (pairs 2t and 2t + 1; row-major over the groups).
__device__ __forceinline__ void call_refs(const BytePhase &f, uint32_t t, ByteRefs (&v)[2])
{
    const uint32_t pi = 2u * t, Y = pi / f.Lq, X = pi - Y * f.Lq;
    const bool wraps = X + 1u == f.Lq;
    v[0] = byte_refs(f, X, Y);
    v[1] = byte_refs(f, wraps ? 0u : X + 1u, wraps ? Y + 1u : Y);
}

// Coh: at device coherence, as ldw and stw of the word form (the state is then
// at a multiple of four bytes).
template <bool Coh>
__device__ __forceinline__ ByteVals byte_fetch(const LAT_GLOBAL uint8_t *st, const ByteRefs &r)
{
    auto word = [&](uint32_t i) -> uint32_t {
        if constexpr (Coh)
            return __hip_atomic_load((const LAT_GLOBAL uint32_t *)(st + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            return *(const LAT_GLOBAL word_any *)(st + i);
    };
    auto byte = [&](uint32_t i) -> uint32_t {
        if constexpr (Coh)
            return __hip_atomic_load(st + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            return st[i];
    };
    return ByteVals{word(r.A), word(r.B), byte(r.ae), byte(r.be), byte(r.au), byte(r.ad), byte(r.bu), byte(r.bd)};
}

template <bool Coh>
__device__ __forceinline__ void byte_apply(LAT_GLOBAL uint8_t *st, const BytePhase &f, const ByteRefs &r,
                                           const ByteVals &v, uint32_t slot8, uint32_t ua, const uint2 *s_tab,
                                           const uint8_t *s_slots, uint32_t &packed)
{
    auto site = [](uint32_t group, uint32_t c) { return (group >> (8u * c)) & 255u; };
    const uint32_t ca = site(v.A, f.p), cb = site(v.B, f.pb);
    const uint32_t al = f.p == 0u ? v.ae : site(v.A, f.p - 1u), ar = f.p == 3u ? v.ae : site(v.A, f.p + 1u);
    const uint32_t bl = f.pb == 0u ? v.be : site(v.B, f.pb - 1u), br = f.pb == 3u ? v.be : site(v.B, f.pb + 1u);
    const uint32_t bpack = contrib_a(al) + contrib_a(ar) + contrib_a(v.au) + contrib_a(v.ad) + contrib_b(bl) +
                           contrib_b(br) + contrib_b(v.bu) + contrib_b(v.bd);
    uint32_t change = 0u;
    pair_step_slot((ca | cb << 2) << 7 | slot8, bpack, ua, s_slots, s_tab, 0x03030000u, packed, change);
    if (change) {
        const uint8_t na = (uint8_t)(ca ^ (change >> 16 & 3u)), nb = (uint8_t)(cb ^ change >> 24);
        if constexpr (Coh) {
            __hip_atomic_store(st + r.oa, na, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(st + r.ob, nb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            st[r.oa] = na;
            st[r.ob] = nb;
        }
    }
}

template <int N>
__global__ void __launch_bounds__(kWordsPhaseMaxThreads) k_phase_bytes(WordsArgsOf<N> a)
{
    __shared__ uint2 s_tab[kDevTabEntries];
    __shared__ __align__(16) uint2 s_slots[kSlotEntries];
    uint8_t *scr = a.scratch[blockIdx.y];
    const uint32_t sweeps = a.sweeps[blockIdx.y], run = a.run[blockIdx.y];
    const uint32_t blocks = run >> 16, block = (run & 0xFFFFu) + blockIdx.x;
    // the whole block: no barrier is skipped by part of it (one condition of all
    // three arguments, for one wait)
    if ((scr == nullptr) | (a.iter >= sweeps) | (block >= blocks)) return;
    const uint32_t threads = a.threads;  // (the launch's own count is in a further line of arguments)
    TableLoads tables;
    tables.load((const uint2 *)(scr + kScrDevTab), threads);
    const LatDesc d = *(const LatDesc *)(scr + kScrDesc);
    LAT_GLOBAL uint8_t *st = (LAT_GLOBAL uint8_t *)d.state;
    // after the descriptor's loads, which would not be scalar behind it
    __builtin_amdgcn_s_setprio(3);
    const uint64_t s = d.next_sweep + a.iter;
    int r, mm[4], kk[4];
    device_schedule(d.L, d.key0, d.key1, s, r, mm, kk);
    const BytePhase f = byte_phase(d.L, (uint32_t)a.p, r, mm[a.p], kk[a.p]);
    const uint32_t calls = f.L * f.L / 16u, step = blocks * threads;
    uint32_t t = block * threads + threadIdx.x;
    ByteRefs at[2];
    ByteVals v[2];
    u32x4 w;
    // threads past the last call load the first one's sites
    auto fetch = [&](uint32_t call) {
        call_refs(f, call, at);
        v[0] = byte_fetch<false>(st, at[0]);
        v[1] = byte_fetch<false>(st, at[1]);
        w = pair_draws(philox4x32_10((uint32_t)s, f.p, call, (uint32_t)(s >> 32), d.key0, d.key1));
    };
    fetch(t < calls ? t : 0u);
    tables.store(s_tab, s_slots, threads);
    __syncthreads();
    int tr[3] = {0, 0, 0};
    while (t < calls) {
        uint32_t packed = 0;
        byte_apply<false>(st, f, at[0], v[0], w.x, w.y, s_tab, (const uint8_t *)s_slots, packed);
        byte_apply<false>(st, f, at[1], v[1], w.z, w.w, s_tab, (const uint8_t *)s_slots, packed);
        unpack_tracker(packed, tr);
        t += step;
        if (t < calls) fetch(t);
    }
    wave_reduce_add3(tr, (unsigned long long *)(scr + kScrSlots) + 3 * (size_t)(block % kMaxSlots));
}

// Persistent form, as k_words_series without records: all sweeps of a call in one
// launch of blocks that are all resident at once, a barrier of a lattice's
// blocks after every phase.  Against one launch per phase (us a sweep): L = 388 17.5 -> 10.7, L = 500
// 17.4 -> 12.4, L = 1000 19.3 -> 15.0; for larger lattices, whose threads take
// several calls a phase, the loads past the caches cost more than the launches
// (L = 4000 72 -> 97).
__global__ void __launch_bounds__(kBytesSeriesMaxThreads) k_bytes_series(WordsSeriesArgs a)
{
    __shared__ uint2 s_tab[kDevTabEntries];
    __shared__ __align__(16) uint2 s_slots[kSlotEntries];
    int li = 0;  // this block's lattice (uniform)
    while (li + 1 < a.count && blockIdx.x >= a.first_block[li + 1]) ++li;
    uint8_t *scr = a.scratch[li];
    // ahead of the meeting: its atomics would make the descriptor's loads vector loads
    const LatDesc d = *(const LatDesc *)(scr + kScrDesc);
    LAT_GLOBAL uint8_t *st = (LAT_GLOBAL uint8_t *)d.state;
    const uint32_t b = blockIdx.x - a.first_block[li], nb = a.first_block[li + 1] - a.first_block[li];
    GridBarrier barrier{(unsigned *)(scr + kScrObsSlots), b, nb, 0u, false};
    unsigned *err = (unsigned *)(scr + kScrErr);
    if (a.alone ? !barrier.alone() : !barrier.first_arrive(a.assemble_ticks)) return;
    TableLoads tables;
    tables.load((const uint2 *)(scr + kScrDevTab), blockDim.x);
    tables.store(s_tab, s_slots, blockDim.x);
    __syncthreads();
    const uint8_t *slots = (const uint8_t *)s_slots;
    const uint32_t sweeps = a.sweeps[li], calls = (uint32_t)d.L * (uint32_t)d.L / 16u;
    const uint32_t first = b * blockDim.x + threadIdx.x, stride = nb * blockDim.x;
    // At most one call a thread (uniform per lattice): its draws and places are
    // made while the block waits at the barrier.
    const bool one = stride >= calls, mine = one && first < calls;
    int r, mm[4], kk[4];
    device_schedule(d.L, d.key0, d.key1, d.next_sweep, r, mm, kk);
    BytePhase f = byte_phase(d.L, 0u, r, mm[0], kk[0]);
    ByteRefs at[2] = {};
    u32x4 w{};
    auto prepare = [&](uint64_t s, uint32_t call) {
        call_refs(f, call, at);
        w = pair_draws(philox4x32_10((uint32_t)s, f.p, call, (uint32_t)(s >> 32), d.key0, d.key1));
    };
    if (mine) prepare(d.next_sweep, first);
    if (!barrier.assemble(a.alone, a.assemble_ticks)) return;
    barrier.rounds = 1u;
    int tr[3] = {0, 0, 0};
    for (uint32_t it = 0; it < sweeps; ++it) {
        const uint64_t s = d.next_sweep + it;
#pragma unroll 1
        for (uint32_t p = 0; p < 4u; ++p) {
            uint32_t packed = 0u;
            auto step = [&] {
                const ByteVals v0 = byte_fetch<true>(st, at[0]), v1 = byte_fetch<true>(st, at[1]);
                byte_apply<true>(st, f, at[0], v0, w.x, w.y, s_tab, slots, packed);
                byte_apply<true>(st, f, at[1], v1, w.z, w.w, s_tab, slots, packed);
            };
            if (mine) step();
            for (uint32_t t = one ? calls : first; t < calls; t += stride) {
                prepare(s, t);
                step();
                unpack_tracker(packed, tr);
                packed = 0u;
            }
            barrier.arrive();
            // the next phase's schedule, draws and places, while the others arrive
            unpack_tracker(packed, tr);
            if (p == 3u) device_schedule(d.L, d.key0, d.key1, s + 1, r, mm, kk);
            const uint32_t q = (p + 1u) & 3u;
            f = byte_phase(d.L, q, r, mm[q], kk[q]);
            if (mine) prepare(p < 3u ? s : s + 1, first);
            barrier.wait(err, a.barrier_ticks);
        }
    }
    wave_reduce_add3(tr, (unsigned long long *)(scr + kScrSlots) + 3 * (size_t)(b % kMaxSlots));
    // every block read the descriptor before its first phase's barrier
    if (b == 0 && threadIdx.x == 0 && sweeps > 0)
        ((LatDesc *)(scr + kScrDesc))->next_sweep = d.next_sweep + sweeps;
}

// ---------------------------------------------------------------------------
// 2-bit layout (see lattice.h): class c = 4*(y&1) + (x&3) is an (L/2) x (L/4)
// array of sites, L/64 words per row, 16 sites per word.
//
// Thread (Y, j) owns word j of row Y of the a-class (p, 0): 16 pairs.  Their
// partners are the 16 consecutive b-class sites starting at class position
// 16j + dX of row Y + k, which straddle two b-words.  Each block holds whole
// class rows, so the b-row of a-row Y is read and written by one block only:
// after the block barrier, thread j assembles b-word jb+1 from its own new
// codes and those of thread j+1 (mod W), and every b-word has one writer.

// MinWaves > 1 asks the compiler to fit MinWaves waves per SIMD (at most
// 512/MinWaves VGPRs), e.g. two 1024-thread blocks per compute unit at 8.
// The ten words one thread reads for its 16 pairs: its a-word, the a-words'
// left/right/up/down neighbour words, and the same five for the 16 partners
// (the b-side words start mid-word and are funnel-shifted into place).
// Seven of them start mid-word (by the same shift for every thread of a
// phase): both words covering each are fetched, and the funnel shift into
// place waits until the group is computed, so a prefetch never waits for its
// own loads.
struct PairWords {
    uint32_t A0, AU, AD;
    uint32_t ALlo, ALhi, ARlo, ARhi, B0lo, B0hi, BLlo, BLhi, BRlo, BRhi, BUlo, BUhi, BDlo, BDhi;
};

// LDS tables of the 2-bit phase kernels, in 8-byte units: the device
// threshold table, one pad entry, the transition slots (16-byte aligned), and
// two spare entries that absorb the writes of threads past the end during
// staging.  Staging moves 16 bytes (two units) at a time.
constexpr int kLdsSlots = kDevTabEntries + 1;             // 934: 16-byte aligned
constexpr int kLdsTabUnits = kLdsSlots + kSlotEntries;    // 1190
constexpr int kLdsTabPairs = kLdsTabUnits / 2;            // 595
static_assert((kLdsSlots * 8) % 16 == 0 && kLdsTabUnits % 2 == 0, "slot table alignment");
static_assert(kScrTrans >= (size_t)kLdsSlots * 8, "the last device-table pair reads scratch, not past it");

// Units 2i and 2i+1 of the LDS tables from the lattice's scratch.  The pair
// holding the pad unit reads the scratch bytes after the device table.  Both
// sources are said to be global memory: a flat load counts as an LDS access too,
// and the wait for the arguments, and the one for the tables, then waited for
// every load of the prologue (50 sweeps, with flat loads and now: L = 2112 1448 ->
// 1406 us, L = 4096 1457 -> 1384, L = 8192 3264 -> 3188).
__device__ __forceinline__ uint4 table_pair(const PhaseArgs &a, int i)
{
    typedef uint32_t quad __attribute__((ext_vector_type(4)));
    const LAT_GLOBAL quad *src = 2 * i < kLdsSlots ? (const LAT_GLOBAL quad *)a.dev_tab + i
                                                   : (const LAT_GLOBAL quad *)kWordSlots.v + (i - kLdsSlots / 2);
    const quad v = *src;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// One phase of the 2-bit lattice by this block: row groups blockIdx.x,
// blockIdx.x + gridDim.x, ...
//
// s_tabs holds kLdsTabUnits + 2 entries.  Stage false: the tables are
// already there.  Stage true: they are copied here; the table loads are
// issued first, then the first group's words, so that the LDS writes wait
// only for the former and the word loads overlap the staging.
template <bool Stage>
__device__ __forceinline__ void phase_2bit(const PhaseArgs &a, int rows_per_block, uint2 *s_tabs, uint32_t *xch,
                                           int (&tr)[3])
{
    const uint2 *s_tab = s_tabs;
    const uint8_t *s_slots = (const uint8_t *)(s_tabs + kLdsSlots);
    const int L = a.L, W = L >> 6, H = L >> 1, Lq = L >> 2;
    const int rr = W == 1 ? (int)threadIdx.x : (int)__umulhi(threadIdx.x, a.magicW), j = (int)threadIdx.x - rr * W;
    const int n_groups = H >> __builtin_ctz((unsigned)rows_per_block);  // a power of two
    uint32_t *st = (uint32_t *)a.state;
    const uint32_t csz = (uint32_t)H * (uint32_t)W;  // words per class; N/16 < 2^32
    const int p = a.p;
    const int pb = (p + a.r) & 3, carry = (p + a.r) >> 2;
    int dX = a.m + carry;
    if (dX >= Lq) dX -= Lq;
    int Xb = 16 * j + dX;
    if (Xb >= Lq) Xb -= Lq;
    const int jb = Xb >> 4, shb = Xb & 15;
    const uint32_t jw_out = (uint32_t)(jb + 1 == W ? 0 : jb + 1);
    const int j_next = j + 1 == W ? 0 : j + 1;
    // word offsets of the classes read on the a side and the b side
    const uint32_t oA0 = (uint32_t)p * csz;
    const uint32_t oAL = (uint32_t)(p > 0 ? p - 1 : 3) * csz;
    const uint32_t oAR = (uint32_t)(p < 3 ? p + 1 : 0) * csz;
    const uint32_t oAV = (uint32_t)(4 + p) * csz;
    const uint32_t oB0 = (uint32_t)(4 + pb) * csz;
    const uint32_t oBL = (uint32_t)(pb > 0 ? 4 + pb - 1 : 7) * csz;
    const uint32_t oBR = (uint32_t)(pb < 3 ? 4 + pb + 1 : 4) * csz;
    const uint32_t oBV = (uint32_t)pb * csz;
    const int xAL = p > 0 ? 16 * j : (j == 0 ? Lq - 1 : 16 * j - 1);
    const int xAR = p < 3 ? 16 * j : 16 * j + 1;
    const int xBL = pb > 0 ? Xb : (Xb == 0 ? Lq - 1 : Xb - 1);
    const int xBR = pb < 3 ? Xb : (Xb + 1 == Lq ? 0 : Xb + 1);

    auto row_of = [&](int g) { return g * rows_per_block + rr; };
    auto brow_of = [&](int Y) { return Y + a.k >= H ? Y + a.k - H : Y + a.k; };
    auto load_words = [&](int g) {
        const int Y = row_of(g), Yb = brow_of(Y);
        const uint32_t ro = (uint32_t)Y * W, rob = (uint32_t)Yb * W;
        const uint32_t roU = (uint32_t)(Y == 0 ? H - 1 : Y - 1) * W;
        const uint32_t robD = (uint32_t)(Yb + 1 == H ? 0 : Yb + 1) * W;
        PairWords w;
        w.A0 = word_at(st, oA0 + ro + j);
        w.AU = word_at(st, oAV + roU + j);
        w.AD = word_at(st, oAV + ro + j);
        load_pair(st, oAL + ro, W, xAL, w.ALlo, w.ALhi);
        load_pair(st, oAR + ro, W, xAR, w.ARlo, w.ARhi);
        load_pair(st, oB0 + rob, W, Xb, w.B0lo, w.B0hi);
        load_pair(st, oBL + rob, W, xBL, w.BLlo, w.BLhi);
        load_pair(st, oBR + rob, W, xBR, w.BRlo, w.BRhi);
        load_pair(st, oBV + rob, W, Xb, w.BUlo, w.BUhi);
        load_pair(st, oBV + robD, W, Xb, w.BDlo, w.BDhi);
        return w;
    };
    // funnel shifts (uniform per phase: 2 * (x mod 16) for each start x)
    const uint32_t fAL = 2u * (uint32_t)(xAL & 15), fAR = 2u * (uint32_t)(xAR & 15);
    const uint32_t fB = 2u * (uint32_t)(Xb & 15), fBL = 2u * (uint32_t)(xBL & 15), fBR = 2u * (uint32_t)(xBR & 15);

    // Draws of the group's 8 Philox calls (call c serves pairs 2c and 2c+1).
    auto call_of = [&](int gg, int c) {
        const uint32_t call0 = (uint32_t)row_of(gg) * (uint32_t)(Lq >> 1) + 8u * (uint32_t)j;
        return philox4x32_10(a.s_lo, (uint32_t)p, call0 + (uint32_t)c, a.s_hi, a.key0, a.key1);
    };
    // Updates the 16 pairs of group gg from its words cw.
    auto group = [&](const PairWords &cw, int gg, int bb) {
        const int Y = row_of(gg), Yb = brow_of(Y);
        const uint32_t B0 = __builtin_amdgcn_alignbit(cw.B0hi, cw.B0lo, fB);
        const SideSums sa = side_sums(__builtin_amdgcn_alignbit(cw.ALhi, cw.ALlo, fAL),
                                      __builtin_amdgcn_alignbit(cw.ARhi, cw.ARlo, fAR), cw.AU, cw.AD);
        const SideSums sb = side_sums(__builtin_amdgcn_alignbit(cw.BLhi, cw.BLlo, fBL),
                                      __builtin_amdgcn_alignbit(cw.BRhi, cw.BRlo, fBR),
                                      __builtin_amdgcn_alignbit(cw.BUhi, cw.BUlo, fB),
                                      __builtin_amdgcn_alignbit(cw.BDhi, cw.BDlo, fB));
        // bpack of site t = (sumS_a+4, sumS_b+4, sumsig_a+4, sumsig_b+4): site
        // t = 4k + g is byte k of nibble plane g (g = 0, 2: even sites, low and
        // high nibbles; g = 1, 3: odd sites).  Philox call c serves t = 2c and
        // 2c+1, so calls 0,2,4,6 need planes 0 and 1, calls 1,3,5,7 planes 2
        // and 3; handling them in that order keeps 8 packed words live.
        uint32_t dacc[4] = {0u, 0u, 0u, 0u}, packed = 0u;  // code changes of pairs 4k .. 4k+3
        const uint32_t st8[2] = {pair_states8(cw.A0, B0, 0), pair_states8(cw.A0, B0, 1)};
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint32_t ge[4], go[4];
            const int sh = 4 * half;
            transpose4((sa.ES >> sh) & kM0F, (sb.ES >> sh) & kM0F, (sa.EG >> sh) & kM0F, (sb.EG >> sh) & kM0F,
                       ge[0], ge[1], ge[2], ge[3]);
            transpose4((sa.OS >> sh) & kM0F, (sb.OS >> sh) & kM0F, (sa.OG >> sh) & kM0F, (sb.OG >> sh) & kM0F,
                       go[0], go[1], go[2], go[3]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = 2 * k + half;
                const u32x4 w = pair_draws(call_of(gg, c));
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int t = 2 * c + h, at = 4 * (t & 7);
                    const uint32_t s7 = at >= 7 ? st8[t >> 3] >> (at >= 7 ? at - 7 : 0) : st8[t >> 3] << (at < 7 ? 7 - at : 0);
                    pair_step_slot((s7 & 0x780u) | (h ? w.z : w.x), h ? go[k] : ge[k], h ? w.w : w.y, s_slots, s_tab,
                                   0x03030000u << (2 * (t & 3)), packed, dacc[k]);
                }
            }
        }
        unpack_tracker(packed, tr);
        const uint32_t Anew = cw.A0 ^ __builtin_amdgcn_perm(__builtin_amdgcn_perm(dacc[3], dacc[2], 0x0C0C0602u),
                                                            __builtin_amdgcn_perm(dacc[1], dacc[0], 0x0C0C0602u),
                                                            0x05040100u);
        const uint32_t Bnew = B0 ^ __builtin_amdgcn_perm(__builtin_amdgcn_perm(dacc[3], dacc[2], 0x0C0C0703u),
                                                         __builtin_amdgcn_perm(dacc[1], dacc[0], 0x0C0C0703u),
                                                         0x05040100u);
        word_put(st, oA0 + (uint32_t)Y * W + j, Anew);
        uint32_t *x = xch + bb * blockDim.x;
        x[threadIdx.x] = Bnew;
        __syncthreads();
        const uint32_t nb = x[rr * W + j_next];
        const uint32_t word = shb ? __builtin_amdgcn_alignbit(nb, Bnew, 32u - 2u * (uint32_t)shb) : nb;
        word_put(st, oB0 + (uint32_t)Yb * W + jw_out, word);
    };

    // Each group's words are fetched before the previous group is computed.
    // Every word read is either never written in this phase or written only
    // by this block in the iteration that owns it, after its read.
    int g = blockIdx.x;
    PairWords cur;  // loaded before it is read
    if (Stage) {
        constexpr int kTot = kLdsTabPairs, kK = 2;  // two 16-byte loads a thread cover 512-thread blocks
        const int bd = rows_per_block * W;  // the block size of every launch of this form
        uint4 sv[kK];
        int si[kK];
#pragma unroll
        for (int k = 0; k < kK; ++k) {
            si[k] = min((int)threadIdx.x + k * bd, kTot);
            sv[k] = table_pair(a, min(si[k], kTot - 1));
        }
        // unconditional (clamped) and kept after the table loads, so that
        // the LDS writes below wait for the table loads only; the loop skips
        // a block without a group
        __builtin_amdgcn_sched_barrier(0);
        cur = load_words(min(g, n_groups - 1));
        uint4 *s_pairs = (uint4 *)s_tabs;
#pragma unroll
        for (int k = 0; k < kK; ++k) s_pairs[si[k]] = sv[k];
        for (int i = (int)threadIdx.x + kK * bd; i < kTot; i += bd) s_pairs[i] = table_pair(a, i);
        __syncthreads();
    } else if (g < n_groups) {
        cur = load_words(g);
    }
    int buf = 0;
    for (; g < n_groups; g += gridDim.x, buf ^= 1) {
        const int gn = g + gridDim.x;
        PairWords nxt;  // read only when loaded
        if (gn < n_groups) nxt = load_words(gn);
        group(cur, g, buf);
        cur = nxt;
    }
    __syncthreads();  // the exchange buffer is reused by the next phase
}

template <int MinWaves>
__global__ void __launch_bounds__(1024, MinWaves) k_phase_2bit(PhaseArgs a, int rows_per_block)
{
    __shared__ __align__(16) uint2 s_tabs[kLdsTabUnits + 2];
    extern __shared__ uint32_t xch[];  // 2 x blockDim (double buffered)
    int tr[3] = {0, 0, 0};
    phase_2bit<true>(a, rows_per_block, s_tabs, xch, tr);
    block_reduce_add<3>(tr, a.track + 3 * (size_t)blockIdx.x);
}

// Persistent form: `sweeps` sweeps from sweep a.s_lo|a.s_hi in one launch of
// co-resident blocks (cooperative launch), tables staged once, schedules
// computed on the device, a device-wide barrier after every phase.
template <int MinWaves>
__global__ void __launch_bounds__(1024, MinWaves) k_sweeps_2bit(PhaseArgs a, int rows_per_block, uint32_t sweeps,
                                                                unsigned *counter, unsigned *err)
{
    __shared__ __align__(16) uint2 s_tabs[kLdsTabUnits + 2];
    extern __shared__ uint32_t xch[];
    for (int i = threadIdx.x; i < kLdsTabPairs; i += blockDim.x) ((uint4 *)s_tabs)[i] = table_pair(a, i);
    __syncthreads();
    int tr[3] = {0, 0, 0};
    const uint64_t s0 = ((uint64_t)a.s_hi << 32) | a.s_lo;
    unsigned arrivals = 0;
    for (uint32_t i = 0; i < sweeps; ++i) {
        const uint64_t s = s0 + i;
        int r, mm[4], kk[4];
        // rows x W threads: the last wave may be a partial one
        device_schedule<false>(a.L, a.key0, a.key1, s, r, mm, kk);
        PhaseArgs b = a;
        b.s_lo = (uint32_t)s;
        b.s_hi = (uint32_t)(s >> 32);
        b.r = r;
        for (int p = 0; p < 4; ++p) {
            b.p = p;
            b.m = mm[p];
            b.k = kk[p];
            phase_2bit<false>(b, rows_per_block, s_tabs, xch, tr);
            arrivals += gridDim.x;
            grid_barrier(counter, arrivals, err);
        }
    }
    block_reduce_add<3>(tr, a.track + 3 * (size_t)blockIdx.x);
}



int g_num_cus = 0;

int num_cus()
{
    if (g_num_cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            g_num_cus = n;
        else
            g_num_cus = 256;
    }
    return g_num_cus;
}

}  // namespace

// ---------------------------------------------------------------------------
const void *bytes_series_kernel() { return (const void *)k_bytes_series; }

namespace {
template <int N>
void phase_bytes(const WordsArgsOf<N> &a, int threads, hipStream_t s)
{
    hipLaunchKernelGGL(k_phase_bytes<N>, dim3(a.max_blocks, (unsigned)a.count), dim3((unsigned)threads), 0, s, a);
}
}  // namespace

hipError_t launch_phase_bytes(const WordsArgs &a, int threads, hipStream_t s)
{
    with_rows(a, [&](const auto &rows) { phase_bytes(rows, threads, s); });
    return hipGetLastError();
}

// Rows per block: a power of two <= 32 (so it divides the L/2 = 32W rows);
// by default the largest giving at most max_threads threads.  Every block
// holds whole class rows.  For one launch per phase the default is blocks of
// at most 512 threads, two per compute unit (16 waves, as one 1024-thread
// block): measured 1.5% faster than one 1024-thread block at L = 8192.
// Never fewer threads than a block has tracker sums, each of which one thread
// adds, whatever number of rows is asked for.
constexpr int kTrackSums = 3;
static int rows_per_block_2bit(int W, int requested, int max_threads)
{
    const int cap = requested > 0 ? requested : 32;
    int r = 1;
    while (r < 32 && ((2 * r <= cap && 2 * r * W <= max_threads) || r * W < kTrackSums)) r *= 2;
    return r;
}

hipError_t launch_phase_2bit(const PhaseArgs &a, const Tuning2Bit &t, hipStream_t s)
{
    const int W = a.L >> 6, H = a.L >> 1;
    const int R = rows_per_block_2bit(W, t.rows_per_block, t.rows_per_block > 0 ? 1024 : 512);
    const int block = R * W;
    int grid = H / R;
    const int bpc = t.blocks_per_cu > 0 ? t.blocks_per_cu : 2;
    if (grid > bpc * num_cus()) grid = bpc * num_cus();
    if (grid > kMaxSlots) grid = kMaxSlots;
    if (t.waves_hint >= 8)
        hipLaunchKernelGGL(k_phase_2bit<8>, dim3(grid), dim3(block), (size_t)block * 8u, s, a, R);
    else
        hipLaunchKernelGGL(k_phase_2bit<1>, dim3(grid), dim3(block), (size_t)block * 8u, s, a, R);
    return hipGetLastError();
}

bool persistent_2bit_supported(int L, const Tuning2Bit &t, int *grid_out, int *rows_out)
{
    int dev = 0, coop = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return false;
    const int W = L >> 6, R = rows_per_block_2bit(W, t.rows_per_block, 1024), block = R * W;
    int per_cu = 0;
    const void *fn = t.waves_hint >= 8 ? (const void *)k_sweeps_2bit<8> : (const void *)k_sweeps_2bit<1>;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, block, (size_t)block * 8u) != hipSuccess ||
        per_cu < 1)
        return false;
    const int want = t.blocks_per_cu > 0 ? t.blocks_per_cu : 1;
    *grid_out = std::min(std::min(per_cu, want) * num_cus(), kMaxSlots);
    *rows_out = R;
    return true;
}

hipError_t launch_sweeps_2bit(const PhaseArgs &a, const Tuning2Bit &t, uint32_t sweeps, unsigned *counter,
                              unsigned *err, hipStream_t s)
{
    int grid = 0, R = 0;
    if (!persistent_2bit_supported(a.L, t, &grid, &R)) return hipErrorNotSupported;
    const int block = R * (a.L >> 6);
    hipError_t e = launch_zero_i64((unsigned long long *)counter, 1, s);  // counter (and the word after it)
    if (e != hipSuccess) return e;
    PhaseArgs args = a;
    int rows = R;
    uint32_t n = sweeps;
    void *kargs[] = {&args, &rows, &n, &counter, &err};
    const void *fn = t.waves_hint >= 8 ? (const void *)k_sweeps_2bit<8> : (const void *)k_sweeps_2bit<1>;
    return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(block), kargs, (size_t)block * 8u, s);
}


}  // namespace lat
