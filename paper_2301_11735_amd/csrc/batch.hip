// gfx950 batched kernels (arXiv:2301.11735 section 3.2: several lattice
// copies processed together): one block per lattice, the lattice resident in
// LDS for all the sweeps of a launch, and the batched observable reduction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "onchip.h"
#include "word_task.h"

namespace lat {
namespace {

// ---------------------------------------------------------------------------
// Per-site form, one byte per site in LDS (row-major), for lattices of any
// side up to kSiteMaxL.  A site's byte is (1 + S) | (1 + sigma) << 4, so that
// the bytes of four neighbours add up to both neighbour sums at once (at
// most 8 a nibble), a site is read with one byte load, and new codes are
// written with plain byte stores (its pair's lane is the only one that reads
// or writes them in the phase).
//
// What bounds these sizes is the chain of a phase (byte loads, two dependent
// table gathers, the store, the block barrier), not the work: L = 32 has 128
// pairs a phase on one compute unit.  So the pairs of a phase are spread over
// as many threads as help (one pair a thread up to kSiteOnePair pairs, else the
// two pairs of a Philox call), a thread with one pair draws the next phase's
// call in the waits of its own loads, the choice slot of a draw does not depend
// on the state, and a launch holds a whole series of observation intervals
// with the observables taken from LDS in between.
//
// Measured against two bits per site, with neighbours from ten shifted word
// reads and codes merged by LDS atomics: L = 32, 1000 sweeps with observables
// every 10 as one series 6230 -> 1381 us; 224 lattices of L = 16, 200 intervals of
// one sweep in a graph 3629 -> 715 us; 40 lattices of L = 100, 50 sweeps 522 ->
// 224 us; 12 of L = 300, 20 sweeps 1295 -> 655 us.

constexpr uint32_t kSiteHash = 0x2B298945u;  // (byte_a | byte_b << 8) -> 4 distinct top bits for the 16 states

constexpr TransSlots make_site_slots()
{
    TransSlots t{};
    for (int st = 0; st < 16; ++st)
        for (int slot = 0; slot < 12; ++slot) {
            uint32_t coef = 0, C = 0;
            int a1 = 0, b1 = 0;
            trans_slot(st, slot, coef, C, a1, b1);
            const uint32_t x = site_byte(st & 3) | site_byte(st >> 2) << 8;
            const uint32_t at = 2u * (16u * ((x * kSiteHash) >> 28) + (uint32_t)slot);
            t.v[at] = coef;
            t.v[at + 1] = C | (site_byte(a1) | site_byte(b1) << 8) << 16;
        }
    return t;
}
constexpr bool site_hash_distinct()
{
    uint32_t seen = 0;
    for (int st = 0; st < 16; ++st) {
        const uint32_t x = site_byte(st & 3) | site_byte(st >> 2) << 8, h = (x * kSiteHash) >> 28;
        if ((seen >> h) & 1u) return false;
        seen |= 1u << h;
    }
    return true;
}
static_assert(site_hash_distinct(), "the 16 pair states get 16 table rows");
__device__ const TransSlots kSiteSlots = make_site_slots();

// Pairs a phase up to which a thread takes one pair: two waves a SIMD, whose
// repeated draws still fit into the chain of a phase.
constexpr uint32_t kSiteOnePair = 512;

__device__ __forceinline__ void stage_sites(uint32_t *lat, const LatDesc &d)
{
    const uint32_t L = (uint32_t)d.L, N = L * L;
    if (d.enc == 0) {
        if (((uintptr_t)d.state & 3u) == 0) {
            const LAT_GLOBAL uint32_t *src = (const LAT_GLOBAL uint32_t *)d.state;
            for (uint32_t i = threadIdx.x; i < N / 4u; i += blockDim.x) lat[i] = site_from_codes(src[i] & 0x03030303u);
        } else {
            const LAT_GLOBAL uint8_t *src = (const LAT_GLOBAL uint8_t *)d.state;
            for (uint32_t i = threadIdx.x; i < N; i += blockDim.x)
                ((uint8_t *)lat)[i] = (uint8_t)(kSiteBytes >> (8u * (src[i] & 3u)));
        }
    } else {
        // words j of the four classes of row y are its sites 64 j .. 64 j + 63: a task
        // takes a quarter of them, 16 bytes a store
        const LAT_GLOBAL uint32_t *src = (const LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = L >> 6, csz = (L >> 1) * W;
        for (uint32_t i = threadIdx.x; i < 4u * L * W; i += blockDim.x) {
            const uint32_t y = (i >> 2) / W, j = (i >> 2) - y * W, at = 4u * (y & 1u) * csz + (y >> 1) * W + j, q = 8u * (i & 3u);
            const uint32_t w0 = src[at] >> q, w1 = src[at + csz] >> q, w2 = src[at + 2u * csz] >> q, w3 = src[at + 3u * csz] >> q;
            uint32_t v[4];
#pragma unroll
            for (uint32_t t = 0; t < 4u; ++t)
                v[t] = site_from_codes(((w0 >> 2u * t) & 3u) | ((w1 >> 2u * t) & 3u) << 8 | ((w2 >> 2u * t) & 3u) << 16 |
                                       ((w3 >> 2u * t) & 3u) << 24);
            ((uint4 *)lat)[i] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    }
}

__device__ __forceinline__ void unstage_sites(const uint32_t *lat, const LatDesc &d)
{
    const uint32_t L = (uint32_t)d.L, N = L * L;
    if (d.enc == 0) {
        if (((uintptr_t)d.state & 3u) == 0) {
            LAT_GLOBAL uint32_t *dst = (LAT_GLOBAL uint32_t *)d.state;
            for (uint32_t i = threadIdx.x; i < N / 4u; i += blockDim.x) dst[i] = codes_from_site(lat[i]);
        } else {
            LAT_GLOBAL uint8_t *dst = (LAT_GLOBAL uint8_t *)d.state;
            for (uint32_t i = threadIdx.x; i < N; i += blockDim.x)
                dst[i] = (uint8_t)codes_from_site(((const uint8_t *)lat)[i]) & 3u;
        }
    } else {
        LAT_GLOBAL uint32_t *dst = (LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = L >> 6, csz = (L >> 1) * W;
        for (uint32_t i = threadIdx.x; i < 8u * csz; i += blockDim.x) {
            const uint32_t c = i / csz, rem = i - c * csz, Y = rem / W, j = rem - Y * W;
            const uint32_t *row = lat + ((2u * Y + (c >> 2)) * L + 64u * j) / 4u;
            uint32_t w = 0;
#pragma unroll
            for (uint32_t t = 0; t < 16u; ++t)
                w |= ((codes_from_site(row[t]) >> (8u * (c & 3u))) & 3u) << (2u * t);
            dst[i] = w;
        }
    }
}

// Byte offsets of a pair's first site in phase 0 (phase p: p more) and its
// surroundings: rows above and below, the left neighbour in phase 0, the
// right one in phase 3.
struct SitePos {
    uint32_t x4, row, a, u, d, l, r;
};
__device__ __forceinline__ SitePos site_pos(uint32_t pi, uint32_t L, uint32_t Lq, uint32_t N, uint32_t magicLq)
{
    const uint32_t Y = Lq == 1u ? pi : __umulhi(pi, magicLq), X = pi - Y * Lq;
    SitePos s;
    s.x4 = 4u * X;
    s.row = 2u * Y * L;
    s.a = s.row + s.x4;
    s.u = (Y == 0 ? N : s.row) - L + s.x4;
    s.d = s.a + L;  // y is even: never the last row
    s.l = X == 0 ? s.row + L - 1u : s.a - 1u;
    s.r = X + 1u == Lq ? s.row : s.a + 4u;
    return s;
}

struct SiteDraw {
    uint32_t slot8, ua;
};
// The call of a task, and its draws from the call's words.
template <int PP>
__device__ __forceinline__ PhiloxRun site_call(uint64_t s, uint32_t p, uint32_t task, uint32_t key0, uint32_t key1)
{
    return PhiloxRun{(uint32_t)s, p, PP == 2 ? task : task >> 1, (uint32_t)(s >> 32), key0, key1};
}
template <int PP>
__device__ __forceinline__ void site_draws(const PhiloxRun &w, uint32_t task, SiteDraw (&o)[PP])
{
    const bool odd = PP == 1 && (task & 1u);
    o[0] = SiteDraw{slot8_of(odd ? w.c2 : w.c0), min(odd ? w.c3 : w.c1, 0xFFFFFFFEu)};
    if constexpr (PP == 2) o[1] = SiteDraw{slot8_of(w.c2), min(w.c3, 0xFFFFFFFEu)};
}

// Byte offsets of a pair's second site in phase P, displaced by (r + 4 m, 1 + 2 k),
// and of its neighbours.  x mod n for x < 2 n is min(x, x - n) in
// unsigned arithmetic.
struct SiteB {
    uint32_t b, l, r, d;
};
template <int P>
__device__ __forceinline__ SiteB site_b(const SitePos &s, uint32_t L, uint32_t N, const SweepWords &w)
{
    const uint32_t Dx = w.r + 4u * w.m[P], DyL = (1u + 2u * w.k[P]) * L;
    uint32_t xb = s.x4 + P + Dx;
    xb = min(xb, xb - L);
    uint32_t rb = s.row + DyL;
    rb = min(rb, rb - N);
    uint32_t rd = rb + L;  // y_b is odd: never the first row
    rd = min(rd, rd - N);
    return SiteB{rb + xb, rb + min(xb - 1u, xb - 1u + L), rb + min(xb + 1u, xb + 1u - L), rd + xb};
}

// One coupled-pair step in phase P on the sites s and q, in its four stages:
// the loads, the transition entry, the move's entry, and the stores.  A stage
// waits for the LDS once, so other work fits between them.
struct SiteLoads {
    uint32_t ea, eb, na[4], nb[4];
};
template <int P>
__device__ __forceinline__ SiteLoads site_load(const uint8_t *lat, const SitePos &s, const SiteB &q, uint32_t L)
{
    return SiteLoads{lat[s.a + P],
                     lat[q.b],
                     {lat[P > 0 ? s.a + P - 1 : s.l], lat[P < 3 ? s.a + P + 1 : s.r], lat[s.u + P], lat[s.d + P]},
                     {lat[q.l], lat[q.r], lat[q.b - L], lat[q.d]}};
}
struct SiteMove {
    uint32_t x, bpack;  // the two site bytes, the packed neighbour sums
    uint2 tr;
};
__device__ __forceinline__ SiteMove site_move(const SiteLoads &v, const SiteDraw &dr, const uint8_t *s_trans)
{
    SiteMove m;
    m.x = v.ea | v.eb << 8;
    m.tr = *(const uint2 *)(s_trans + ((((m.x * kSiteHash) >> 21) & 0x780u) | dr.slot8));
    const uint32_t t = (v.na[0] + v.na[1] + v.na[2] + v.na[3]) | (v.nb[0] + v.nb[1] + v.nb[2] + v.nb[3]) << 8;
    m.bpack = (t & 0x0F0Fu) | (t & 0xF0F0u) << 12;
    return m;
}
__device__ __forceinline__ uint2 site_entry(const SiteMove &m, const uint8_t *s_tab)
{
    const uint32_t idx = (uint32_t)__builtin_amdgcn_sdot4((int)m.tr.x, (int)m.bpack, (int)m.tr.y, false);
    return *(const uint2 *)(s_tab + (uint32_t)(uint16_t)(idx << 3));
}
template <int P>
__device__ __forceinline__ void site_store(uint8_t *lat, const SitePos &s, uint32_t qb, const SiteDraw &dr,
                                           const SiteMove &m, const uint2 &e, uint32_t &packed)
{
    const bool acc = dr.ua < e.x;
    packed += acc ? e.y : 0u;
    const uint32_t nw = acc ? m.tr.y >> 16 : m.x;
    lat[s.a + P] = (uint8_t)nw;
    lat[qb] = (uint8_t)(nw >> 8);
}

// `intervals` times `every` sweeps of the lattice in LDS from sweep first on,
// each interval followed by observe(k).  PP pairs a task; One: every thread
// has at most one task, whose draws and second sites of the next phase are
// made while the current phase's loads are in flight.
template <int PP, bool One, typename F>
__device__ __forceinline__ void site_sweeps(uint8_t *lat, uint32_t *sched, const LatDesc &d, uint64_t first,
                                            uint32_t intervals, uint32_t every, const uint8_t *s_tab,
                                            const uint8_t *s_trans, int (&tr)[3], F observe)
{
    const uint32_t L = (uint32_t)d.L, Lq = L >> 2, N = L * L;
    const uint32_t magicLq = Lq == 1u ? 0u : 0xFFFFFFFFu / Lq + 1u;
    const uint32_t tasks = N / (8u * PP), n = intervals * every;
    const bool mine = threadIdx.x < tasks;
    make_schedules(sched, first, n, d.key0, d.key1, L);
    __syncthreads();
    SweepWords sc = sweep_words(sweep_loads(sched));
    SitePos pos[PP];
    SiteDraw dr[PP];
    SiteB q[PP];
    if (One) {
        PhiloxRun call = site_call<PP>(first, 0u, threadIdx.x, d.key0, d.key1);
        philox_rounds<10>(call);
        site_draws<PP>(call, threadIdx.x, dr);
#pragma unroll
        for (int h = 0; h < PP; ++h) {
            pos[h] = site_pos(mine ? threadIdx.x * PP + (uint32_t)h : 0u, L, Lq, N, magicLq);
            q[h] = site_b<0>(pos[h], L, N, sc);
        }
    }
    uint32_t left = every, k = 0;  // sweeps left of interval k
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t s = first + i;
        SweepWords next = sc;
        SweepLoads coming{};  // of the next sweep's schedule
        uint32_t packed = 0u;  // One: at most 8 accepted moves a sweep
        auto phase = [&](auto pc) {
            constexpr int P = decltype(pc)::value;
            constexpr int P1 = (P + 1) & 3;
            // the words of the next kSchedSweeps sweeps, into the half of the
            // buffer that was last read a sweep or more ago
            const uint32_t j = i + 1u;
            if (P == 0 && j % kSchedSweeps == 0 && j < n)
                make_schedules(sched + 12u * (j % (2u * kSchedSweeps)), s + 1, n - j, d.key0, d.key1, L);
            if (P == 2) coming = sweep_loads(sched + 12u * (j % (2u * kSchedSweeps)));
            if (P == 3) next = sweep_words(coming);
            if (One) {
                if (mine) {
                    SiteDraw nd[PP];
                    PhiloxRun call = site_call<PP>(P < 3 ? s : s + 1, P1, threadIdx.x, d.key0, d.key1);
                    auto next_b = [&](int h) {
                        return site_b<P1>(pos[h], L, N, P < 3 ? sc : next);
                    };
                    if constexpr (PP == 1) {
                        // The next phase's call in three parts between the stages:
                        // left to itself the compiler draws first and loads then
                        // (L = 32, 100 intervals of 10 sweeps: 1690 us, so 1460).
                        const uint32_t b = q[0].b;
                        const SiteLoads v = site_load<P>(lat, pos[0], q[0], L);
                        __builtin_amdgcn_sched_barrier(0);
                        philox_rounds<4>(call);
                        __builtin_amdgcn_sched_barrier(0);
                        const SiteMove m = site_move(v, dr[0], s_trans);
                        __builtin_amdgcn_sched_barrier(0);
                        philox_rounds<3>(call);
                        __builtin_amdgcn_sched_barrier(0);
                        const uint2 e = site_entry(m, s_tab);
                        __builtin_amdgcn_sched_barrier(0);
                        philox_rounds<3>(call);
                        site_draws<PP>(call, threadIdx.x, nd);
                        q[0] = next_b(0);
                        __builtin_amdgcn_sched_barrier(0);
                        site_store<P>(lat, pos[0], b, dr[0], m, e, packed);
                        dr[0] = nd[0];
                    } else {
                        // two pairs a thread have enough waves to fill the gaps
                        // (40 of L = 100, 50 sweeps: in stages 241 us, so 227)
                        philox_rounds<10>(call);
                        site_draws<PP>(call, threadIdx.x, nd);
#pragma unroll
                        for (int h = 0; h < PP; ++h) {
                            const SiteMove m = site_move(site_load<P>(lat, pos[h], q[h], L), dr[h], s_trans);
                            site_store<P>(lat, pos[h], q[h].b, dr[h], m, site_entry(m, s_tab), packed);
                            dr[h] = nd[h];
                            q[h] = next_b(h);
                        }
                    }
                }
            } else {
                for (uint32_t t = threadIdx.x; t < tasks; t += blockDim.x) {
                    PhiloxRun call = site_call<PP>(s, P, t, d.key0, d.key1);
                    philox_rounds<10>(call);
                    site_draws<PP>(call, t, dr);
                    packed = 0u;
#pragma unroll
                    for (int h = 0; h < PP; ++h) {
                        const SitePos at = site_pos(t * PP + (uint32_t)h, L, Lq, N, magicLq);
                        const SiteB to = site_b<P>(at, L, N, sc);
                        const SiteMove m = site_move(site_load<P>(lat, at, to, L), dr[h], s_trans);
                        site_store<P>(lat, at, to.b, dr[h], m, site_entry(m, s_tab), packed);
                    }
                    unpack_tracker(packed, tr);
                }
            }
            __syncthreads();
        };
        phase(std::integral_constant<int, 0>{});
        phase(std::integral_constant<int, 1>{});
        phase(std::integral_constant<int, 2>{});
        phase(std::integral_constant<int, 3>{});
        sc = next;
        if (One) unpack_tracker(packed, tr);
        if (--left == 0) {
            observe(k);
            ++k;
            left = every;
        }
    }
}

// This thread's share of the seven observable sums.
__device__ __forceinline__ void site_observables(const uint32_t *lat, uint32_t L, uint32_t magicLq, int (&v)[7])
{
    const uint32_t Lq = L >> 2, n = L * Lq;
    SiteSums sums;
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t y = Lq == 1u ? i : __umulhi(i, magicLq), X = i - y * Lq, w = lat[i];
        const uint32_t w1 = lat[X + 1u == Lq ? i + 1u - Lq : i + 1u];
        sums.add(w, __builtin_amdgcn_alignbit(w1, w, 8u), lat[y + 1u == L ? X : i + Lq], row_signs(y));
    }
    sums.get(v);
}

__global__ void __launch_bounds__(1024) k_sweep_site(BatchArgs args)
{
    __shared__ __align__(16) uint2 s_tab[kDevTabEntries + 1];
    __shared__ __align__(16) uint32_t s_trans[2 * 256];
    __shared__ uint32_t sched[2 * 12 * kSchedSweeps];
    __shared__ ObsStage obs;
    extern __shared__ __align__(16) uint32_t lat[];
    uint8_t *scr = args.scratch[blockIdx.x];
    const LatDesc d = *(const LatDesc *)(scr + kScrDesc);
    {
        const uint2 *g_tab = (const uint2 *)(scr + kScrDevTab);
        for (int i = threadIdx.x; i < kDevTabEntries; i += blockDim.x) s_tab[i] = g_tab[i];
        for (int i = threadIdx.x; i < 2 * 256; i += blockDim.x) s_trans[i] = kSiteSlots.v[i];
    }
    stage_sites(lat, d);
    if (args.obs_out) tracker_before(scr, obs);
    __syncthreads();

    const uint32_t L = (uint32_t)d.L, N = L * L, my_sweeps = args.sweeps[blockIdx.x];
    const uint32_t intervals = args.obs_out ? args.intervals : 1u;
    const bool single = N / 8u <= min(blockDim.x, kSiteOnePair), one = N / 16u <= blockDim.x;
    const uint8_t *tab = (const uint8_t *)s_tab, *trans = (const uint8_t *)s_trans;
    const uint32_t magicLq = L == 4u ? 0u : 0xFFFFFFFFu / (L >> 2) + 1u;
    int tr[3] = {0, 0, 0};
    auto observe = [&](uint32_t k) {
        if (!args.obs_out) return;
        int o[7];
        site_observables(lat, L, magicLq, o);
        write_record(args, obs, tr, o, k, d.next_sweep + (uint64_t)my_sweeps * (k + 1u));
    };
    if (my_sweeps > 0) {
        uint8_t *bytes = (uint8_t *)lat;
        if (single)
            site_sweeps<1, true>(bytes, sched, d, d.next_sweep, intervals, my_sweeps, tab, trans, tr, observe);
        else if (one)
            site_sweeps<2, true>(bytes, sched, d, d.next_sweep, intervals, my_sweeps, tab, trans, tr, observe);
        else
            site_sweeps<2, false>(bytes, sched, d, d.next_sweep, intervals, my_sweeps, tab, trans, tr, observe);
    }
    unstage_sites(lat, d);
    if (threadIdx.x == 0) ((LatDesc *)(scr + kScrDesc))->next_sweep = d.next_sweep + (uint64_t)my_sweeps * intervals;
    block_reduce_add<3>(tr, (unsigned long long *)(scr + kScrTrackBase));
}

// ---------------------------------------------------------------------------
// Half-byte form, for sides above kSiteMaxL up to kLdsMaxL, whose bytes do not
// fit: row-major, sites 2j and 2j + 1 as the codes in the low and the high half of
// byte j.  In a phase only one site of a byte can change (the updated sites of a
// row are of one class), so its pair's lane writes the byte with a plain store;
// a site's byte also holds one of its two neighbours in the row, and which half
// any of them is in depends on the phase alone.
//
// One compute unit takes longer for such a lattice than the whole chip (a lattice
// of L = 500 116 us a sweep, spread over the chip 13.6), so this form is for
// calls that bring many: 256 of L = 500, 20 sweeps, 6460 us together on the chip,
// 3370 with two bits a site in LDS and atomics, 2371 in this form; of L = 388 4945, 2066 and 1451.
template <int P>
__device__ __forceinline__ void half_step(uint8_t *lat, const SitePos &s, const SiteB &q, uint32_t L, uint32_t pb,
                                          uint32_t slot8, uint32_t ua, const uint2 *s_tab, const uint8_t *s_slots,
                                          uint32_t &packed)
{
    constexpr uint32_t ha = 4u * (P & 1u);
    const uint32_t hb = 4u * (pb & 1u);
    const uint32_t a = (s.a + P) >> 1, b = q.b >> 1;
    // the neighbour beside the byte: the left one of an even x, the right one of an odd x
    const uint32_t ea = P == 0 ? s.l : P == 3 ? s.r : P == 1 ? s.a + 2u : s.a + 1u;
    const uint32_t A = lat[a], B = lat[b], Ae = lat[ea >> 1], Be = lat[(hb ? q.r : q.l) >> 1];
    const uint32_t Au = lat[(s.u + P) >> 1], Ad = lat[(s.d + P) >> 1], Bu = lat[(q.b - L) >> 1], Bd = lat[q.d >> 1];
    const uint32_t ca = (A >> ha) & 3u, cb = (B >> hb) & 3u;
    const uint32_t bpack = contrib_a((A >> (4u - ha)) & 3u) + contrib_a((Ae >> (4u - ha)) & 3u) + contrib_a((Au >> ha) & 3u) +
                           contrib_a((Ad >> ha) & 3u) + contrib_b((B >> (4u - hb)) & 3u) + contrib_b((Be >> (4u - hb)) & 3u) +
                           contrib_b((Bu >> hb) & 3u) + contrib_b((Bd >> hb) & 3u);
    uint32_t change = 0u;
    pair_step_slot((ca | cb << 2) << 7 | slot8, bpack, ua, s_slots, s_tab, 0x03030000u, packed, change);
    lat[a] = (uint8_t)(A ^ ((change >> 16) & 3u) << ha);
    lat[b] = (uint8_t)(B ^ (change >> 24) << hb);
}

// Four codes, one a byte, to two bytes of this form, and back.
__device__ __forceinline__ uint32_t halves_of(uint32_t c)
{
    const uint32_t x = c & 0x03030303u, y = x | x >> 4;
    return (y & 0xFFu) | (y >> 8 & 0xFF00u);
}
__device__ __forceinline__ uint32_t codes_of_halves(uint32_t h)
{
    const uint32_t x = (h & 0xFFu) | (h & 0xFF00u) << 8;
    return (x & 0x00030003u) | (x & 0x00300030u) << 4;
}

__device__ __forceinline__ void stage_halves(uint16_t *lat, const LatDesc &d)
{
    const uint32_t L = (uint32_t)d.L;
    if (d.enc == 0) {
        const LAT_GLOBAL word_any *src = (const LAT_GLOBAL word_any *)d.state;
        for (uint32_t i = threadIdx.x; i < L * L / 4u; i += blockDim.x) lat[i] = (uint16_t)halves_of(src[i]);
    } else {
        // words j of the four classes of a row: 64 sites of it
        const LAT_GLOBAL uint32_t *src = (const LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = L >> 6, csz = (L >> 1) * W;
        for (uint32_t i = threadIdx.x; i < L * W; i += blockDim.x) {
            const uint32_t y = i / W, j = i - y * W, at = 4u * (y & 1u) * csz + (y >> 1) * W + j;
            const uint32_t w0 = src[at], w1 = src[at + csz], w2 = src[at + 2u * csz], w3 = src[at + 3u * csz];
            for (uint32_t t = 0; t < 16u; ++t)
                lat[16u * i + t] = (uint16_t)(((w0 >> 2u * t) & 3u) | ((w1 >> 2u * t) & 3u) << 4 | ((w2 >> 2u * t) & 3u) << 8 |
                                              ((w3 >> 2u * t) & 3u) << 12);
        }
    }
}

__device__ __forceinline__ void unstage_halves(const uint16_t *lat, const LatDesc &d)
{
    const uint32_t L = (uint32_t)d.L;
    if (d.enc == 0) {
        LAT_GLOBAL word_any *dst = (LAT_GLOBAL word_any *)d.state;
        for (uint32_t i = threadIdx.x; i < L * L / 4u; i += blockDim.x) dst[i] = codes_of_halves(lat[i]);
    } else {
        LAT_GLOBAL uint32_t *dst = (LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = L >> 6, csz = (L >> 1) * W;
        for (uint32_t i = threadIdx.x; i < L * W; i += blockDim.x) {
            const uint32_t y = i / W, j = i - y * W, at = 4u * (y & 1u) * csz + (y >> 1) * W + j;
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            for (uint32_t t = 0; t < 16u; ++t)
#pragma unroll
                for (uint32_t c = 0; c < 4u; ++c) w[c] |= ((uint32_t)lat[16u * i + t] >> (4u * c) & 3u) << (2u * t);
#pragma unroll
            for (uint32_t c = 0; c < 4u; ++c) dst[at + c * csz] = w[c];
        }
    }
}

// This thread's share of the seven observable sums.
__device__ __forceinline__ void half_observables(const uint16_t *lat, uint32_t L, uint32_t magicLq, int (&v)[7])
{
    const uint32_t Lq = L >> 2, n = L * Lq;
    auto sites = [&](uint32_t i) { return site_from_codes(codes_of_halves(lat[i])); };
    SiteSums sums;
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t y = Lq == 1u ? i : __umulhi(i, magicLq), X = i - y * Lq, w = sites(i);
        const uint32_t w1 = sites(X + 1u == Lq ? i + 1u - Lq : i + 1u);
        sums.add(w, __builtin_amdgcn_alignbit(w1, w, 8u), sites(y + 1u == L ? X : i + Lq), row_signs(y));
    }
    sums.get(v);
}

__global__ void __launch_bounds__(1024) k_sweep_half(BatchArgs args)
{
    __shared__ __align__(16) uint2 s_tab[kDevTabEntries + 1];
    __shared__ __align__(16) uint2 s_slots[kSlotEntries];
    __shared__ uint32_t sched[2 * 12 * kSchedSweeps];
    __shared__ ObsStage obs;
    extern __shared__ uint32_t smem[];
    uint8_t *lat = (uint8_t *)smem;
    uint8_t *scr = args.scratch[blockIdx.x];
    const LatDesc d = *(const LatDesc *)(scr + kScrDesc);
    {
        const uint2 *g_tab = (const uint2 *)(scr + kScrDevTab), *g_slots = (const uint2 *)kWordSlots.v;
        for (int i = threadIdx.x; i < kDevTabEntries; i += blockDim.x) s_tab[i] = g_tab[i];
        for (int i = threadIdx.x; i < kSlotEntries; i += blockDim.x) s_slots[i] = g_slots[i];
    }
    stage_halves((uint16_t *)lat, d);
    if (args.obs_out) tracker_before(scr, obs);
    const uint32_t L = (uint32_t)d.L, Lq = L >> 2, N = L * L, my_sweeps = args.sweeps[blockIdx.x];
    const uint32_t intervals = args.obs_out ? args.intervals : 1u, n = intervals * my_sweeps;
    const uint32_t magicLq = Lq == 1u ? 0u : 0xFFFFFFFFu / Lq + 1u;
    if (n > 0) make_schedules(sched, d.next_sweep, n, d.key0, d.key1, L);
    __syncthreads();
    int tr[3] = {0, 0, 0};
    uint32_t left = my_sweeps, k = 0;  // sweeps left of interval k
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t s = d.next_sweep + i;
        const SweepWords sc = sweep_words(sweep_loads(sched + 12u * (i % (2u * kSchedSweeps))));
        auto phase = [&](auto pc) {
            constexpr int P = decltype(pc)::value;
            const uint32_t j = i + 1u;
            if (P == 0 && j % kSchedSweeps == 0 && j < n)
                make_schedules(sched + 12u * (j % (2u * kSchedSweeps)), s + 1, n - j, d.key0, d.key1, L);
            const uint32_t pb = (P + sc.r) & 3u;
            for (uint32_t t = threadIdx.x; t < N / 16u; t += blockDim.x) {
                const u32x4 w = pair_draws(philox4x32_10((uint32_t)s, (uint32_t)P, t, (uint32_t)(s >> 32), d.key0, d.key1));
                uint32_t packed = 0u;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const SitePos at = site_pos(2u * t + (uint32_t)h, L, Lq, N, magicLq);
                    half_step<P>(lat, at, site_b<P>(at, L, N, sc), L, pb, h ? w.z : w.x, h ? w.w : w.y, s_tab,
                                 (const uint8_t *)s_slots, packed);
                }
                unpack_tracker(packed, tr);
            }
            __syncthreads();
        };
        phase(std::integral_constant<int, 0>{});
        phase(std::integral_constant<int, 1>{});
        phase(std::integral_constant<int, 2>{});
        phase(std::integral_constant<int, 3>{});
        if (--left == 0) {
            if (args.obs_out) {
                int o[7];
                half_observables((const uint16_t *)lat, L, magicLq, o);
                write_record(args, obs, tr, o, k, d.next_sweep + (uint64_t)my_sweeps * (k + 1u));
            }
            ++k;
            left = my_sweeps;
        }
    }
    unstage_halves((const uint16_t *)lat, d);
    if (threadIdx.x == 0) ((LatDesc *)(scr + kScrDesc))->next_sweep = d.next_sweep + n;
    block_reduce_add<3>(tr, (unsigned long long *)(scr + kScrTrackBase));
}

__global__ void k_advance(LatDesc *desc, uint32_t sweeps)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) desc->next_sweep += sweeps;
}

// Observables of many lattices from their global state: block b reduces
// lattice b and writes (tracker, 7 sums) to out[10b ..].
__global__ void __launch_bounds__(256) k_obs_batch(BatchArgs args, unsigned long long *out)
{
    uint8_t *scr = args.scratch[blockIdx.x];
    const LatDesc d = *(const LatDesc *)(scr + kScrDesc);
    const int L = d.L;
    long long v[7] = {0, 0, 0, 0, 0, 0, 0};
    if (d.enc == 0) {
        const uint8_t *st = (const uint8_t *)d.state;
        SiteSums sums;
        if (L % 16 == 0 && ((uintptr_t)st & 15u) == 0)
            for (uint32_t t = threadIdx.x; t < (uint32_t)L * L / 16u; t += blockDim.x)
                obs_group_int8<4>(st, (uint32_t)L, t, sums);
        else
            for (uint32_t t = threadIdx.x; t < (uint32_t)L * L / 4u; t += blockDim.x)
                obs_group_int8<1>(st, (uint32_t)L, t, sums);
        sums.get(v);
    } else {
        for (uint32_t i = threadIdx.x; i < (uint32_t)L * L / 16u; i += blockDim.x)
            obs_word_2bit((const uint32_t *)d.state, (uint32_t)L, i, v);
    }
    unsigned long long *o = out + 10 * (size_t)blockIdx.x;
    if (threadIdx.x < 10) o[threadIdx.x] = 0ull;
    __syncthreads();
    block_reduce_add<7>(v, o + 3);
    long long t3[3] = {0, 0, 0};
    tracker_partial(scr, t3);
    block_reduce_add<3>(t3, o);
}

}  // namespace

hipError_t init_kernel_attributes()
{
    // allow more than the default 64 KiB of dynamic LDS
    hipError_t e = hipFuncSetAttribute((const void *)k_sweep_site, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kSiteMaxL * kSiteMaxL);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k_sweep_half, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMaxL * kLdsMaxL / 2);
    if (e == hipSuccess) e = init_quad_kernel_attributes();
    return e;
}

hipError_t launch_sweep_lds(const BatchArgs &a, int max_L, int threads, bool quad, hipStream_t s)
{
    if (quad) return launch_sweep_quad(a, max_L, threads, s);
    // default block: one thread per pair up to kSiteOnePair pairs a phase, else
    // one per Philox call (two pairs)
    const uint32_t sq = (uint32_t)max_L * (uint32_t)max_L;
    const uint32_t units = sq / 8u <= kSiteOnePair ? sq / 8u : sq / 16u;
    uint32_t block = std::min(1024u, (units + 63u) / 64u * 64u);
    if (threads > 0) block = (uint32_t)std::min(1024, std::max(64, threads / 64 * 64));
    if (max_L > kSiteMaxL)
        hipLaunchKernelGGL(k_sweep_half, dim3((unsigned)a.count), dim3(block), (size_t)sq / 2, s, a);
    else
        hipLaunchKernelGGL(k_sweep_site, dim3((unsigned)a.count), dim3(block), (size_t)sq, s, a);
    return hipGetLastError();
}

hipError_t launch_advance(LatDesc *desc, uint32_t sweeps, hipStream_t s)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, desc, sweeps);
    return hipGetLastError();
}

hipError_t launch_observables_batch(const BatchArgs &a, unsigned long long *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_obs_batch, dim3((unsigned)a.count), dim3(256), 0, s, a, out);
    return hipGetLastError();
}

}  // namespace lat
