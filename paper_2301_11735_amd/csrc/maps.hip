// gfx950 kernel of the map mode (arXiv:2301.11735 section 3.2): the paper's
// random maps of non-interacting coupled pairs, built on the device.
//
// One block per lattice (up to 256 lattices per launch, L <= 256).  Per map:
//   1. the block clears a bitmap of marked sites;
//   2. one wave a map builds it with the paper's sequential algorithm -- draw
//      a site until an unmarked one comes up, mark it; the same for the
//      partner; record the pair; mark the neighbours of both -- taking 64
//      draws at a time (build_map), or one after another for the smallest
//      lattices (walk_map); the block's waves build the next maps of the launch
//      side by side;
//   3. all threads apply one coupled-pair Metropolis step (section 3.1) to the
//      map's pairs in parallel.  No two pairs of a map interact, so this equals
//      applying them one after another; a pair's own sites may be neighbours,
//      and the bond between them then enters the energy change once.
// The codes (one byte per site), the bitmap, the pair list and the full
// threshold table over (nD, nV, nJ) live in LDS for all maps of the launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.h"

namespace lat {
namespace {

constexpr uint32_t kDomMap = 0x400u;      // site draws of a map's construction
constexpr uint32_t kDomMapStep = 0x500u;  // configuration and acceptance draws of its pairs

// Same-charge configurations of a pair (section 3.1 listing), nibble j of the
// constant for q = +1, 0, -1 holding code_a | code_b << 2.
constexpr uint32_t kSetQp1 = 0x9862u;    // (2,0) (2,1) (0,2) (1,2)
constexpr uint32_t kSetQ0 = 0x1450BEu;   // (2,3) (3,2) (0,0) (1,1) (0,1) (1,0)
constexpr uint32_t kSetQm1 = 0xDC73u;    // (3,0) (3,1) (0,3) (1,3)

__device__ __forceinline__ int sigma_of(uint32_t c) { return (c & 2u) ? 0 : 1 - 2 * (int)(c & 1u); }

// Sites s < 2^16 and sides L <= 256: y = s / L from magic = ceil(2^32 / L)
// (the rounding error s (magic L - 2^32) stays below 2^24).
__device__ __forceinline__ void site_neighbours(int L, uint32_t magic, uint32_t s, uint32_t (&nb)[4])
{
    const uint32_t y = __umulhi(s, magic), row = y * (uint32_t)L, x = s - row;
    nb[0] = row + (x + 1 == (uint32_t)L ? 0 : x + 1);
    nb[1] = row + (x == 0 ? (uint32_t)L - 1 : x - 1);
    nb[2] = (y + 1 == (uint32_t)L ? 0 : row + (uint32_t)L) + x;
    nb[3] = (y == 0 ? (uint32_t)L * ((uint32_t)L - 1) : row - (uint32_t)L) + x;
}

__device__ __forceinline__ uint32_t marked(const uint32_t *bitmap, uint32_t s)
{
    return (__hip_atomic_load(&bitmap[s >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >> (s & 31u)) & 1u;
}
__device__ __forceinline__ uint32_t mark(uint32_t *bitmap, uint32_t s)
{
    return (atomicOr(&bitmap[s >> 5], 1u << (s & 31u)) >> (s & 31u)) & 1u;  // was it marked?
}
__device__ __forceinline__ void unmark(uint32_t *bitmap, uint32_t s) { atomicAnd(&bitmap[s >> 5], ~(1u << (s & 31u))); }

__device__ __forceinline__ uint32_t rank_in(uint64_t mask)  // set bits of the mask below this lane
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Map m into pairs[] (a in the low half, b in the high half), by the calling
// wave (several waves of a block build different maps at once, each in its
// own bitmap).  The paper's walk over the draws is sequential, but its
// outcome only depends on the order where two draws interact: a draw is
// taken unless its site is marked, and taking it marks it and (once its pair
// is whole) its neighbours.  So the wave takes the next 64 draws at once:
//   1. lanes whose site is unmarked are candidates; each marks its site
//      tentatively and then looks whether a neighbour's mark is new, or its
//      own was set by another lane (one of two equal sites sees that, and
//      the other is found by comparison);
//   2. a candidate that saw nothing is what the walk takes, whatever the
//      others do; those that did are decided in order, by comparing their
//      site with all lanes: one is rejected if an accepted lane before it has
//      the same site, or is next to it and belongs to a pair that is whole by
//      then (a site carried over from the window before likewise);
//   3. the marks of rejected candidates are withdrawn, the accepted sites get
//      their place in the pair list by their rank, and the neighbours of
//      whole pairs are marked.
// A mark never goes away once its draw is accepted, so a draw rejected
// against the marks before the window is rejected in the walk as well.  A
// pair without its second site at the end of a window carries over.
//
// The build is bound by the chain of dependent LDS operations of a window
// (about five) and by the draws decided in order, not by bandwidth; a walk one draw at a time took a chain of LDS round trips per
// candidate.  A call on 256 lattices of L = 128, 10 maps each: 2098 -> 213 us.
//
// NN (nearest-neighbour partners): a draw on an unmarked site takes the
// next draw as its direction.  Runs of unmarked draws are independent (the
// draw before a run is marked: rejected, or the direction of the run before),
// so the first sites are the draws of each run at even distance from its
// start: runs that start on an even lane are the bits of U that the carry of
// U + (their starts) clears.  A dropped pair (marked partner) still marks its
// first site tentatively, since whether that draw is a first site at all
// depends on the pairs before it.  An interaction moves the first sites after
// it, so here a window ends before the first lane f that saw one (after f if
// its own sites were not double: its neighbours then are all later lanes, and
// always if it is the first), and the next one starts there.
template <bool NN>
__device__ void build_map(uint32_t *bitmap, uint32_t *pairs, int L, uint32_t magic, uint32_t N, uint32_t n_pairs,
                          uint32_t m_lo, uint32_t m_hi, uint32_t key0, uint32_t key1)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t self = 1ull << lane;
    uint16_t *half = (uint16_t *)pairs;  // half[2 i] = a, half[2 i + 1] = b of pair i
    uint32_t k = 0, count = 0, pend = 0, pend_site = 0;
    uint32_t base = 0;  // lane l holds draws base + 4 l .. + 3
    u32x4 w = philox4x32_10(m_lo, kDomMap, lane, m_hi, key0, key1);
    while (count < n_pairs) {
        if (k - base > 192u) {  // the window's 64 draws are not all held
            base = k & ~3u;
            w = philox4x32_10(m_lo, kDomMap, (base >> 2) + lane, m_hi, key0, key1);
        }
        const uint32_t d = k - base + lane;  // < 256
        const int from = (int)(d >> 2);
        const uint32_t r0 = __shfl(w.x, from, 64), r1 = __shfl(w.y, from, 64), r2 = __shfl(w.z, from, 64),
                       r3 = __shfl(w.w, from, 64);
        const uint32_t raw = d & 2u ? (d & 1u ? r3 : r2) : (d & 1u ? r1 : r0);
        const uint32_t a = mulhi_u32(raw, N);
        uint32_t an[4], was[4];
        site_neighbours(L, magic, a, an);
        const uint32_t was_a = marked(bitmap, a);
#pragma unroll
        for (int e = 0; e < 4; ++e) was[e] = marked(bitmap, an[e]);
        if constexpr (!NN) {
            const bool cand = !was_a;
            const uint64_t C = __ballot(cand);
            if (C == 0) {
                k += 64u;
                continue;
            }
            uint32_t dup = 0, hit = 0, carried = 0;
            if (cand) dup = mark(bitmap, a);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                hit |= marked(bitmap, an[e]) & ~was[e];
                carried |= pend && an[e] == pend_site;
            }
            // candidates that interact with another one or with the carried site
            uint64_t F = __ballot(cand && (dup | hit | carried));
            for (uint64_t D = __ballot(cand && dup); D; D &= D - 1ull)
                F |= __ballot(cand && a == (uint32_t)__builtin_amdgcn_readlane((int)a, (int)__builtin_ctzll(D)));
            const uint64_t P = __ballot(carried);
            uint64_t acc = C & ~F;
            for (uint64_t rest = F; rest; rest &= rest - 1ull) {
                const int j = (int)__builtin_ctzll(rest);
                const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)a, j);
                const uint64_t before = acc & ((1ull << j) - 1ull);  // all decided
                // a first site that waits for its partner has not marked its neighbours
                const bool waiting = ((uint32_t)__popcll(before) + pend) & 1u;
                const uint64_t last = waiting && before ? 1ull << (63 - (int)__builtin_clzll(before)) : 0ull;
                const uint64_t same = __ballot(a == t);
                const uint64_t next_to = __ballot(an[0] == t || an[1] == t || an[2] == t || an[3] == t);
                const bool taken_before = (before & (same | (next_to & ~last))) != 0 || (before && ((P >> j) & 1u));
                if (!taken_before) acc |= 1ull << j;
            }
            const uint32_t left = 2u * (n_pairs - count) - pend;  // sites the map still takes
            const uint32_t rank = rank_in(acc);
            acc = __ballot((acc & self) && rank < left);
            const bool mine = acc & self;
            if (F || acc != C) {
                __builtin_amdgcn_wave_barrier();
                if (cand && !mine) unmark(bitmap, a);
                __builtin_amdgcn_wave_barrier();
                if (mine) mark(bitmap, a);  // a withdrawn double shared its bit
            }
            const uint32_t sites = (uint32_t)__popcll(acc) + pend, whole = sites >> 1;
            const uint32_t r = rank + pend;
            if (mine) {
                half[2u * count + r] = (uint16_t)a;
                if ((r >> 1) < whole) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) mark(bitmap, an[e]);
                }
            }
            if (pend && whole > 0 && lane < 4u) {  // the carried first site's neighbours
                uint32_t pn[4];
                site_neighbours(L, magic, pend_site, pn);
                mark(bitmap, lane == 0 ? pn[0] : lane == 1 ? pn[1] : lane == 2 ? pn[2] : pn[3]);
            }
            if (sites & 1u) {
                // the last accepted site waits for its partner (none accepted: the carried one still does)
                if (acc) pend_site = (uint32_t)__builtin_amdgcn_readlane((int)a, 63 - (int)__builtin_clzll(acc));
                pend = 1u;
            } else {
                pend = 0u;
            }
            count += whole;
            k += 64u;
        } else {
            const uint64_t kEven = 0x5555555555555555ull;
            const uint64_t U = __ballot(!was_a);
            const uint64_t even_starts = U & ~(U << 1) & kEven;
            const uint64_t even_runs = U & ~(U + even_starts);
            uint64_t C = (even_runs & kEven) | (U & ~even_runs & ~kEven);
            uint32_t taken = (C >> 63) ? 63u : 64u;  // a first site on the last lane waits for the next window
            C &= ~(1ull << 63);
            if (C == 0) {
                k += taken;
                continue;
            }
            const uint32_t dir = __shfl_down(raw, 1, 64) >> 30;
            const uint32_t b = dir == 0 ? an[0] : dir == 1 ? an[1] : dir == 2 ? an[2] : an[3];
            const uint32_t was_b = dir == 0 ? was[0] : dir == 1 ? was[1] : dir == 2 ? was[2] : was[3];
            uint32_t bn[4], wasb[4];
            site_neighbours(L, magic, b, bn);
#pragma unroll
            for (int e = 0; e < 4; ++e) wasb[e] = marked(bitmap, bn[e]);
            const bool cand = C & self, keep = cand && !was_b;
            uint32_t dup = 0, hit = 0;
            if (cand) dup = mark(bitmap, a);
            if (keep) dup |= mark(bitmap, b);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (!(keep && an[e] == b)) hit |= marked(bitmap, an[e]) & ~was[e];
                if (keep && bn[e] != a) hit |= marked(bitmap, bn[e]) & ~wasb[e];
            }
            const uint64_t F = __ballot(cand && (dup | hit));
            uint64_t acc = C;
            if (F) {
                const uint32_t f = (uint32_t)__builtin_ctzll(F);
                const uint64_t D = __ballot(cand && dup);
                const bool with_f = f == (uint32_t)__builtin_ctzll(C) || !((D >> f) & 1u);
                acc = C & ((1ull << f) - 1ull);
                if (with_f) acc |= 1ull << f;
                taken = with_f ? f + 2u : f;
            }
            acc = __ballot((acc & self) && keep);
            const uint32_t rank = rank_in(acc);
            acc = __ballot((acc & self) && rank < n_pairs - count);
            const bool mine = acc & self;
            __builtin_amdgcn_wave_barrier();
            if (cand && !mine) {
                unmark(bitmap, a);
                if (keep) unmark(bitmap, b);
            }
            __builtin_amdgcn_wave_barrier();
            if (mine) {
                pairs[count + rank] = a | (b << 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {  // a and b are among each other's neighbours
                    mark(bitmap, an[e]);
                    mark(bitmap, bn[e]);
                }
            }
            count += (uint32_t)__popcll(acc);
            k += taken;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// The same map by the walk itself, one draw after another with uniform control
// flow, for the smallest lattices: there most of a window's 64 draws interact or
// are not needed.  The lanes hold the next 256 draws; a draw that was marked when
// they were taken is rejected without touching LDS, any other is looked up in
// the live bitmap (a broadcast read, behind the marks already issued).
template <bool NN>
__device__ __forceinline__ void walk_map(uint32_t *bitmap, uint32_t *pairs, int L, uint32_t magic, uint32_t N,
                                         uint32_t n_pairs, uint32_t m_lo, uint32_t m_hi, uint32_t key0, uint32_t key1)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t k = 0, count = 0, site_a = 0;
    bool pend = false;              // site_a waits for its partner
    uint32_t an[4] = {0, 0, 0, 0};  // its neighbours
    auto all = [](uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    auto is_marked = [&](uint32_t s) { return __builtin_amdgcn_readfirstlane((int)marked(bitmap, s)) != 0; };
    while (count < n_pairs) {
        const u32x4 w = philox4x32_10(m_lo, kDomMap, (k >> 2) + lane, m_hi, key0, key1);
        const uint32_t raw[4] = {w.x, w.y, w.z, w.w};
        uint32_t site[4], nb[4][4];
        uint64_t was[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            site[q] = mulhi_u32(raw[q], N);
            site_neighbours(L, magic, site[q], nb[q]);
            was[q] = __ballot(marked(bitmap, site[q]));
        }
        for (int l = 0; l < 64 && count < n_pairs; ++l) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (count >= n_pairs) continue;
                uint32_t b, bn[4];
                if (NN && pend) {  // the draw's direction picks b
                    const uint32_t dir = all(raw[q], l) >> 30;
                    b = dir == 0 ? an[0] : dir == 1 ? an[1] : dir == 2 ? an[2] : an[3];
                    pend = false;
                    if (is_marked(b)) continue;
                    site_neighbours(L, magic, b, bn);
                    if (lane == 0) mark(bitmap, site_a);
                } else {
                    if ((was[q] >> l) & 1u) continue;
                    b = all(site[q], l);
                    if (is_marked(b)) continue;
#pragma unroll
                    for (int e = 0; e < 4; ++e) bn[e] = all(nb[q][e], l);
                    if (!pend) {
                        if (!NN && lane == 0) mark(bitmap, b);
                        site_a = b;
#pragma unroll
                        for (int e = 0; e < 4; ++e) an[e] = bn[e];
                        pend = true;
                        continue;
                    }
                    pend = false;
                }
                if (lane == 0) {
                    pairs[count] = site_a | (b << 16);
                    mark(bitmap, b);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        mark(bitmap, an[e]);
                        mark(bitmap, bn[e]);
                    }
                }
                ++count;
            }
        }
        k += 256u;
    }
}

// Sums of S and sigma over the neighbours of s other than `other`; adj = 1 if
// `other` is one of them.
__device__ __forceinline__ void side_sum(const uint8_t *codes, int L, uint32_t magic, uint32_t s, uint32_t other,
                                         int &sS, int &sG, int &adj)
{
    uint32_t nb[4];
    site_neighbours(L, magic, s, nb);
    sS = 0;
    sG = 0;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (nb[d] == other) {
            adj = 1;
            continue;
        }
        const uint32_t c = codes[nb[d]];
        sS += charge_of(c);
        sG += sigma_of(c);
    }
}

// One coupled-pair Metropolis step on sites (a, b), a and b possibly adjacent.
__device__ __forceinline__ void map_pair_step(uint8_t *codes, const uint32_t *thr, int L, uint32_t magic,
                                              uint32_t a, uint32_t b, uint32_t uc, uint32_t ua, int (&tr)[3])
{
    const uint32_t ca = codes[a], cb = codes[b];
    const int Sa = charge_of(ca), Sb = charge_of(cb), q = Sa + Sb;
    if (q == 2 || q == -2) return;
    const uint32_t kq = q == 0 ? 6u : 4u;
    const uint32_t j = ((uc >> 8) * kq) >> 24;
    const uint32_t cfg = ((q == 1 ? kSetQp1 : q == 0 ? kSetQ0 : kSetQm1) >> (4u * j)) & 15u;
    const uint32_t na = cfg & 3u, nb = cfg >> 2;
    int sSa, sGa, sSb, sGb, adj = 0;
    side_sum(codes, L, magic, a, b, sSa, sGa, adj);
    side_sum(codes, L, magic, b, a, sSb, sGb, adj);
    const int Ga = sigma_of(ca), Gb = sigma_of(cb);
    const int Sna = charge_of(na), Snb = charge_of(nb), Gna = sigma_of(na), Gnb = sigma_of(nb);
    const int nD = Sna * Sna - Sa * Sa + Snb * Snb - Sb * Sb;
    const int nV = (Sna - Sa) * sSa + (Snb - Sb) * sSb + adj * (Sna * Snb - Sa * Sb);
    const int nJ = (Gna - Ga) * sGa + (Gnb - Gb) * sGb + adj * (Gna * Gnb - Ga * Gb);
    const uint32_t t = thr[(nD + 2) * (kTabV * kTabJ) + (nV + 16) * kTabJ + (nJ + 16)];
    if (min(ua, 0xFFFFFFFEu) < t) {
        codes[a] = (uint8_t)na;
        codes[b] = (uint8_t)nb;
        tr[0] += nD;
        tr[1] += nV;
        tr[2] += nJ;
    }
}

// Largest sides of the walk, for either partner rule.
// us a call of 256 lattices, one map / 20 maps, walk and windows: any partner,
// L = 4 43 / 68 and 54 / 107, L = 12 54 / 113 and 55 / 125, L = 16 62 / 133 and 55 / 122;
// nearest neighbours, L = 16 51 / 108 and 59 / 121, L = 28 67 / 158 and 74 / 148,
// L = 32 75 / 177 and 76 / 152.
constexpr int kWalkMaxL[2] = {12, 28};

__global__ void __launch_bounds__(kMapThreads) k_map_steps(MapArgs args)
{
    extern __shared__ uint32_t smem[];
    uint8_t *scr = args.scratch[blockIdx.x];
    const LatDesc d = *(const LatDesc *)(scr + kScrDesc);
    const int L = d.L;
    const uint32_t N = (uint32_t)L * (uint32_t)L;
    const uint32_t per = args.nn ? 20u : 10u;
    const uint32_t n_pairs = N / per < 1u ? 1u : N / per;
    const uint32_t G = (uint32_t)args.builders;             // maps built at once, one per wave
    const uint32_t magic = 0xFFFFFFFFu / (uint32_t)L + 1u;  // ceil(2^32 / L)
    const uint32_t bwords = (N + 31u) / 32u;
    uint32_t *thr = smem;                                   // kTabSize
    uint8_t *codes = (uint8_t *)(smem + kTabSize);          // N bytes
    uint32_t *bitmaps = smem + kTabSize + (N + 3u) / 4u;    // G x bwords
    uint32_t *pairs = bitmaps + G * bwords;                 // G x n_pairs

    const uint32_t *g_thr = (const uint32_t *)(scr + kScrFullTab);
    for (uint32_t i = threadIdx.x; i < (uint32_t)kTabSize; i += blockDim.x) thr[i] = g_thr[i];
    if (d.enc == 0) {
        const LAT_GLOBAL uint8_t *src = (const LAT_GLOBAL uint8_t *)d.state;
        for (uint32_t i = threadIdx.x; i < N; i += blockDim.x) codes[i] = src[i];
    } else {
        // 2-bit class layout: class 4*(y&1) + (x&3), (L/2) rows of L/64 words
        const LAT_GLOBAL uint32_t *src = (const LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = (uint32_t)L >> 6, csz = ((uint32_t)L >> 1) * W;
        for (uint32_t i = threadIdx.x; i < N; i += blockDim.x) {
            const uint32_t y = i / (uint32_t)L, x = i - y * (uint32_t)L;
            const uint32_t c = 4u * (y & 1u) + (x & 3u), X = x >> 2;
            codes[i] = (uint8_t)((src[c * csz + (y >> 1) * W + (X >> 4)] >> (2u * (X & 15u))) & 3u);
        }
    }
    __syncthreads();

    int tr[3] = {0, 0, 0};
    const uint64_t first = ((uint64_t)args.first_map_hi << 32) | args.first_map_lo;
    const uint32_t wave = threadIdx.x >> 6;
    uint32_t m0 = 0, left = args.n_maps;  // m0 + left is n_maps, so m0 never passes it
    for (uint32_t group = 0; left > 0; m0 += group, left -= group) {
        group = min(G, left);
        // maps depend only on the seed and their index: build `group` of them at once
        for (uint32_t i = threadIdx.x; i < group * bwords; i += blockDim.x) bitmaps[i] = 0u;
        __syncthreads();
        if (wave < group) {
            const uint64_t m = first + m0 + wave;
            uint32_t *bm = bitmaps + wave * bwords, *pr = pairs + wave * n_pairs;
            const uint32_t m_lo = (uint32_t)m, m_hi = (uint32_t)(m >> 32);
            if (args.nn) {
                if (L <= kWalkMaxL[1])
                    walk_map<true>(bm, pr, L, magic, N, n_pairs, m_lo, m_hi, d.key0, d.key1);
                else
                    build_map<true>(bm, pr, L, magic, N, n_pairs, m_lo, m_hi, d.key0, d.key1);
            } else {
                if (L <= kWalkMaxL[0])
                    walk_map<false>(bm, pr, L, magic, N, n_pairs, m_lo, m_hi, d.key0, d.key1);
                else
                    build_map<false>(bm, pr, L, magic, N, n_pairs, m_lo, m_hi, d.key0, d.key1);
            }
        }
        __syncthreads();
        // ...then apply them in map order
        for (uint32_t g = 0; g < group; ++g) {
            const uint64_t m = first + m0 + g;
            const uint32_t m_lo = (uint32_t)m, m_hi = (uint32_t)(m >> 32);
            const uint32_t *mp = pairs + g * n_pairs;
            // pairs 2c and 2c+1 share Philox call c
            for (uint32_t c = threadIdx.x; 2u * c < n_pairs; c += blockDim.x) {
                const u32x4 w = philox4x32_10(m_lo, kDomMapStep, c, m_hi, d.key0, d.key1);
                const uint32_t p0 = mp[2u * c];
                map_pair_step(codes, thr, L, magic, p0 & 0xFFFFu, p0 >> 16, w.x, w.y, tr);
                if (2u * c + 1u < n_pairs) {
                    const uint32_t p1 = mp[2u * c + 1u];
                    map_pair_step(codes, thr, L, magic, p1 & 0xFFFFu, p1 >> 16, w.z, w.w, tr);
                }
            }
            __syncthreads();
        }
    }

    if (d.enc == 0) {
        LAT_GLOBAL uint8_t *dst = (LAT_GLOBAL uint8_t *)d.state;
        for (uint32_t i = threadIdx.x; i < N; i += blockDim.x) dst[i] = codes[i];
    } else {
        LAT_GLOBAL uint32_t *dst = (LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = (uint32_t)L >> 6, H = (uint32_t)L >> 1, csz = H * W;
        for (uint32_t i = threadIdx.x; i < 8u * csz; i += blockDim.x) {
            const uint32_t c = i / csz, rem = i - c * csz, Y = rem / W, jw = rem - Y * W;
            const uint32_t y = 2u * Y + (c >> 2), x0 = c & 3u;
            uint32_t v = 0;
            for (uint32_t t = 0; t < 16u; ++t) v |= (uint32_t)codes[y * (uint32_t)L + 4u * (16u * jw + t) + x0] << (2u * t);
            dst[i] = v;
        }
    }
    block_reduce_add<3>(tr, (unsigned long long *)(scr + kScrTrackBase));
}

}  // namespace

hipError_t launch_map_steps(const MapArgs &a, int max_L, hipStream_t s)
{
    MapArgs b = a;
    b.builders = map_builders(max_L, a.n_maps);
    hipLaunchKernelGGL(k_map_steps, dim3((unsigned)b.count), dim3(kMapThreads), map_lds_bytes(max_L, b.builders), s,
                       b);
    return hipGetLastError();
}

hipError_t init_map_kernel_attributes()
{
    return hipFuncSetAttribute((const void *)k_map_steps, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kMapLdsMax);
}

}  // namespace lat
