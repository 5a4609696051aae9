// gfx950 on-chip kernel for lattices whose side is a multiple of 16
// (arXiv:2301.11735 section 3.1 update, section 3.2 parallel form and lattice
// copies): one block per lattice, the lattice resident in LDS for all the
// sweeps of a launch, four pairs a thread.
//
// LDS holds one byte per site, (1 + S) | (1 + sigma) << 4, by sublattice
// class: class c = 4 (y mod 2) + (x mod 4) is an (L/2) x (L/4) array of sites
// x = 4X + (x mod 4), y = 2Y + (y mod 2).  In phase p the updated a-sites are
// class (p, 0) and their partners class ((p + r) mod 4, 1), shifted by
// (dX, k) as a whole, so four consecutive sites of the a-class are one 32-bit
// word, their partners and all neighbours are 32-bit words of other classes
// (at any byte address), and three additions of neighbour words give both
// neighbour sums of all four sites, a nibble each (at most 8).  Two bits per
// site and 16 sites of a word at once spend most of a phase on taking the
// planes of the words apart, on exchanging sums between the lanes that share a
// word, and on masks; here a thread's four pairs share nothing with other lanes:
// the a-codes are one store, the partners' changes two XORs (a word of partners
// at an odd position is shared with the neighbouring task).
//
// Class rows have kQuadHalo bytes after their L/4 sites, the first four of which
// repeat the row's first four sites, so that four sites from any position of
// the row are contiguous; a change that touches them is repeated at the other
// place.  The words behind them are read with them, and hold nothing.  Words at
// odd positions are two words and a shift: an odd address takes the LDS several
// passes (256 lattices of L = 128, ten intervals of 50 sweeps: 4050 us with
// odd addresses, 2391 us with two words and a shift, 2240 us with the partners'
// changes as two XORs instead of a word store at an odd address).
//
// What bounds it: VALU issue (about 205 lane-ops per four pairs, 92 of them
// the two Philox calls) where the block fills its compute unit, and the chain of
// a phase (loads, two dependent table gathers, stores, block barrier) for
// small sides.  Launches with a record per interval, two bits per site (16
// sites of a word at once) and this form (us): 200 lattices of L = 96, 4 x 50
// sweeps, 2058 and 838; 256 of L = 128, 10 x 50, 3572 and 2172; 200 of L = 192,
// 4 x 20, 1377 and 855; 100 of L = 256, 4 x 20, 1420 and 1294.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "onchip.h"

namespace lat {
namespace {

// Row of the transition slots for the states (id_a, id_b): a site byte's id
// is its bits 5 or 1 and its bit 4: code 0 -> 2, 1 -> 0, 2 -> 3, 3 -> 1.
constexpr int quad_id(int code) { return code == 0 ? 2 : code == 1 ? 0 : code == 2 ? 3 : 1; }
constexpr TransSlots make_quad_slots()
{
    TransSlots t{};
    for (int st = 0; st < 16; ++st)
        for (int slot = 0; slot < 12; ++slot) {
            uint32_t coef = 0, C = 0;
            int a1 = 0, b1 = 0;
            trans_slot(st, slot, coef, C, a1, b1);
            const int row = quad_id(st & 3) << 2 | quad_id(st >> 2);
            const uint32_t at = 2u * (16u * (uint32_t)row + (uint32_t)slot);
            t.v[at] = coef;
            // the changes (XOR) of the two site bytes
            t.v[at + 1] = C | ((site_byte(a1) ^ site_byte(st & 3)) | (site_byte(b1) ^ site_byte(st >> 2)) << 8) << 16;
        }
    return t;
}
__device__ const TransSlots kQuadSlots = make_quad_slots();

struct QuadGeom {
    uint32_t L, Lq, H, P, rows, csz;  // rows: H rows of P bytes; csz: bytes of a class
};
__device__ __forceinline__ QuadGeom quad_geom(uint32_t L)
{
    const uint32_t P = (L >> 2) + kQuadHalo, rows = (L >> 1) * P;
    return QuadGeom{L, L >> 2, L >> 1, P, rows, rows};
}

// Four 2-bit codes in the low byte of v, one a byte, and back.
__device__ __forceinline__ uint32_t spread_codes(uint32_t v)
{
    uint32_t x = (v & 0xFFu) | (v & 0xFFu) << 12;
    x &= 0x000F000Fu;
    return (x | x << 6) & 0x03030303u;
}
__device__ __forceinline__ uint32_t gather_codes(uint32_t c)
{
    uint32_t x = (c | c >> 6) & 0x000F000Fu;
    return (x | x >> 12) & 0xFFu;
}

// Writes four sites of a class row (X0 a multiple of 4), and the halo.
__device__ __forceinline__ void put_quad(uint8_t *at, uint32_t X0, uint32_t Lq, uint32_t v)
{
    *(uint32_t *)at = v;
    if (X0 == 0) *(uint32_t *)(at + Lq) = v;
}

__device__ void stage_quads(uint8_t *lat, const LatDesc &d, const QuadGeom &g)
{
    const uint32_t q_row = g.Lq >> 2;  // quads of a class row
    if (d.enc == 0) {
        // 16 sites of a row: a 4 x 4 byte transpose gives a quad of each class
        const uint8_t *src = (const uint8_t *)d.state;
        for (uint32_t t = threadIdx.x; t < g.L * q_row; t += blockDim.x) {
            const uint32_t y = t / q_row, X0 = 4u * (t - y * q_row);
            const word_any *row = (const word_any *)(src + y * g.L + 4u * X0);
            uint32_t c[4];
            transpose4(site_from_codes(row[0]), site_from_codes(row[1]), site_from_codes(row[2]), site_from_codes(row[3]),
                       c[0], c[1], c[2], c[3]);
#pragma unroll
            for (uint32_t x = 0; x < 4u; ++x) put_quad(lat + (4u * (y & 1u) + x) * g.csz + (y >> 1) * g.P + X0, X0, g.Lq, c[x]);
        }
    } else {
        const LAT_GLOBAL uint32_t *src = (const LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = g.L >> 6;
        for (uint32_t t = threadIdx.x; t < 8u * g.H * W; t += blockDim.x) {
            const uint32_t row = t / W, j = t - row * W, c = row / g.H, Y = row - c * g.H, w = src[t];
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) {
                const uint32_t X0 = 16u * j + 4u * k;
                put_quad(lat + c * g.csz + Y * g.P + X0, X0, g.Lq, site_from_codes(spread_codes(w >> (8u * k))));
            }
        }
    }
}

__device__ void unstage_quads(const uint8_t *lat, const LatDesc &d, const QuadGeom &g)
{
    const uint32_t q_row = g.Lq >> 2;
    if (d.enc == 0) {
        uint8_t *dst = (uint8_t *)d.state;
        for (uint32_t t = threadIdx.x; t < g.L * q_row; t += blockDim.x) {
            const uint32_t y = t / q_row, X0 = 4u * (t - y * q_row);
            uint32_t c[4], w[4];
#pragma unroll
            for (uint32_t x = 0; x < 4u; ++x)
                c[x] = codes_from_site(*(const uint32_t *)(lat + (4u * (y & 1u) + x) * g.csz + (y >> 1) * g.P + X0));
            transpose4(c[0], c[1], c[2], c[3], w[0], w[1], w[2], w[3]);
            word_any *row = (word_any *)(dst + y * g.L + 4u * X0);
#pragma unroll
            for (int k = 0; k < 4; ++k) row[k] = w[k];
        }
    } else {
        LAT_GLOBAL uint32_t *dst = (LAT_GLOBAL uint32_t *)d.state;
        const uint32_t W = g.L >> 6;
        for (uint32_t t = threadIdx.x; t < 8u * g.H * W; t += blockDim.x) {
            const uint32_t row = t / W, j = t - row * W, c = row / g.H, Y = row - c * g.H;
            uint32_t w = 0;
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k)
                w |= gather_codes(codes_from_site(*(const uint32_t *)(lat + c * g.csz + Y * g.P + 16u * j + 4u * k))) << (8u * k);
            dst[t] = w;
        }
    }
}

// A task: four pairs of a class row.  Byte offsets within a class.
struct QuadPos {
    uint32_t X0, row, a, up, left;  // left: the a-sites' left neighbours in phase 0 (class 3)
};
__device__ __forceinline__ QuadPos quad_pos(uint32_t task, const QuadGeom &g, uint32_t magic)
{
    const uint32_t q_row = g.Lq >> 2, Y = q_row == 1u ? task : __umulhi(task, magic);
    QuadPos s;
    s.X0 = 4u * (task - Y * q_row);
    s.row = Y * g.P;
    s.a = s.row + s.X0;
    s.up = (Y == 0 ? g.rows : s.row) - g.P + s.X0;
    s.left = s.X0 == 0 ? s.row + g.Lq - 1u : s.a - 1u;
    return s;
}

// The phase's shift (dX, k rows) and the class of the partners (uniform).
struct QuadPhase {
    uint32_t dX, kP, pb;
};

struct QuadDraws {
    u32x4 c[2];
};
__device__ __forceinline__ QuadDraws quad_draws(uint64_t s, uint32_t p, uint32_t task, uint32_t key0, uint32_t key1)
{
    QuadDraws d;
#pragma unroll
    for (uint32_t i = 0; i < 2u; ++i)
        d.c[i] = pair_draws(philox4x32_10((uint32_t)s, p, 2u * task + i, (uint32_t)(s >> 32), key0, key1));
    return d;
}

// Four sites from byte i on: the two words that hold them, shifted into place
// (a word read at an odd address takes several passes of the LDS).
__device__ __forceinline__ uint32_t quad_at(const uint8_t *lat, uint32_t i)
{
    const uint32_t *w = (const uint32_t *)(lat + (i & ~3u));
    return __builtin_amdgcn_alignbit(w[1], w[0], 8u * (i & 3u));
}

// The four coupled-pair steps of a task in phase P.
template <int P>
__device__ __forceinline__ void quad_step(uint8_t *lat, const QuadGeom &g, const QuadPos &s, const QuadPhase &f,
                                          const QuadDraws &d, const uint2 *s_tab, const uint8_t *s_slots,
                                          uint32_t &packed)
{
    // partners: positions Xb .. Xb + 3 of the row kP below; x mod n for x < 2n is min(x, x - n)
    uint32_t Xb = s.X0 + f.dX;
    Xb = min(Xb, Xb - g.Lq);
    uint32_t rb = s.row + f.kP;
    rb = min(rb, rb - g.rows);
    uint32_t rd = rb + g.P;
    rd = min(rd, rd - g.rows);
    uint32_t Xl = Xb - (f.pb == 0u ? 1u : 0u);  // left neighbours' position; the right ones' needs no wrap
    Xl = min(Xl, Xl + g.Lq);
    const uint32_t cBL = (f.pb == 0u ? 7u : 3u + f.pb) * g.csz, cBR = f.pb == 3u ? 4u * g.csz + 1u : (5u + f.pb) * g.csz;
    const uint32_t b = rb + Xb + (4u + f.pb) * g.csz;
    uint8_t *pa = lat + P * g.csz + s.a;

    const uint32_t A = *(const uint32_t *)pa, B = quad_at(lat, b);
    const uint32_t sa = (P > 0 ? *(const uint32_t *)(pa - (P > 0 ? g.csz : 0u)) : quad_at(lat, 3u * g.csz + s.left)) +
                        (P < 3 ? *(const uint32_t *)(pa + (P < 3 ? g.csz : 0u)) : quad_at(lat, s.a + 1u)) +
                        *(const uint32_t *)(lat + (4 + P) * g.csz + s.up) + *(const uint32_t *)(pa + 4u * g.csz);
    const uint32_t sb = quad_at(lat, rb + Xl + cBL) + quad_at(lat, rb + Xb + cBR) + quad_at(lat, rb + Xb + f.pb * g.csz) +
                        quad_at(lat, rd + Xb + f.pb * g.csz);
    // (sum S_a + 4, sum S_b + 4, sum sigma_a + 4, sum sigma_b + 4) of each pair
    uint32_t n[4];
    transpose4(sa & kM0F, sb & kM0F, (sa >> 4) & kM0F, (sb >> 4) & kM0F, n[0], n[1], n[2], n[3]);
    // ids of both sites of each pair, at bits 5:4 and 3:2 of its byte
    const uint32_t id = ((A & 0x30303030u) | ((A << 4) & 0x20202020u)) |
                        (((B >> 2) & 0x0C0C0C0Cu) | ((B << 2) & 0x08080808u));
    uint32_t ch[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const u32x4 &w = d.c[i >> 1];
        const uint32_t row = i == 0 ? id << 5 : id >> (i == 0 ? 0 : 8 * i - 5);
        const uint2 tr2 = *(const uint2 *)(s_slots + ((row & 0x780u) | ((i & 1) ? w.z : w.x)));
        const uint32_t idx = (uint32_t)__builtin_amdgcn_sdot4((int)tr2.x, (int)n[i], (int)tr2.y, false);
        const uint2 e = *(const uint2 *)((const uint8_t *)s_tab + (uint32_t)(uint16_t)(idx << 3));
        const bool acc = ((i & 1) ? w.w : w.y) < e.x;
        packed += acc ? e.y : 0u;
        ch[i] = acc ? tr2.y : 0u;
    }
    const uint32_t An = A ^ __builtin_amdgcn_perm(__builtin_amdgcn_perm(ch[3], ch[2], 0x0C0C0602u),
                                                  __builtin_amdgcn_perm(ch[1], ch[0], 0x0C0C0602u), 0x05040100u);
    const uint32_t dB = __builtin_amdgcn_perm(__builtin_amdgcn_perm(ch[3], ch[2], 0x0C0C0703u),
                                                  __builtin_amdgcn_perm(ch[1], ch[0], 0x0C0C0703u), 0x05040100u);
    *(uint32_t *)pa = An;
    if (s.X0 == 0) *(uint32_t *)(pa + g.Lq) = An;
    const uint32_t sh = 8u * (f.dX & 3u);
    const uint32_t lo = dB << sh, hi = sh ? dB >> (32u - sh) : 0u;
    uint32_t *pb = (uint32_t *)(lat + (b & ~3u));
    atomicXor(pb, lo);
    atomicXor(pb + 1, hi);
    if (Xb < 4u) atomicXor((uint32_t *)((uint8_t *)pb + g.Lq), lo);
    if (Xb + 3u >= g.Lq) atomicXor((uint32_t *)((uint8_t *)(pb + 1) - g.Lq), hi);
}

// `intervals` times `every` sweeps of the lattice in LDS from sweep first on,
// each interval followed by observe(k).  One: every thread has at most one
// task, whose draws of the next phase are made while the current phase's loads
// are in flight.
template <bool One, typename F>
__device__ __forceinline__ void quad_sweeps(uint8_t *lat, uint32_t *sched, const LatDesc &d, const QuadGeom &g,
                                            uint32_t intervals, uint32_t every, const uint2 *s_tab,
                                            const uint8_t *s_slots, int (&tr)[3], F observe)
{
    const uint32_t q_row = g.Lq >> 2, magic = q_row == 1u ? 0u : 0xFFFFFFFFu / q_row + 1u;
    const uint32_t tasks = g.H * q_row, n = intervals * every;
    const uint64_t first = d.next_sweep;
    const bool mine = threadIdx.x < tasks;
    make_schedules(sched, first, n, d.key0, d.key1, g.L);
    __syncthreads();
    QuadPos pos{};
    QuadDraws dr{};
    if (One) {
        pos = quad_pos(mine ? threadIdx.x : 0u, g, magic);
        dr = quad_draws(first, 0u, threadIdx.x, d.key0, d.key1);
    }
    SweepLoads coming = sweep_loads(sched);  // of the next sweep's schedule
    uint32_t left = every, k = 0;  // sweeps left of interval k
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t s = first + i;
        uint32_t packed = 0u;  // One: at most 16 accepted moves a sweep
        const SweepWords w = sweep_words(coming);
        auto phase = [&](auto pc) {
            constexpr int P = decltype(pc)::value;
            const uint32_t j = i + 1u;
            if (P == 0 && j % kSchedSweeps == 0 && j < n)
                make_schedules(sched + 12u * (j % (2u * kSchedSweeps)), s + 1, n - j, d.key0, d.key1, g.L);
            if (P == 3) coming = sweep_loads(sched + 12u * (j % (2u * kSchedSweeps)));
            QuadPhase f;
            f.pb = (P + w.r) & 3u;
            f.dX = w.m[P] + ((P + w.r) >> 2);
            if (f.dX >= g.Lq) f.dX -= g.Lq;
            f.kP = w.k[P] * g.P;
            if (One) {
                if (mine) {
                    const QuadDraws next = quad_draws(P < 3 ? s : s + 1, (P + 1) & 3, threadIdx.x, d.key0, d.key1);
                    quad_step<P>(lat, g, pos, f, dr, s_tab, s_slots, packed);
                    dr = next;
                }
            } else {
                for (uint32_t t = threadIdx.x; t < tasks; t += blockDim.x) {
                    packed = 0u;
                    quad_step<P>(lat, g, quad_pos(t, g, magic), f, quad_draws(s, P, t, d.key0, d.key1), s_tab, s_slots, packed);
                    unpack_tracker(packed, tr);
                }
            }
            __syncthreads();
        };
        phase(std::integral_constant<int, 0>{});
        phase(std::integral_constant<int, 1>{});
        phase(std::integral_constant<int, 2>{});
        phase(std::integral_constant<int, 3>{});
        if (One) unpack_tracker(packed, tr);
        if (--left == 0) {
            observe(k);
            ++k;
            left = every;
        }
    }
}

// This thread's share of the seven observable sums, four sites at a time.
__device__ __forceinline__ void quad_observables(const uint8_t *lat, const QuadGeom &g, int (&v)[7])
{
    const uint32_t q_row = g.Lq >> 2, n = 8u * g.H * q_row;
    SiteSums sums;
    for (uint32_t t = threadIdx.x; t < n; t += blockDim.x) {
        const uint32_t row = t / q_row, X0 = 4u * (t - row * q_row), c = row / g.H, Y = row - c * g.H;
        const uint32_t cx = c & 3u, cy = c >> 2, at = Y * g.P + X0;
        const uint32_t w = *(const uint32_t *)(lat + c * g.csz + at);
        const uint32_t wr = cx < 3u ? *(const uint32_t *)(lat + (c + 1u) * g.csz + at) : quad_at(lat, (c - 3u) * g.csz + at + 1u);
        const uint32_t wd = cy == 0 ? *(const uint32_t *)(lat + (c + 4u) * g.csz + at)
                                    : *(const uint32_t *)(lat + cx * g.csz + (Y + 1u == g.H ? X0 : at + g.P));
        sums.add(w, wr, wd, ((cx + cy) & 1u) ? -1 : 0x01010101);
    }
    sums.get(v);
}

__global__ void __launch_bounds__(1024) k_sweep_quad(BatchArgs args)
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
        const uint2 *g_tab = (const uint2 *)(scr + kScrDevTab), *g_slots = (const uint2 *)kQuadSlots.v;
        for (int i = threadIdx.x; i < kDevTabEntries; i += blockDim.x) s_tab[i] = g_tab[i];
        for (int i = threadIdx.x; i < kSlotEntries; i += blockDim.x) s_slots[i] = g_slots[i];
    }
    const QuadGeom g = quad_geom((uint32_t)d.L);
    stage_quads(lat, d, g);
    if (args.obs_out) tracker_before(scr, obs);
    __syncthreads();

    const uint32_t my_sweeps = args.sweeps[blockIdx.x], intervals = args.obs_out ? args.intervals : 1u;
    const uint8_t *slots = (const uint8_t *)s_slots;
    int tr[3] = {0, 0, 0};
    auto observe = [&](uint32_t k) {
        if (!args.obs_out) return;
        int o[7];
        quad_observables(lat, g, o);
        write_record(args, obs, tr, o, k, d.next_sweep + (uint64_t)my_sweeps * (k + 1u));
    };
    if (my_sweeps > 0) {
        if (g.H * (g.Lq >> 2) <= blockDim.x)
            quad_sweeps<true>(lat, sched, d, g, intervals, my_sweeps, s_tab, slots, tr, observe);
        else
            quad_sweeps<false>(lat, sched, d, g, intervals, my_sweeps, s_tab, slots, tr, observe);
    }
    unstage_quads(lat, d, g);
    if (threadIdx.x == 0) ((LatDesc *)(scr + kScrDesc))->next_sweep = d.next_sweep + (uint64_t)my_sweeps * intervals;
    block_reduce_add<3>(tr, (unsigned long long *)(scr + kScrTrackBase));
}

}  // namespace

hipError_t init_quad_kernel_attributes()
{
    return hipFuncSetAttribute((const void *)k_sweep_quad, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)quad_lds_bytes(kQuadMaxL));
}

hipError_t launch_sweep_quad(const BatchArgs &a, int max_L, int threads, hipStream_t s)
{
    // one thread per task (four pairs) up to 1024: where they take several
    // passes, equally many threads in fewer waves measured slower (L = 192:
    // 11.8 us a sweep with two passes of 576, 9.7 with 1024 and 128)
    const uint32_t tasks = (uint32_t)max_L * (uint32_t)max_L / 32u;
    uint32_t block = std::min(1024u, (tasks + 63u) / 64u * 64u);
    if (threads > 0) block = (uint32_t)std::min(1024, std::max(64, threads / 64 * 64));
    hipLaunchKernelGGL(k_sweep_quad, dim3((unsigned)a.count), dim3(block), quad_lds_bytes(max_L), s, a);
    return hipGetLastError();
}

}  // namespace lat
