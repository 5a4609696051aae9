// gfx950 kernel of the penalty mode (arXiv:2301.11735 section 2.2): the prior
// method the paper replaces, kept to show its defect.  The energy gets
// -mu sum S, sites are updated one at a time by the Metropolis rule on a
// checkerboard (sites of one colour never neighbour each other), and the
// host adjusts mu between sweeps.  Int8 states.
//
// Four sites in a row (one 32-bit word of codes) hold two sites of a colour,
// at bytes o and o + 2 with o = (y + c) & 1, and these are the two sites of
// Philox call y L/4 + X.  As bytes (1 + S) | (1 + sigma) << 4 the four
// neighbour words add up to both sums of all four sites (at most 8 a
// nibble), and the sum byte indexes the table directly.  NW = 4: a thread takes
// 16 sites with 16-byte loads, where L is a multiple of 16 and the state is
// aligned to it; NW = 1 serves every other side and address.
//
// What bounds it: the draws (about 46 of 90 lane-ops a call) and, at L = 4096,
// the 33 MB that a half-sweep reads and writes.  A half-sweep at L = 4096 takes
// 17 us (byte gathers, one neighbour at a time: 41 us); a sweep with its mu
// step 51 us of wall time (158 us with the whole table of 4335 thresholds
// rebuilt and all observables reduced for the charge).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_common.h"

namespace lat {
namespace {

constexpr uint32_t kDomMu = 0x600u;

// Packed changes of a move, summed over a thread's (at most 8) accepted moves
// of one group: count << 27 | (nD + 1) << 22 | (nV + 8) << 14 | (nJ + 8) << 6 |
// (dS + 2).
struct MuMoves {
    uint32_t v[kMuTabSize];
};
constexpr MuMoves make_mu_moves()
{
    constexpr int S[4] = {0, 0, 1, -1}, G[4] = {1, -1, 0, 0};
    MuMoves t{};
    for (int c = 0; c < 16; ++c)
        for (int s = -4; s <= 4; ++s)
            for (int g = -4; g <= 4; ++g) {
                const int c0 = c >> 2, c1 = c & 3, dS = S[c1] - S[c0];
                if ((s < 0 ? -s : s) + (g < 0 ? -g : g) > 4) continue;
                t.v[mu_index(c0, c1, s, g)] = 1u << 27 | (uint32_t)(S[c1] * S[c1] - S[c0] * S[c0] + 1) << 22 |
                                              (uint32_t)(dS * s + 8) << 14 | (uint32_t)((G[c1] - G[c0]) * g + 8) << 6 |
                                              (uint32_t)(dS + 2);
            }
    return t;
}
__device__ const MuMoves kMuMoves = make_mu_moves();

template <int NW>
__global__ void __launch_bounds__(1024) k_mu_half(MuArgs a)
{
    __shared__ uint2 s_tab[kMuTabSize];
    for (int i = threadIdx.x; i < kMuTabSize; i += blockDim.x) s_tab[i] = make_uint2(a.tab[i], kMuMoves.v[i]);
    __syncthreads();
    const uint32_t L = (uint32_t)a.L, Lq = L >> 2, per_row = Lq / NW, n = L * per_row;
    uint8_t *st = (uint8_t *)a.state;
    int tr[4] = {0, 0, 0, 0};
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        const uint32_t y = t / per_row, X = (t - y * per_row) * NW;
        const size_t row = (size_t)y * L, at = row + 4u * X;
        const size_t up = (y == 0 ? (size_t)(L - 1) * L : row - L) + 4u * X;
        const size_t dn = (y + 1 == L ? 0 : row + L) + 4u * X;
        const uint32_t o = (y + (uint32_t)a.colour) & 1u;
        // the neighbour word beside the group that byte 0 (o = 0) or its last byte (o = 1) needs
        const uint32_t Xs = o ? (X + NW == Lq ? 0u : X + NW) : (X == 0 ? Lq - 1u : X - 1u);
        uint32_t c[NW], u[NW], d[NW], e[NW];
        load_codes<NW>(st + at, c);
        load_codes<NW>(st + up, u);
        load_codes<NW>(st + dn, d);
        const uint32_t side = site_from_codes(*(const word_any *)(st + row + 4u * Xs));
#pragma unroll
        for (int i = 0; i < NW; ++i) e[i] = site_from_codes(c[i]);
        uint32_t packed = 0u, out[NW];
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const u32x4 w = philox4x32_10(a.s_lo, kDomMu + (uint32_t)a.colour, y * Lq + X + (uint32_t)i, a.s_hi, a.key0,
                                          a.key1);
            const uint32_t left = __builtin_amdgcn_alignbit(e[i], i > 0 ? e[i > 0 ? i - 1 : 0] : side, 24u);
            const uint32_t right = __builtin_amdgcn_alignbit(i < NW - 1 ? e[i < NW - 1 ? i + 1 : 0] : side, e[i], 8u);
            const uint32_t sum = (left + right + site_from_codes(u[i]) + site_from_codes(d[i])) >> (8u * o);
            const uint32_t code = c[i] >> (8u * o);
            uint32_t flip = 0u;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t c0 = (code >> (16 * h)) & 3u, c1 = (h ? w.z : w.x) >> 30;
                const uint2 q = s_tab[mu_index(c0, c1) + ((sum >> (16 * h)) & 0xFFu)];
                const bool acc = min(h ? w.w : w.y, 0xFFFFFFFEu) < q.x;
                packed += acc ? q.y : 0u;
                flip |= acc ? (c0 ^ c1) << (16 * h) : 0u;
            }
            out[i] = c[i] ^ (flip << (8u * o));
        }
        if constexpr (NW == 4)
            *(uint4 *)(st + at) = make_uint4(out[0], out[1], out[2], out[3]);
        else
            *(word_any *)(st + at) = out[0];
        const int cnt = (int)(packed >> 27);
        tr[0] += (int)((packed >> 22) & 31u) - cnt;
        tr[1] += (int)((packed >> 14) & 255u) - 8 * cnt;
        tr[2] += (int)((packed >> 6) & 255u) - 8 * cnt;
        tr[3] += (int)(packed & 63u) - 2 * cnt;
    }
    __shared__ int part[16][4];
    wave_partials<4, int>(tr, part);
    __syncthreads();
    if (threadIdx.x < 4) {
        long long s = 0;
        for (uint32_t w = 0; w < blockDim.x >> 6; ++w) s += (long long)part[w][threadIdx.x];
        unsigned long long *dst = threadIdx.x < 3 ? a.track + 3 * (size_t)blockIdx.x + threadIdx.x
                                                  : a.charge + kMuChargeStride * (blockIdx.x % kMuChargeSlots);
        if (s != 0) atomicAdd(dst, (unsigned long long)s);
    }
}

}  // namespace

hipError_t launch_mu_half(const MuArgs &a, hipStream_t s)
{
    const bool wide = a.L % 16 == 0 && ((uintptr_t)a.state & 15u) == 0;
    const uint32_t groups = (uint32_t)a.L * (uint32_t)a.L / (wide ? 16u : 4u);
    // At most kMaxSlots blocks (each has a tracker slot): the smallest blocks
    // that take every group in one pass, since a block's waves hide the loads
    // better than a second pass does (L = 4096: 21.5 us a half-sweep with four
    // passes of 256 threads, 17 us with one of 1024), and small lattices
    // spread over more compute units.
    uint32_t threads = 256;
    while (threads < 1024u && groups > threads * (uint32_t)kMaxSlots) threads *= 2;
    const uint32_t grid = std::min((groups + threads - 1u) / threads, (uint32_t)kMaxSlots);
    if (wide)
        hipLaunchKernelGGL(k_mu_half<4>, dim3(grid), dim3(threads), 0, s, a);
    else
        hipLaunchKernelGGL(k_mu_half<1>, dim3(grid), dim3(threads), 0, s, a);
    return hipGetLastError();
}

}  // namespace lat
