// Host side of the penalty mode (section 2.2, the prior method): per sweep,
// the thresholds at the current mu, two checkerboard half-sweeps, the change of
// the charge read back, and the controller step mu += kappa (Q - sum S) / N, all
// in the same FP64 expressions the method's definition gives.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <cstring>
#include <memory>

#include "../../include/lattice.h"
#include "internal.h"
#include "kernels.h"

using namespace lat;
using namespace lat::detail;

namespace {

// Thresholds of the moves that occur at this mu: 12 moves (a site's own code
// again is always accepted) at 41 pairs of neighbour sums.
void build_mu_table(double Delta, double V, double J, double T, double mu, uint32_t *tab)
{
    static const int S[4] = {0, 0, 1, -1}, G[4] = {1, -1, 0, 0};
    for (int c0 = 0; c0 < 4; ++c0)
        for (int c1 = 0; c1 < 4; ++c1) {
            const int dS = S[c1] - S[c0], dG = G[c1] - G[c0], nD = S[c1] * S[c1] - S[c0] * S[c0];
            for (int s = -4; s <= 4; ++s)
                for (int g = std::abs(s) - 4; g <= 4 - std::abs(s); ++g) {
                    const int nV = dS * s, nJ = dG * g;
                    const double dE = Delta * nD + V * nV + 0.25 * J * nJ - mu * dS;
                    uint32_t t;
                    if (dE <= 0.0) {
                        t = 0xFFFFFFFFu;
                    } else {
                        const double f = std::floor(std::exp(-dE / T) * 4294967296.0);
                        t = f >= 4294967294.0 ? 0xFFFFFFFEu : (uint32_t)f;
                    }
                    tab[mu_index(c0, c1, s, g)] = t;
                }
        }
}

// Host side of a call's copies.
struct MuStage {
    uint32_t tab[kMuTabSize];
    int64_t charge[kMuChargeSlots * kMuChargeStride];
    int64_t sum_S;  // before the call's first sweep
    uint32_t err;   // the lattice's error flags
};
static_assert(sizeof(MuStage) <= kPinnedBytes, "a pinned block holds a call's copies");
static_assert(kScrObsSlots + sizeof(MuStage::charge) <= kScrSlots, "the charge sums fit the observable slots");

}  // namespace

extern "C" {

int lattice_mu_sweeps(lattice *h, uint64_t first_sweep, uint32_t n_sweeps, double kappa, double *mu,
                      double *mu_series, int64_t *sumS_series)
{
    return guarded("lattice_mu_sweeps", [&]() -> int {
        if (!live(h)) return fail(LAT_ESTATE, "null or destroyed handle");
        if (!mu || !std::isfinite(*mu) || !std::isfinite(kappa)) return fail(LAT_EINVAL, "mu and kappa must be finite");
        if (h->enc != LAT_ENC_INT8) return fail(LAT_EINVAL, "the penalty mode takes int8 lattices");
        if (n_sweeps == 0) return LAT_OK;
        PinnedBlock pinned;
        std::unique_ptr<MuStage> own;
        if (!pinned.p) own = std::make_unique<MuStage>();
        MuStage &st = pinned.p ? *(MuStage *)pinned.p : *own;
        std::memset(st.tab, 0, sizeof(st.tab));
        st.err = 0;
        MuArgs a{};
        a.state = (int8_t *)h->d_state;
        a.tab = (const uint32_t *)(h->d_scratch + kScrMuTab);
        a.track = (unsigned long long *)(h->d_scratch + kScrSlots);
        a.charge = (unsigned long long *)(h->d_scratch + kScrObsSlots);
        a.L = h->L;
        a.key0 = (uint32_t)h->seed;
        a.key1 = (uint32_t)(h->seed >> 32);
        // the charge before the call, by one reduction; then the sweeps count its changes
        hipError_t e = launch_observables(h->d_scratch, h->d_state, h->L, h->enc, h->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(&st.sum_S, h->d_scratch + kScrObs, sizeof(st.sum_S), hipMemcpyDeviceToHost, h->stream);
        if (e == hipSuccess && barrier_may_time_out(h))
            e = hipMemcpyAsync(&st.err, h->d_scratch + kScrErr, sizeof(st.err), hipMemcpyDeviceToHost, h->stream);
        if (e == hipSuccess) e = launch_zero_i64(a.charge, kMuChargeSlots * kMuChargeStride, h->stream);
        for (uint32_t i = 0; i < n_sweeps; ++i) {
            const uint64_t s = first_sweep + i;
            build_mu_table(h->Delta, h->V, h->J, h->T, *mu, st.tab);
            if (e == hipSuccess)
                e = hipMemcpyAsync(h->d_scratch + kScrMuTab, st.tab, sizeof(st.tab), hipMemcpyHostToDevice, h->stream);
            a.s_lo = (uint32_t)s;
            a.s_hi = (uint32_t)(s >> 32);
            for (int c = 0; c < 2 && e == hipSuccess; ++c) {
                a.colour = c;
                e = launch_mu_half(a, h->stream);
            }
            if (e == hipSuccess)
                e = hipMemcpyAsync(st.charge, a.charge, sizeof(st.charge), hipMemcpyDeviceToHost, h->stream);
            const hipError_t waited = hipStreamSynchronize(h->stream);  // the next table is written after its copy
            if (waited != hipSuccess) pinned.abandon();
            if (e == hipSuccess) e = waited;
            if (e != hipSuccess) return hip_fail(e, "lattice_mu_sweeps");
            if (st.err & 1u) return barrier_timed_out();
            int64_t sumS = st.sum_S;
            for (int k = 0; k < kMuChargeSlots; ++k) sumS += st.charge[k * kMuChargeStride];
            if (mu_series) mu_series[i] = *mu;
            if (sumS_series) sumS_series[i] = sumS;
            *mu = *mu + kappa * (double)(h->Q - sumS) / (double)h->N;
        }
        return LAT_OK;
    });
}

}  // extern "C"
