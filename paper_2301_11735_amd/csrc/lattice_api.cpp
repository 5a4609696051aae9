// Host side of liblattice.so: the C-ABI of include/lattice.h.
//
// Parameter checks and the charge target (eq. 2), the stage-1 initial
// configuration (section 3.1), the FP64 Metropolis threshold table (section
// 3.1, eq. 3), the per-sweep schedule of non-interacting pairs (section 3.2)
// and the layout conversion between canonical codes and the device encodings.
// All sweep and reduction work runs in the kernels of phase.hip, obs.hip and
// batch.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <memory>
#include <tuple>
#include <type_traits>
#include <mutex>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <string>
#include <thread>
#include <vector>

#include "../../include/lattice.h"
#include "internal.h"
#include "kernels.h"
#include "philox.h"

using namespace lat;
using namespace lat::detail;

namespace {

constexpr uint32_t kMagic = 0x1A771CEu;
constexpr int kMaxL = 32768;

thread_local std::string g_err;
thread_local const char *g_err_fixed = nullptr;  // set when g_err could not be formatted

}  // namespace

namespace lat {
namespace detail {

int fail(int code, const std::string &msg)
{
    g_err_fixed = nullptr;
    g_err = msg;
    return code;
}

int fail_nothrow(int code, const char *what, const char *msg) noexcept
{
    try {
        g_err_fixed = nullptr;
        g_err = std::string(what) + ": " + msg;
    } catch (...) {
        g_err_fixed = code == LAT_ENOMEM ? "out of host memory" : "error (its message could not be stored)";
    }
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(LAT_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

int barrier_timed_out() { return fail(LAT_EHIP, "a device-wide phase barrier timed out; the state is invalid"); }

bool live(const lattice *h) { return h != nullptr && h->magic == kMagic; }

namespace {
// (no destructor: threads that outlive main may still be in a call)
struct PinnedPool {
    size_t bytes, keep;
    size_t n = 0;
    void *free[kPinnedKeep] = {};
};
static_assert(std::is_trivially_destructible_v<PinnedPool> && kPinnedLargeKeep <= kPinnedKeep);
std::mutex g_pinned_mu;
PinnedPool g_pinned[2] = {{kPinnedBytes, kPinnedKeep}, {kPinnedLarge, kPinnedLargeKeep}};
}  // namespace

PinnedBlock::PinnedBlock(bool large) : large_(large)
{
    PinnedPool &pool = g_pinned[large_];
    {
        std::lock_guard<std::mutex> lock(g_pinned_mu);
        if (pool.n > 0) p = pool.free[--pool.n];
    }
    // portable: usable with every device of the process
    if (!p && hipHostMalloc(&p, pool.bytes, hipHostMallocPortable) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
    }
}

PinnedBlock::~PinnedBlock()
{
    if (!p) return;
    PinnedPool &pool = g_pinned[large_];
    {
        std::lock_guard<std::mutex> lock(g_pinned_mu);
        if (pool.n < pool.keep) {
            pool.free[pool.n++] = p;
            return;
        }
    }
    (void)hipHostFree(p);
}

}  // namespace detail
}  // namespace lat

namespace {

bool valid_geometry(int32_t L, int32_t enc)
{
    if (L < 4 || L > kMaxL) return false;
    if (enc == LAT_ENC_INT8) return L % 4 == 0;
    if (enc == LAT_ENC_2BIT) return L % 64 == 0;
    return false;
}

// Eq. (2) made an integer: Q nearest nN with the parity of the charged count
// (ties to the smaller); without a requested count, Nc = max(N/4, |Q|).
int charge_target(int32_t L, double n, int64_t n_req, int64_t *Q_out, int64_t *Nc_out)
{
    const int64_t N = (int64_t)L * L;
    const double target = n * (double)N;
    if (!std::isfinite(target) || std::fabs(target) > (double)N) return fail(LAT_EINVAL, "n must satisfy |n| <= 1");
    const int64_t nc0 = n_req >= 0 ? n_req : N / 4;
    if (nc0 > N) return fail(LAT_EINVAL, "n_charged exceeds N");
    const int64_t parity = nc0 & 1;
    int64_t lo = (int64_t)std::floor(target);
    if ((lo & 1) != parity) lo -= 1;  // two's complement: & 1 is the parity for negatives too
    const int64_t hi = lo + 2;
    const int64_t Q = ((double)hi - target < target - (double)lo) ? hi : lo;
    int64_t Nc = nc0;
    if (std::llabs(Q) > nc0) {
        if (n_req >= 0) return fail(LAT_EINVAL, "|Q| exceeds the requested number of charged sites");
        Nc = std::llabs(Q);
    }
    if (Nc > N) return fail(LAT_EINVAL, "no charge target fits the lattice");
    *Q_out = Q;
    *Nc_out = Nc;
    return LAT_OK;
}

// Stage 1 of section 3.1 where the device cannot decide it (seed.hip): site i gets key (w0 << 32 | w1) of Philox counter
// (0, 0x200, i, 0); the N+ smallest (key, i) become +1, the next N- become -1,
// the others are spins with sigma from bit 0 of w2.  Selection (two
// nth_element passes) gives the same sets as a full sort.
void seeded_init(int32_t L, uint64_t seed, int64_t n_plus, int64_t n_minus, std::vector<int8_t> &codes)
{
    const int64_t N = (int64_t)L * L;
    struct Key {
        uint64_t k;
        uint32_t i;
        bool operator<(const Key &o) const { return k != o.k ? k < o.k : i < o.i; }
    };
    std::vector<Key> keys((size_t)N);
    codes.assign((size_t)N, 0);
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    unsigned nt = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    if (N < (1 << 16)) nt = 1;
    std::vector<std::thread> pool;
    for (unsigned t = 0; t < nt; ++t) {
        pool.emplace_back([&, t] {
            const int64_t b = N * t / nt, e = N * (t + 1) / nt;
            for (int64_t i = b; i < e; ++i) {
                const u32x4 w = philox4x32_10(0u, kDomInit, (uint32_t)i, 0u, k0, k1);
                keys[(size_t)i] = Key{((uint64_t)w.x << 32) | w.y, (uint32_t)i};
                codes[(size_t)i] = (int8_t)(w.z & 1u);
            }
        });
    }
    for (auto &th : pool) th.join();
    const int64_t nc = n_plus + n_minus;
    if (nc > 0) {
        if (nc < N) std::nth_element(keys.begin(), keys.begin() + nc, keys.end());
        if (n_plus > 0 && n_plus < nc) std::nth_element(keys.begin(), keys.begin() + n_plus, keys.begin() + nc);
        for (int64_t r = 0; r < nc; ++r) codes[keys[(size_t)r].i] = (int8_t)(r < n_plus ? 2 : 3);
    }
}

// Section 3.1: classical Metropolis acceptance for every energy-change triple,
// dE = Delta*nD + V*nV + 0.25*J*nJ (eq. 3) in FP64; "always" for dE <= 0.
void build_threshold_table(double Delta, double V, double J, double T, std::vector<uint32_t> &tab)
{
    tab.assign(kTabSize, 0u);
    for (int nD = -2; nD <= 2; ++nD)
        for (int nV = -16; nV <= 16; ++nV)
            for (int nJ = -16; nJ <= 16; ++nJ) {
                const double dE = Delta * nD + V * nV + 0.25 * J * nJ;
                uint32_t t;
                if (dE <= 0.0) {
                    t = 0xFFFFFFFFu;
                } else {
                    const double f = std::floor(std::exp(-dE / T) * 4294967296.0);
                    t = f >= 4294967294.0 ? 0xFFFFFFFEu : (uint32_t)f;
                }
                tab[(size_t)(nD + 2) * (kTabV * kTabJ) + (size_t)(nV + 16) * kTabJ + (size_t)(nJ + 16)] = t;
            }
}

// Packed triple an accepted move adds to the per-thread tracker.
uint32_t packed_triple(int nD, int nV, int nJ)
{
    return (1u << 27) | ((uint32_t)(nD + 2) << 20) | ((uint32_t)(nV + 16) << 10) | (uint32_t)(nJ + 16);
}

uint32_t threshold_of(const std::vector<uint32_t> &tab, int nD, int nV, int nJ)
{
    return tab[(size_t)(nD + 2) * (kTabV * kTabJ) + (size_t)(nV + 16) * kTabJ + (size_t)(nJ + 16)];
}

// Device threshold table: the reachable triples only (regions in kernels.h),
// each entry paired with its packed tracker triple.
void build_device_table(const std::vector<uint32_t> &tab, std::vector<uint32_t> &dev)
{
    dev.assign(2 * (size_t)kDevTabEntries, 0u);
    auto put = [&](size_t i, int nD, int nV, int nJ) {
        dev[2 * i] = threshold_of(tab, nD, nV, nJ);
        dev[2 * i + 1] = packed_triple(nD, nV, nJ);
    };
    for (int s = 0; s < 3; ++s)
        for (int nV = -8; nV <= 8; ++nV)
            for (int nJ = -8; nJ <= 8; ++nJ)
                put((size_t)s * kDevSlice + (size_t)(nV + 8) * 17 + (size_t)(nJ + 8), 2 * s - 2, nV, nJ);
    for (int v = -16; v <= 16; ++v) {
        put((size_t)kDevVLine + (size_t)(v + 16), 0, v, 0);
        put((size_t)kDevJLine + (size_t)(v + 16), 0, 0, v);
    }
}

// Transition table of section 3.1's coupled-pair move.  For pair state
// st = code_a | code_b << 2 and choice j < k_q: the j-th configuration of the
// same-charge set in the paper's listing order,
//   q=+1: (2,0) (2,1) (0,2) (1,2)
//   q= 0: (2,3) (3,2) (0,0) (1,1) (0,1) (1,0)
//   q=-1: (3,0) (3,1) (0,3) (1,3),
// and the coefficients that turn the neighbour sums (each offset by +4) into
// the device-table index of the move's (nD, nV, nJ).  Since the pair keeps its
// charge, dS_a + dS_b = 0 and the +4 offsets of the charge sums cancel; the
// spin offsets 4*(dsig_a + dsig_b) are folded into C.  The frozen states
// (|q| = 2) get one null move.  trans_d is the delta form (4 words an entry).
// The kernels' own tables (slots of device_common.h, quad.hip and batch.hip) are
// made at compile time; this one lists the moves for the host check of the tables.
[[maybe_unused]] void build_transition_table(std::vector<uint32_t> &trans, std::vector<uint32_t> &trans_d)
{
    static const int kS[4] = {0, 0, 1, -1}, kG[4] = {1, -1, 0, 0};
    static const int kPlus1[4][2] = {{2, 0}, {2, 1}, {0, 2}, {1, 2}};
    static const int kZero[6][2] = {{2, 3}, {3, 2}, {0, 0}, {1, 1}, {0, 1}, {1, 0}};
    static const int kMinus1[4][2] = {{3, 0}, {3, 1}, {0, 3}, {1, 3}};
    trans.assign(2 * (size_t)kTransEntries, 0u);
    trans_d.assign(4 * (size_t)kTransEntries, 0u);
    auto i8 = [](int v) { return (uint32_t)(uint8_t)(int8_t)v; };
    for (int st = 0; st < 16; ++st) {
        const int ca = st & 3, cb = st >> 2, q = kS[ca] + kS[cb];
        const int (*set)[2] = q == 1 ? kPlus1 : (q == 0 ? kZero : (q == -1 ? kMinus1 : nullptr));
        const int kq = set ? (q == 0 ? 6 : 4) : 1;
        for (int j = 0; j < kq; ++j) {
            const int a1 = set ? set[j][0] : ca, b1 = set ? set[j][1] : cb;
            const int dSa = kS[a1] - kS[ca], dSb = kS[b1] - kS[cb];
            const int dGa = kG[a1] - kG[ca], dGb = kG[b1] - kG[cb];
            const int nD = kS[a1] * kS[a1] + kS[b1] * kS[b1] - kS[ca] * kS[ca] - kS[cb] * kS[cb];
            uint32_t coef;
            int C;
            if (dSa == 2 || dSa == -2) {  // charge swap: V line, nJ = 0
                coef = i8(dSa) | (i8(dSb) << 8);
                C = kDevVLine + 16;
            } else if (dGa == 2 || dGa == -2 || dGb == 2 || dGb == -2) {  // spin change: J line, nV = 0
                coef = (i8(dGa) << 16) | (i8(dGb) << 24);
                C = kDevJLine + 16 - 4 * (dGa + dGb);
            } else {  // |dS|, |dsig| <= 1: slice nD/2 + 1
                coef = i8(17 * dSa) | (i8(17 * dSb) << 8) | (i8(dGa) << 16) | (i8(dGb) << 24);
                C = (nD / 2 + 1) * kDevSlice + 8 * 17 + 8 - 4 * (dGa + dGb);
            }
            trans[2 * (size_t)(st * 6 + j)] = coef;
            trans[2 * (size_t)(st * 6 + j) + 1] = (uint32_t)C | ((uint32_t)(a1 | (b1 << 2)) << 16);
            uint32_t *d = &trans_d[4 * (size_t)(st * 6 + j)];
            d[0] = coef;
            d[1] = (uint32_t)C;
            d[2] = (uint32_t)(a1 ^ ca) * 0x5555u | ((uint32_t)(b1 ^ cb) * 0x5555u) << 16;
            d[3] = 0u;
        }
    }
}

Tuning2Bit tuning_from_env()
{
    Tuning2Bit t{0, 0, 0, 0};
    if (const char *v = std::getenv("LATTICE_2BIT_ROWS")) t.rows_per_block = std::atoi(v);
    if (const char *v = std::getenv("LATTICE_2BIT_BLOCKS_PER_CU")) t.blocks_per_cu = std::atoi(v);
    if (const char *v = std::getenv("LATTICE_2BIT_WAVES")) t.waves_hint = std::atoi(v);
    if (const char *v = std::getenv("LATTICE_PERSISTENT")) t.persistent = std::atoi(v);
    return t;
}

// Canonical row-major codes <-> device encoding.
void to_device_layout(int32_t L, int32_t enc, const std::vector<int8_t> &codes, std::vector<uint8_t> &out)
{
    const size_t N = (size_t)L * L;
    if (enc == LAT_ENC_INT8) {
        out.assign((const uint8_t *)codes.data(), (const uint8_t *)codes.data() + N);
        return;
    }
    const size_t W = (size_t)L / 64, H = (size_t)L / 2, csz = H * W;
    std::vector<uint32_t> words(N / 16, 0u);
    for (size_t y = 0; y < (size_t)L; ++y)
        for (size_t x = 0; x < (size_t)L; ++x) {
            const size_t c = 4 * (y & 1) + (x & 3), X = x >> 2, Y = y >> 1;
            words[c * csz + Y * W + (X >> 4)] |= (uint32_t)(codes[y * L + x] & 3) << (2 * (X & 15));
        }
    out.resize(N / 4);
    std::memcpy(out.data(), words.data(), N / 4);
}

// The initial state of lattice_create in the device encoding.
void initial_state(const lat_params &p, int64_t Q, int64_t Nc, std::vector<uint8_t> &dev)
{
    std::vector<int8_t> codes;
    if (p.init_codes)
        codes.assign(p.init_codes, p.init_codes + (int64_t)p.L * p.L);
    else
        seeded_init(p.L, p.seed, (Nc + Q) / 2, (Nc - Q) / 2, codes);
    to_device_layout(p.L, p.encoding, codes, dev);
}

// Seeded states are made on the device at every side (L = 8: 0.117 ms a lattice
// with the host's keys, 0.102 with the device's; L = 64 0.149 and 0.088).
// Without a device the host's state is still made first, and what it lacks for
// that is what the caller is told.
bool seeds_on_device(const lat_params &p)
{
    int device = 0;
    return launch_seed && !p.init_codes && hipGetDevice(&device) == hipSuccess;
}

// Elements the device keeps at a rank; LATTICE_SEED_CANDIDATES lowers it (tests
// take the host's way out with 0).
uint32_t seed_candidates()
{
    const char *v = std::getenv("LATTICE_SEED_CANDIDATES");
    return v ? (uint32_t)std::min(std::max(std::atoi(v), 0), (int)kSeedCap) : kSeedCap;
}

// Staging of lattice_create: the scratch up to its observable slots, the full
// threshold table, and the seeding's overflow flag.
constexpr size_t kCreateFlag = kScrObsSlots + ((size_t)kTabSize * 4 + 255) / 256 * 256;
constexpr size_t kCreateBytes = kCreateFlag + 256;
static_assert(kCreateBytes <= kPinnedLarge, "lattice_create's staging");

// Codes of a state in the 2-bit class layout.
void codes_from_words(int32_t L, const uint32_t *words, int8_t *codes)
{
    const size_t W = (size_t)L / 64, H = (size_t)L / 2, csz = H * W;
    for (size_t y = 0; y < (size_t)L; ++y)
        for (size_t x = 0; x < (size_t)L; ++x) {
            const size_t c = 4 * (y & 1) + (x & 3), X = x >> 2, Y = y >> 1;
            codes[y * L + x] = (int8_t)((words[c * csz + Y * W + (X >> 4)] >> (2 * (X & 15))) & 3u);
        }
}

// Schedule of sweep s (section 3.2: non-interacting pairs, long-range
// partners): r in {1,2,3}; phase p has D_p = (r + 4 m_p, 1 + 2 k_p).
struct Schedule {
    int r, m[4], k[4];
};

Schedule sweep_schedule(int32_t L, uint64_t seed, uint64_t s)
{
    uint32_t Wd[12];
    for (uint32_t t = 0; t < 3; ++t) {
        const u32x4 w = philox4x32_10((uint32_t)s, kDomSchedule, t, (uint32_t)(s >> 32), (uint32_t)seed,
                                      (uint32_t)(seed >> 32));
        Wd[4 * t] = w.x;
        Wd[4 * t + 1] = w.y;
        Wd[4 * t + 2] = w.z;
        Wd[4 * t + 3] = w.w;
    }
    Schedule sc;
    sc.r = 1 + (int)(((uint64_t)(Wd[0] >> 8) * 3u) >> 24);
    for (int p = 0; p < 4; ++p) {
        sc.m[p] = (int)mulhi_u32(Wd[1 + 2 * p], (uint32_t)(L / 4));
        sc.k[p] = (int)mulhi_u32(Wd[2 + 2 * p], (uint32_t)(L / 2));
    }
    return sc;
}

}  // namespace

namespace lat {
namespace detail {

namespace {

// The buffer and encoding the off-chip kernels sweep: the lattice's own
// state, or the 2-bit copy of a packed int8 lattice.
void *swept_state(const lattice *h) { return h->packed ? (void *)(h->d_scratch + kScrWork) : h->d_state; }
int swept_enc(const lattice *h) { return h->packed ? LAT_ENC_2BIT : h->enc; }
// Off the chip and swept as the int8 sites they are.
bool by_bytes(const lattice *h)
{
    return h->path != kPathLds && h->path != kPathWords && swept_enc(h) == LAT_ENC_INT8;
}

// Host-scheduled path: four phase launches per sweep, then the device-side
// sweep counter is advanced to match.
int enqueue_phase_sweeps(lattice *h, uint32_t sweeps, hipStream_t stream)
{
    PhaseArgs a{};
    a.state = swept_state(h);
    a.dev_tab = (const uint2 *)(h->d_scratch + kScrDevTab);
    a.track = (unsigned long long *)(h->d_scratch + kScrSlots);
    a.L = h->L;
    a.magicW = magic_div((uint32_t)h->L >> 6);
    a.key0 = (uint32_t)h->seed;
    a.key1 = (uint32_t)(h->seed >> 32);
    uint32_t left = sweeps;
    if (h->tuning.persistent && !stream) {  // as enqueue_words_persistent: on the default stream only
        // one cooperative launch per chunk; the barrier counter stays far below 2^32
        constexpr uint32_t kChunk = 65536;
        while (left > 0) {
            const uint32_t n = std::min(left, kChunk);
            const uint64_t s = h->start_sweep + h->done + (sweeps - left);
            a.s_lo = (uint32_t)s;
            a.s_hi = (uint32_t)(s >> 32);
            const hipError_t e = launch_sweeps_2bit(a, h->tuning, n, (unsigned *)(h->d_scratch + kScrBarrier),
                                                    (unsigned *)(h->d_scratch + kScrErr), stream);
            if (e == hipErrorNotSupported) break;  // no co-residency guarantee: per-phase launches below
            if (e != hipSuccess) return hip_fail(e, "persistent sweep launch");
            left -= n;
        }
    }
    for (uint32_t i = sweeps - left; i < sweeps; ++i) {
        const uint64_t s = h->start_sweep + h->done + i;
        const Schedule sc = sweep_schedule(h->L, h->seed, s);
        a.s_lo = (uint32_t)s;
        a.s_hi = (uint32_t)(s >> 32);
        a.r = sc.r;
        for (int p = 0; p < 4; ++p) {
            a.p = p;
            a.m = sc.m[p];
            a.k = sc.k[p];
            const hipError_t e = launch_phase_2bit(a, h->tuning, stream);
            if (e != hipSuccess) return hip_fail(e, "phase kernel launch");
        }
    }
    if (sweeps > 0) {
        const hipError_t e = launch_advance((LatDesc *)(h->d_scratch + kScrDesc), sweeps, stream);
        if (e != hipSuccess) return hip_fail(e, "advance kernel launch");
    }
    h->done += sweeps;
    return LAT_OK;
}

// Threads per block of the per-phase word kernel (LATTICE_WORDS_BLOCK: a
// multiple of 64 up to 1024).
int words_phase_threads()
{
    const char *v = std::getenv("LATTICE_WORDS_BLOCK");
    const int want = v ? std::atoi(v) : 0;
    return want >= 64 && want <= kWordsPhaseMaxThreads && want % 64 == 0 ? want : kWordsThreads;
}

// The rows of a per-phase launch over the a.count lattices of a, lattice i with nb[i]
// blocks: runs as short as the arguments' room for rows allows, so that lattices of unequal
// sides leave few blocks without work.  (L = 2048 with seven of L = 320, one sweep: 63 us
// with a row a lattice, 39 us so; L = 1024 with forty of 320 59 and 44.)
void rows_of_runs(WordsArgs &a, const uint32_t *nb)
{
    const WordsArgs lattices = a;
    const int count = a.count;
    auto rows = [&](uint32_t run) {
        uint32_t n = 0;
        for (int i = 0; i < count; ++i) n += (nb[i] + run - 1) / run;
        return n;
    };
    uint32_t least = nb[0], most = nb[0];
    for (int i = 1; i < count; ++i) least = std::min(least, nb[i]), most = std::max(most, nb[i]);
    const uint32_t room = (uint32_t)(count <= kWordsFew ? kWordsFew : kWordsBatch);
    uint32_t run = least;
    while (run < most && rows(run) > room) run = std::min(most, run + (run + 3) / 4);
    a.max_blocks = run;
    a.count = 0;
    for (int i = 0; i < count; ++i)
        for (uint32_t first = 0; first < nb[i]; first += run) {
            a.scratch[a.count] = lattices.scratch[i];
            a.sweeps[a.count] = lattices.sweeps[i];
            a.run[a.count++] = first | nb[i] << 16;
        }
}

// Multi-block word path: lattices in groups of up to kWordsBatch per launch,
// one launch per phase of every sweep of the series (the lattice i of a
// group skips the sweeps past sweeps[i]), then the device sweep counters
// are advanced.  Q (lanes per a-word) is chosen by the largest L of the
// group; every lattice's blocks must fit its kMaxSlots tracker slots.
// bytes: int8 lattices as they are.
int enqueue_words_sweeps(lattice *const *hs, int32_t count, const uint32_t *sweeps, uint32_t uniform,
                         hipStream_t stream, bool bytes)
{
    for (int32_t b = 0; b < count; b += kWordsBatch) {
        WordsArgs a{};
        a.count = std::min<int32_t>(kWordsBatch, count - b);
        int max_L = 0;
        for (int i = 0; i < a.count; ++i) max_L = std::max(max_L, hs[b + i]->L);
        int Q = bytes ? 0 : words_lanes(max_L);
        // LATTICE_WORDS_PHASE_LANES (1, 2, 4 or 8) overrides the lanes per a-word
        if (const char *v = bytes ? nullptr : std::getenv("LATTICE_WORDS_PHASE_LANES")) {
            const int want = std::atoi(v);
            if (want == 1 || want == 2 || want == 4 || want == 8) Q = want;
        }
        const int threads = words_phase_threads();
        a.threads = (uint32_t)threads;
        uint32_t most = 0, nb[kWordsBatch];
        for (int i = 0; i < a.count; ++i) {
            const lattice *h = hs[b + i];
            nb[i] = bytes ? bytes_blocks(h->L, threads) : words_blocks(h->L, Q, threads);
            if (!bytes && nb[i] > (uint32_t)kMaxSlots) return fail(LAT_EINVAL, "lattice too large for the multi-block word kernel");
            a.scratch[i] = h->d_scratch;
            a.sweeps[i] = sweeps ? sweeps[b + i] : uniform;
            most = std::max(most, a.sweeps[i]);
        }
        if (most == 0) continue;
        WordsArgs rows = a;
        rows_of_runs(rows, nb);
        for (uint32_t it = 0; it < most; ++it) {
            rows.iter = it;
            for (int p = 0; p < 4; ++p) {
                rows.p = p;
                const hipError_t e = launch_phase_words(rows, Q, threads, stream);
                if (e != hipSuccess) return hip_fail(e, "word phase kernel launch");
            }
        }
        const hipError_t e = launch_advance_words(a, stream);
        if (e != hipSuccess) return hip_fail(e, "advance kernel launch");
        for (int i = 0; i < a.count; ++i) hs[b + i]->done += a.sweeps[i];
    }
    return LAT_OK;
}

}  // namespace

constexpr int kWordsPersistentMaxL = 2048;

namespace {

// Resident-block capacity of the persistent word kernel per (device, Q),
// looked up once.
int words_capacity(int Q, int threads)
{
    static std::mutex mu;
    static auto &cache = *new std::map<std::tuple<int, int, int>, int>;  // never destroyed, as the pinned pool
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_tuple(dev, Q, threads);
    auto it = cache.find(key);
    if (it == cache.end()) it = cache.emplace(key, words_persistent_capacity(Q, threads)).first;
    return it->second;
}

// Bounds of the waits of the persistent kernels, in ticks: of each device-wide
// barrier, kBarrierTimeoutTicks, and of the blocks' first meeting, kAssembleTicks,
// unless the environment asks for another (non-negative) count.  Tests use 0 to
// force the way out of a wait that takes too long: a barrier flags the state
// invalid and goes on, the first meeting calls the launch off.
long long ticks_from_env(const char *name, long long ticks)
{
    if (const char *v = std::getenv(name)) {
        const long long want = std::atoll(v);
        if (want >= 0) return want;
    }
    return ticks;
}
void set_bounds(WordsSeriesArgs &a)
{
    a.barrier_ticks = ticks_from_env("LATTICE_BARRIER_TICKS", kBarrierTimeoutTicks);
    a.assemble_ticks = ticks_from_env("LATTICE_ASSEMBLE_TICKS", kAssembleTicks);
}

// Lanes per a-word and block size of the persistent word kernel for the n
// lattices of a launch.  A phase is a chain of latencies, which more lanes
// shorten (8 lanes: two pairs each) as long as a lattice's blocks still meet on
// one counter, which is faster up to 64 of them; so for one lattice as many
// lanes as 64 blocks of 256 threads hold, but at least 2.  Above L = 1024 the
// blocks meet in two levels anyway, and 4 lanes in blocks of 512 threads
// measured best.  us a sweep, plain / with observables, for 2 lanes, 4 lanes, 4 in
// blocks of 512, 8 lanes: L = 512 12.8/14.4, 10.6/12.1, 12.3/13.9, 9.6/12.0;
// L = 1024 12.3/14.7, 13.3/16.3, 12.4/14.9, 12.2/15.0; L = 2048 15.8/19.2,
// 16.2/19.5, 14.2/18.3, 20.3/25.2.  Several lattices take fewer lanes until
// a block a compute unit holds them all, since more lanes load more words in
// all: 8 of L = 512 with 8 / 4 / 2 lanes 11.7 / 10.7 / 13.1 us, 48 of them
// with 8 / 1 33.6 / 21.8, 4 of L = 2048 with 4 / 1 45.6 / 24.3.
// LATTICE_WORDS_LANES (1, 2, 4 or 8) and LATTICE_WORDS_SERIES_BLOCK (a multiple
// of 64 up to the largest for the lanes) override.
struct WordsShape {
    int Q, threads;
};
WordsShape words_series_shape(lattice *const *hs, int32_t n)
{
    auto blocks = [&](const WordsShape &w) {
        uint32_t sum = 0;
        for (int32_t i = 0; i < n; ++i) sum += words_blocks(hs[i]->L, w.Q, w.threads);
        return sum;
    };
    int max_L = 0;
    for (int32_t i = 0; i < n; ++i) max_L = std::max(max_L, hs[i]->L);
    WordsShape w{8, kWordsThreads};
    if (max_L > 1024)
        w = {4, kWordsSeriesMaxThreads};
    else
        while (w.Q > 2 && words_blocks(max_L, w.Q) > 64u) w.Q /= 2;
    while (n > 1 && w.Q > 1 && blocks(w) > 256u) {
        w.Q /= 2;
        if (w.Q < 4) w.threads = kWordsThreads;
    }
    if (const char *v = std::getenv("LATTICE_WORDS_LANES")) {
        const int want = std::atoi(v);
        if (want == 1 || want == 2 || want == 4 || want == 8) w.Q = want;
    }
    const int most = w.Q >= 4 ? kWordsSeriesMaxThreads : kWordsThreads;
    w.threads = std::min(w.threads, most);
    if (const char *v = std::getenv("LATTICE_WORDS_SERIES_BLOCK")) {
        const int want = std::atoi(v);
        if (want >= 64 && want <= most && want % 64 == 0) w.threads = want;
    }
    return w;
}
// Of int8 lattices: the smallest blocks of which one a compute unit holds a
// call a thread, up to 512 threads; bytes_fit: whether there are such.
uint32_t blocks_of_all(lattice *const *hs, int32_t n, int threads)
{
    uint32_t sum = 0;
    for (int32_t i = 0; i < n; ++i) sum += bytes_blocks(hs[i]->L, threads);
    return sum;
}
bool bytes_fit(lattice *const *hs, int32_t n) { return n <= kWordsBatch && blocks_of_all(hs, n, 2 * kWordsThreads) <= 256u; }
WordsShape bytes_series_shape(lattice *const *hs, int32_t n)
{
    WordsShape w{0, blocks_of_all(hs, n, kWordsThreads) <= 256u ? kWordsThreads : 2 * kWordsThreads};
    if (const char *v = std::getenv("LATTICE_WORDS_SERIES_BLOCK")) {
        const int want = std::atoi(v);
        if (want >= 64 && want <= kBytesSeriesMaxThreads && want % 64 == 0) w.threads = want;
    }
    return w;
}

}  // namespace

namespace {
// A captured kernel node would not guarantee that all blocks are resident at once.
bool captured(hipStream_t stream)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess) (void)hipGetLastError();
    return capture != hipStreamCaptureStatusNone;
}
}  // namespace

int enqueue_words_persistent(lattice *const *hs, int32_t count, const uint32_t *sweeps, uint32_t intervals,
                             uint32_t every, long long *records, hipStream_t stream, bool bytes, bool *ran)
{
    *ran = false;
    if (count <= 0 || intervals == 0 || every == 0 || stream) return LAT_OK;
    int max_L = 0;
    uint32_t longest = 0;
    for (int32_t i = 0; i < count; ++i) {
        if (bytes && (records || (uintptr_t)hs[i]->d_state % 4 != 0)) return LAT_OK;
        max_L = std::max(max_L, hs[i]->L);
        longest = std::max(longest, sweeps ? sweeps[i] : every);
    }
    // default: on for every lattice of this path, against one launch per phase
    // (us a sweep, plain / with observables after every sweep): L = 512
    // 9.5 / 11.8 against 15.5 / 25.6, L = 1024 12.0 / 14.5 against 15.8 /
    // 26.0, L = 2048 14.6 / 17.8 against 17.9 / 28.2.
    // A call of one sweep is the other way round (from an idle stream to its end
    // 30.2 us against 28.3 at L = 512, 35.7 against 31.2 at L = 2048; with its record
    // 41.9 against 38.3 and 48.3 against 41.5).  Of int8 lattices
    // as they are: as long as a block a compute unit holds a call a thread (us a
    // sweep, persistent / launches: L = 388 10.7 / 17.5, L = 1000 15.0 / 19.3, 8 of
    // L = 500 22.6 / 24.9; but L = 2000 32.8 / 34.2, 48 of L = 500 75 / 69, L = 4000 97 / 72).
    // Never on a stream of the caller's own, whatever is asked for: launches of
    // several streams would take places that the blocks of the others wait for, and a
    // program that ran them (as cooperative launches) from six threads with a
    // stream each ended in a segmentation fault at its exit whose cause is not
    // known.
    // LATTICE_WORDS_PERSISTENT=0|1 overrides the other rules.
    const char *v = std::getenv("LATTICE_WORDS_PERSISTENT");
    if (v) {
        if (std::atoi(v) == 0) return LAT_OK;
    } else {
        if (longest < 2 && intervals == 1) return LAT_OK;
        if (bytes ? !bytes_fit(hs, count) : max_L > kWordsPersistentMaxL) return LAT_OK;
    }
    if (records && count != 1) return fail(LAT_EINVAL, "an observation series holds one lattice");
    if (captured(stream)) return LAT_OK;
    // the barrier counter counts blocks x barriers: at most 2^20 barriers per
    // launch keeps it below 2^32 for any resident grid
    constexpr uint64_t kMaxBarriers = 1u << 20;
    const uint64_t per_interval = 4ull * every;
    if (per_interval > kMaxBarriers && records) return LAT_OK;  // such intervals take the per-phase launches
    const uint32_t sweeps_cap = (uint32_t)(kMaxBarriers / 4);
    const uint32_t intervals_cap = records ? (uint32_t)std::max<uint64_t>(1, kMaxBarriers / per_interval) : 1u;

    // lattices in launches of at most kWordsBatch, each with its share of the
    // resident blocks
    for (int32_t g0 = 0; g0 < count; g0 += kWordsBatch) {
        const int32_t n = std::min<int32_t>(kWordsBatch, count - g0);
        const WordsShape shape = bytes ? bytes_series_shape(hs + g0, n) : words_series_shape(hs + g0, n);
        const int Q = shape.Q, threads = shape.threads;
        const int capacity = words_capacity(Q, threads);
        if (capacity <= 0) return *ran ? fail(LAT_EHIP, "persistent word launch is not possible") : LAT_OK;
        // every lattice the blocks it asks for, or, where they are not resident
        // together, at most an equal share
        uint32_t nb[kWordsBatch];
        auto give = [&](uint32_t most) {
            uint32_t sum = 0;
            for (int32_t i = 0; i < n; ++i) {
                const int L = hs[g0 + i]->L;
                sum += nb[i] = std::min(bytes ? bytes_blocks(L, threads) : words_blocks(L, Q, threads), most);
            }
            return sum;
        };
        uint32_t total = give((uint32_t)kMaxSlots);
        if (total > (uint32_t)capacity)
            total = give(std::min((uint32_t)kMaxSlots, std::max(1u, (uint32_t)capacity / (uint32_t)n)));
        if (total > (uint32_t)capacity) return *ran ? fail(LAT_EHIP, "persistent word launch does not fit") : LAT_OK;
        if (records) {
            lattice *h = hs[g0];
            for (uint32_t k = 0; k < intervals; k += intervals_cap) {
                WordsSeriesArgs a{};
                a.count = 1;
                a.threads = threads;
                set_bounds(a);
                a.intervals = std::min(intervals_cap, intervals - k);
                a.every = every;
                a.records = records + (kSeriesRecord / 8) * (size_t)k;
                a.scratch[0] = h->d_scratch;
                a.sweeps[0] = a.intervals * every;
                a.first_block[0] = 0;
                a.first_block[1] = nb[0];
                // the state before the launch into its first record, by the reduction
                // over many blocks (one block took 60 us at L = 1024 and 200 at L = 2048)
                hipError_t e = launch_observables(h->d_scratch, swept_state(h), h->L, LAT_ENC_2BIT, stream, a.records);
                if (e == hipSuccess) e = launch_words_series(a, Q, stream);
                if (e != hipSuccess) return hip_fail(e, "persistent word kernel launch");
                h->done += (uint64_t)a.sweeps[0];
            }
            h->ran_persistent = true;
            *ran = true;
            continue;
        }
        uint32_t most = 0;
        for (int32_t i = 0; i < n; ++i) most = std::max(most, sweeps ? sweeps[g0 + i] : every);
        for (uint32_t c = 0; c < most; c += sweeps_cap) {
            WordsSeriesArgs a{};
            a.threads = threads;
            set_bounds(a);
            a.intervals = 1;
            a.every = 0;
            uint32_t blocks = 0;
            for (int32_t i = 0; i < n; ++i) {
                const uint32_t want = sweeps ? sweeps[g0 + i] : every;
                const uint32_t k = want > c ? std::min(sweeps_cap, want - c) : 0u;
                if (k == 0) continue;
                a.scratch[a.count] = hs[g0 + i]->d_scratch;
                a.sweeps[a.count] = k;
                a.first_block[a.count] = blocks;
                blocks += nb[i];
                a.every = std::max(a.every, k);
                ++a.count;
                hs[g0 + i]->done += k;
                hs[g0 + i]->ran_persistent = true;
            }
            a.first_block[a.count] = blocks;
            if (a.count == 0) continue;
            const hipError_t e = launch_words_series(a, Q, stream);
            if (e != hipSuccess) return hip_fail(e, "persistent word kernel launch");
        }
        *ran = true;
    }
    return LAT_OK;
}

// Whether few on-chip lattices of large sides are faster spread over many blocks
// in the persistent kernels than with a compute unit each, for calls of
// `sweeps` sweeps that cost `extra` ns more that way.  ns a sweep: on the chip
// 0.229 L^2 in the four-pair form and 0.34 L^2 per site (L = 256 14.9 us, L = 340
// 38.5); spread 9.9 us with two bits a site (also 16 lattices of L = 256), and as bytes
// 10.5 and up to 3 more when every compute unit has a block (L = 200 10.6, L = 340
// 10.5, L = 384 with 63 of L = 100 13.5).
// Lattices whose path was asked for stay on it, and so do those on a stream of
// their own: side by side with others, a compute unit each is the better use.
bool spreads(lattice *const *hs, int32_t count, uint64_t sweeps, double extra, hipStream_t stream)
{
    if (count < 1 || count > kWordsBatch || stream) return false;
    int max_L = 0;
    bool quad = true;
    for (int32_t i = 0; i < count; ++i) {
        if (hs[i]->path_asked || hs[i]->enc != hs[0]->enc || (uintptr_t)hs[i]->d_state % 4 != 0) return false;
        max_L = std::max(max_L, hs[i]->L);
        quad = quad && hs[i]->L % 16 == 0;
    }
    const uint32_t blocks = blocks_of_all(hs, count, kWordsThreads);
    if (blocks > 256u) return false;
    const double on_chip = (quad ? 0.229 : 0.34) * max_L * max_L;
    const double spread = hs[0]->enc == LAT_ENC_INT8 ? 10500.0 + 13.0 * blocks : 9900.0;
    return (double)sweeps * (on_chip - spread) > extra && !captured(stream);
}
// Three launches against one (two sweeps of one lattice of L = 256 on the chip and
// spread 48.5 and 40.2 us; of 16 53.6 and 47.9).
constexpr double kSpreadCall = 4000.0;

// Lattices that the whole chip does together in the time of one on its compute unit.
constexpr double kUnitsWorth = 75.0;

// Sweeps of on-chip lattices outside the server and graphs.
int enqueue_small_sweeps(lattice *const *hs, int32_t count, uint32_t sweeps, hipStream_t stream)
{
    if (spreads(hs, count, sweeps, kSpreadCall, stream)) {
        bool ran = false;
        const int rc = enqueue_words_persistent(hs, count, nullptr, 1, sweeps, nullptr, stream,
                                                hs[0]->enc == LAT_ENC_INT8, &ran);
        if (rc || ran) return rc;
    }
    return enqueue_lds_sweeps(hs, count, nullptr, sweeps, stream);
}

// Whether int8 lattices off the chip (lattice i by sweeps[i]) are faster with a
// compute unit each, all side by side, than spread over the chip together: the
// longest of them takes 0.46 ns a site and sweep that way, all of them together
// 0.0050 to 0.0067 ns this way (us for 20 sweeps of 64 / 80 / 96 / 256 lattices, a unit
// each and together: L = 388 1418 / 1420 / 1422 / 1451 and 1226 / 1787 / 2017 / 4945, L = 500
// 2329 / 2330 / 2330 / 2371 and 1588 / 2276 / 2687 / 6460).
bool one_unit_each(lattice *const *hs, const uint32_t *sweeps, size_t n)
{
    double sum = 0, longest = 0;
    for (size_t i = 0; i < n; ++i) {
        if (hs[i]->path != kPathBytes) return false;
        const double sites = (double)hs[i]->N * sweeps[i];
        sum += sites;
        longest = std::max(longest, sites);
    }
    return sum > kUnitsWorth * longest;
}

int enqueue_offchip_sweeps(lattice *const *hs, int32_t count, const uint32_t *sweeps, uint32_t uniform,
                           hipStream_t stream, bool convert, bool persistent)
{
    auto n_of = [&](int32_t i) { return sweeps ? sweeps[i] : uniform; };
    for (int32_t i = 0; i < count && convert; ++i) {
        if (!hs[i]->packed || n_of(i) == 0) continue;
        const hipError_t e = launch_pack_int8((const int8_t *)hs[i]->d_state,
                                              (uint32_t *)(hs[i]->d_scratch + kScrWork), hs[i]->L, stream);
        if (e != hipSuccess) return hip_fail(e, "int8 pack launch");
    }
    std::vector<lattice *> words, bytes;
    std::vector<uint32_t> words_n, bytes_n;
    for (int32_t i = 0; i < count; ++i) {
        if (hs[i]->path == kPathWords) {
            words.push_back(hs[i]);
            words_n.push_back(n_of(i));
        } else if (by_bytes(hs[i])) {
            bytes.push_back(hs[i]);
            bytes_n.push_back(n_of(i));
        } else {
            const int rc = enqueue_phase_sweeps(hs[i], n_of(i), stream);
            if (rc) return rc;
        }
    }
    if (!words.empty()) {
        bool ran = false;
        int rc = persistent ? enqueue_words_persistent(words.data(), (int32_t)words.size(), words_n.data(), 1, 1,
                                                       nullptr, stream, /*bytes=*/false, &ran)
                            : LAT_OK;
        if (rc == LAT_OK && !ran)
            rc = enqueue_words_sweeps(words.data(), (int32_t)words.size(), words_n.data(), 0, stream, /*bytes=*/false);
        if (rc) return rc;
    }
    // as many as there are compute units: one each
    for (size_t b = 0; b < bytes.size();) {
        const size_t n = std::min(bytes.size() - b, (size_t)kMaxBatch);
        if (!one_unit_each(&bytes[b], &bytes_n[b], n)) {
            b += n;
            continue;
        }
        const int rc = enqueue_lds_sweeps(&bytes[b], (int32_t)n, &bytes_n[b], 0, stream);
        if (rc) return rc;
        bytes.erase(bytes.begin() + (ptrdiff_t)b, bytes.begin() + (ptrdiff_t)(b + n));
        bytes_n.erase(bytes_n.begin() + (ptrdiff_t)b, bytes_n.begin() + (ptrdiff_t)(b + n));
    }
    if (!bytes.empty()) {
        bool ran = false;
        int rc = persistent ? enqueue_words_persistent(bytes.data(), (int32_t)bytes.size(), bytes_n.data(), 1, 1,
                                                       nullptr, stream, /*bytes=*/true, &ran)
                            : LAT_OK;
        if (rc == LAT_OK && !ran)
            rc = enqueue_words_sweeps(bytes.data(), (int32_t)bytes.size(), bytes_n.data(), 0, stream, /*bytes=*/true);
        if (rc) return rc;
    }
    for (int32_t i = 0; i < count && convert; ++i) {
        if (!hs[i]->packed || n_of(i) == 0) continue;
        const hipError_t e = launch_unpack_int8((const uint32_t *)(hs[i]->d_scratch + kScrWork),
                                                (int8_t *)hs[i]->d_state, hs[i]->L, stream);
        if (e != hipSuccess) return hip_fail(e, "int8 unpack launch");
    }
    return LAT_OK;
}

int enqueue_observables_batch(lattice *const *hs, int32_t count, unsigned long long *dev, hipStream_t stream)
{
    for (int32_t b = 0; b < count; b += kMaxBatch) {
        BatchArgs a{};
        a.count = std::min<int32_t>(kMaxBatch, count - b);
        for (int i = 0; i < a.count; ++i) a.scratch[i] = hs[b + i]->d_scratch;
        const hipError_t e = launch_observables_batch(a, dev + 10 * (size_t)b, stream);
        if (e != hipSuccess) return hip_fail(e, "batched observables launch");
    }
    return LAT_OK;
}

// Batches whose sides are all multiples of 16 take the quad form from this
// largest side on: below, its few threads leave the chain of a phase longer than
// the per-site form's (us a sweep, quad / per site: L = 48 2.9 / 2.0, L = 64
// 2.9 / 2.2, L = 80 3.0 / 3.2, L = 128 4.1 / 4.7, L = 256 15.0 / 22.0).
constexpr int kQuadMinL = 80;

// Batched path: lattices resident in LDS, up to kMaxBatch per launch.
int enqueue_lds_sweeps(lattice *const *hs, int32_t count, const uint32_t *sweeps, uint32_t uniform,
                       hipStream_t stream, const ObsTarget *obs)
{
    // LATTICE_BATCH_THREADS pins the block size
    const char *pinned = std::getenv("LATTICE_BATCH_THREADS");
    const int threads = pinned ? std::atoi(pinned) : 0;
    // LATTICE_LDS_SITE=1 keeps every batch on the per-site form (tests compare the two)
    const char *env = std::getenv("LATTICE_LDS_SITE");
    const bool force_site = env && env[0] == '1';
    for (int32_t b = 0; b < count; b += kMaxBatch) {
        BatchArgs a{};
        a.count = std::min<int32_t>(kMaxBatch, count - b);
        int max_L = 0;
        bool quad = !force_site;
        for (int i = 0; i < a.count; ++i) {
            a.scratch[i] = hs[b + i]->d_scratch;
            a.sweeps[i] = sweeps ? sweeps[b + i] : uniform;
            max_L = std::max(max_L, hs[b + i]->L);
            quad = quad && hs[b + i]->L % 16 == 0;
        }
        quad = quad && max_L >= kQuadMinL && max_L <= kQuadMaxL;
        const uint32_t intervals = obs ? obs->intervals : 1u;
        // one launch holds as many intervals as kFusedSweeps sweeps allow
        const uint32_t most = *std::max_element(a.sweeps, a.sweeps + a.count);
        const uint32_t per_launch = std::max(1u, kFusedSweeps / std::max(1u, most));
        a.obs_words = obs ? obs->words : 10u;
        a.obs_stride = obs ? obs->stride : 0u;
        for (uint32_t k = 0; k < intervals; k += per_launch) {
            a.intervals = std::min(per_launch, intervals - k);
            a.obs_out = obs ? obs->dev + (size_t)obs->stride * k + (size_t)obs->words * (size_t)b : nullptr;
            const hipError_t e = launch_sweep_lds(a, max_L, threads, quad, stream);
            if (e != hipSuccess) return hip_fail(e, "batched kernel launch");
            for (int i = 0; i < a.count; ++i) hs[b + i]->done += (uint64_t)a.sweeps[i] * a.intervals;
        }
    }
    return LAT_OK;
}

// v = (tracker nD, nV, nJ, sum S, sum S^2, bonds SS, bonds ss, M, M_st, C_st).
bool barrier_may_time_out(const lattice *h)
{
    return h->ran_persistent || (h->path == kPathPhase && h->tuning.persistent);
}

// The records come through pinned memory, those that do not fit at once in two
// halves of it: one is copied while the other is handed out.  (A copy of 3.6 MB
// takes 205 us into ordinary memory whose pages are there and 1450 us into new
// pages, 70 us into pinned memory and 95 in pieces of 1 MiB.)  Without pinned
// memory, an ordinary buffer holds them all.
int read_records(const char *what, const void *dev, uint32_t words, size_t n, lattice *const *hs, size_t count,
                 bool always, hipStream_t stream, const std::function<void(size_t, const int64_t *, size_t)> &fill)
{
    const size_t size = 8 * (size_t)words;
    std::vector<uint8_t *> swept;  // scratch of the lattices whose flags are read
    for (size_t i = 0; i < count; ++i)
        if (always || barrier_may_time_out(hs[i])) swept.push_back(hs[i]->d_scratch);
    // A copy a flag is 2.7 us each; kernels gather those of up to kMaxBatch
    // lattices into a word of pinned memory (records of 256 lattices of L = 256, 64
    // of them swept by persistent launches: 200 -> 62 us, 59 without a flag).
    constexpr size_t kCopies = 2;
    size_t n_flags = swept.size() > kCopies ? (swept.size() + kMaxBatch - 1) / kMaxBatch : swept.size();
    size_t flag_bytes = (4 * n_flags + 7) / 8 * 8, bytes = flag_bytes + size * n;
    const bool large = bytes > kPinnedBytes;
    PinnedBlock stage(large);
    size_t room = large ? kPinnedLarge : kPinnedBytes;
    std::vector<int64_t> own;
    if (!stage.p || !launch_gather_flags || flag_bytes > room / 2) {
        n_flags = swept.size();  // kernels cannot write to ordinary memory
        flag_bytes = (4 * n_flags + 7) / 8 * 8;
        bytes = flag_bytes + size * n;
        own.resize(bytes / 8);
        room = bytes;
    }
    uint8_t *base = own.empty() ? (uint8_t *)stage.p : (uint8_t *)own.data(), *ring = base + flag_bytes;
    const size_t piece = bytes <= room ? n : (room - flag_bytes) / 2 / size;
    auto copy = [&](size_t k, size_t half) {
        const size_t m = std::min(piece, n - k);
        if (m == 0) return hipSuccess;
        return hipMemcpyAsync(ring + half * piece * size, (const uint8_t *)dev + k * size, m * size,
                              hipMemcpyDeviceToHost, stream);
    };
    hipError_t e = hipSuccess;
    for (size_t i = 0; i < n_flags && e == hipSuccess; ++i)
        if (n_flags == swept.size()) {
            e = hipMemcpyAsync(base + 4 * i, swept[i] + kScrErr, sizeof(uint32_t), hipMemcpyDeviceToHost, stream);
        } else {
            BatchArgs a{};
            const size_t first = i * kMaxBatch;
            a.count = (int)std::min(swept.size() - first, (size_t)kMaxBatch);
            std::copy_n(&swept[first], a.count, a.scratch);
            e = launch_gather_flags(a, (uint32_t *)base + i, stream);
        }
    if (e == hipSuccess) e = copy(0, 0);
    size_t k = 0, half = 0;
    do {
        const hipError_t waited = hipStreamSynchronize(stream);
        if (waited != hipSuccess) stage.abandon();
        if (e == hipSuccess) e = waited;
        if (e != hipSuccess) return hip_fail(e, what);
        if (k == 0)
            for (size_t i = 0; i < n_flags; ++i)
                if (((const uint32_t *)base)[i] & 1u) return barrier_timed_out();
        const int64_t *v = (const int64_t *)(ring + half * piece * size);
        const size_t m = std::min(piece, n - k);
        if (k + m < n) e = copy(k + m, half ^= 1u);
        fill(k, v, m);
        k += m;
    } while (k < n);
    return LAT_OK;
}

void fill_obs(const lattice *h, const int64_t *v, lat_obs *out)
{
    out->sweep = h->done;
    out->track_nD = v[0];
    out->track_nV = v[1];
    out->track_nJ = v[2];
    out->sum_S = v[3];
    out->n_charged = v[4];
    out->bond_SS = v[5];
    out->bond_ss = v[6];
    out->M = v[7];
    out->M_stag = v[8];
    out->C_stag = v[9];
    out->E = h->Delta * (double)out->n_charged + h->V * (double)out->bond_SS + 0.25 * h->J * (double)out->bond_ss;
}

// Parameter checks shared by lattice_create and the server's submit:
// geometry, finite couplings, T > 0, and the charge target of eq. (2) (from
// the given codes, which must lie in 0..3, or from n and n_charged).
int validate_params(const lat_params *p, int64_t *Q_out, int64_t *Nc_out)
{
    if (!valid_geometry(p->L, p->encoding))
        return fail(LAT_EINVAL, "invalid L for the encoding (int8: L%4==0; 2-bit: L%64==0; 4 <= L <= 32768)");
    if (!std::isfinite(p->Delta) || !std::isfinite(p->V) || !std::isfinite(p->J) || !std::isfinite(p->T) ||
        !std::isfinite(p->n))
        return fail(LAT_EINVAL, "parameters must be finite");
    if (!(p->T > 0.0)) return fail(LAT_EINVAL, "T must be > 0");
    int64_t Q = 0, Nc = 0;
    if (p->init_codes) {
        const int64_t N = (int64_t)p->L * p->L;
        for (int64_t i = 0; i < N; ++i) {
            const int c = p->init_codes[i];
            if (c < 0 || c > 3) return fail(LAT_EINVAL, "init code outside 0..3");
            Q += c == 2 ? 1 : (c == 3 ? -1 : 0);
            Nc += c >= 2;
        }
    } else {
        const int rc = charge_target(p->L, p->n, p->n_charged, &Q, &Nc);
        if (rc) return rc;
    }
    *Q_out = Q;
    *Nc_out = Nc;
    return LAT_OK;
}

}  // namespace detail
}  // namespace lat

namespace {

int enqueue_sweeps(lattice *h, uint32_t sweeps, hipStream_t stream)
{
    if (sweeps == 0) return LAT_OK;
    lattice *one[1] = {h};
    // the multi-block path takes the persistent launch where it can run
    if (h->path != kPathLds) return enqueue_offchip_sweeps(one, 1, nullptr, sweeps, stream);
    return enqueue_small_sweeps(one, 1, sweeps, stream);
}

// Sweep path of a new lattice.  Default: the one-block LDS kernel up to
// kLdsRouteMaxL, whose single compute unit is then still faster than a
// multi-block launch series; the multi-block word kernel up to kWordsMaxL;
// the one-thread-per-word phase kernel above.  LATTICE_PATH=lds|words|phase
// forces a path where it applies (lds: up to kLdsMaxL) (tests run every path at small sizes);
// LATTICE_FORCE_PHASE_KERNELS=1 is the same as LATTICE_PATH=phase.
constexpr int kLdsRouteMaxL = 256;
constexpr int kWordsMaxL = 2048;

int choose_path(int L, int enc)
{
    const bool words_ok = L % 64 == 0 && L <= kWordsMaxL;
    if (const char *v = std::getenv("LATTICE_PATH")) {
        const std::string want(v);
        if (want == "lds" && L <= kLdsMaxL) return kPathLds;
        if (want == "words" && words_ok) return kPathWords;
        if (want == "phase") return kPathPhase;
    }
    if (const char *force = std::getenv("LATTICE_FORCE_PHASE_KERNELS"))
        if (std::atoi(force) != 0) return kPathPhase;
    (void)enc;
    if (L <= (L % 64 == 0 ? kLdsRouteMaxL : kSiteMaxL)) return kPathLds;
    if (L % 64 != 0 && L <= kLdsMaxL) return kPathBytes;
    return words_ok ? kPathWords : kPathPhase;
}

}  // namespace

extern "C" {

size_t lattice_state_bytes(int32_t L, int32_t encoding)
{
    if (!valid_geometry(L, encoding)) return 0;
    const size_t N = (size_t)L * L;
    return encoding == LAT_ENC_INT8 ? N : N / 4;
}

size_t lattice_scratch_bytes(int32_t L, int32_t encoding)
{
    if (!valid_geometry(L, encoding)) return kScrBytes;
    return kScrBytes + (int8_packs(L, encoding) ? (size_t)L * L / 4 : 0);
}

int lattice_charge_target(int32_t L, double n, int64_t n_charged, int64_t *Q, int64_t *Nc)
{
    return guarded("lattice_charge_target", [&]() -> int {
        if (!Q || !Nc) return fail(LAT_EINVAL, "null output pointer");
        if (L < 1 || L > kMaxL) return fail(LAT_EINVAL, "L out of range");
        return charge_target(L, n, n_charged, Q, Nc);
    });
}

int lattice_create(const lat_params *p, void *d_state, size_t state_bytes, void *d_scratch, size_t scratch_bytes,
                   void *hip_stream, lattice **out)
{
    return guarded("lattice_create", [&]() -> int {
        g_err.clear();
        if (!p || !out) return fail(LAT_EINVAL, "null params or output handle");
        *out = nullptr;
        int64_t Q = 0, Nc = 0;
        int rc = validate_params(p, &Q, &Nc);
        if (rc) return rc;
        if (!d_state || !d_scratch) return fail(LAT_EINVAL, "null device buffer");
        if (state_bytes < lattice_state_bytes(p->L, p->encoding)) return fail(LAT_ENOMEM, "state buffer too small");
        if (scratch_bytes < lattice_scratch_bytes(p->L, p->encoding)) return fail(LAT_ENOMEM, "scratch buffer too small");

        const bool on_device = seeds_on_device(*p);
        std::vector<uint8_t> dev;
        if (!on_device) initial_state(*p, Q, Nc, dev);
        {
            static std::once_flag once;
            static hipError_t init_err = hipSuccess;
            std::call_once(once, [] {
                init_err = init_kernel_attributes();
                if (init_err == hipSuccess) init_err = init_map_kernel_attributes();
            });
            if (init_err != hipSuccess) return hip_fail(init_err, "kernel set-up");
        }

        std::unique_ptr<lattice> made(new lattice());
        lattice *h = made.get();
        h->L = p->L;
        h->enc = p->encoding;
        h->N = (int64_t)p->L * p->L;
        h->Q = Q;
        h->Nc = Nc;
        h->n = p->n;
        h->Delta = p->Delta;
        h->V = p->V;
        h->J = p->J;
        h->T = p->T;
        h->seed = p->seed;
        h->start_sweep = p->start_sweep;
        h->d_state = d_state;
        h->d_scratch = (uint8_t *)d_scratch;
        h->stream = (hipStream_t)hip_stream;
        h->tuning = tuning_from_env();
        h->path = choose_path(p->L, p->encoding);
        h->path_asked = std::getenv("LATTICE_PATH") != nullptr;
        h->packed = h->path != kPathLds && int8_packs(p->L, p->encoding);
        h->magic = kMagic;
        LatDesc desc{};
        desc.state = d_state;
        desc.L = p->L;
        desc.enc = p->encoding;
        desc.key0 = (uint32_t)p->seed;
        desc.key1 = (uint32_t)(p->seed >> 32);
        desc.next_sweep = p->start_sweep;

        // The seeded state is made on the device while the tables are made here;
        // nothing is allocated in between, so that the wait below is reached.
        std::vector<uint32_t> tab, dev_tab;
        tab.reserve(kTabSize);
        dev_tab.reserve(2 * (size_t)kDevTabEntries);
        PinnedBlock stage(/*large=*/true);
        std::vector<uint8_t> own;
        if (!stage.p) own.resize(kCreateBytes);
        uint8_t *img = stage.p ? (uint8_t *)stage.p : own.data();
        std::memset(img, 0, kCreateBytes);
        uint32_t *overflow = (uint32_t *)(img + kCreateFlag);
        hipError_t e = hipSuccess;
        if (on_device) {
            const SeedArgs s{d_state, h->d_scratch, stage.p ? overflow : (uint32_t *)(h->d_scratch + kScrErr),
                             (uint32_t)h->N, (uint32_t)h->L, (uint32_t)h->enc, desc.key0, desc.key1,
                             {(uint32_t)((Nc + Q) / 2), (uint32_t)Nc}, seed_candidates()};
            e = launch_seed(s, h->stream);
            if (e == hipSuccess && !stage.p)
                e = hipMemcpyAsync(overflow, s.overflow, sizeof(uint32_t), hipMemcpyDeviceToHost, h->stream);
        } else {
            e = hipMemcpyAsync(d_state, dev.data(), dev.size(), hipMemcpyHostToDevice, h->stream);
        }
        build_threshold_table(p->Delta, p->V, p->J, p->T, tab);
        build_device_table(tab, dev_tab);
        // tables, descriptor and a cleared tracker in two copies
        std::memcpy(img + kScrDevTab, dev_tab.data(), dev_tab.size() * 4);
        std::memcpy(img + kScrDesc, &desc, sizeof(desc));
        std::memcpy(img + kScrObsSlots, tab.data(), tab.size() * 4);
        if (e == hipSuccess) e = hipMemcpyAsync(h->d_scratch, img, kScrObsSlots, hipMemcpyHostToDevice, h->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(h->d_scratch + kScrFullTab, img + kScrObsSlots, tab.size() * 4, hipMemcpyHostToDevice,
                               h->stream);
        if (e == hipSuccess) e = launch_zero_i64((unsigned long long *)(h->d_scratch + kScrSlots), 3 * kMaxSlots, h->stream);
        hipError_t waited = hipStreamSynchronize(h->stream);  // host staging buffers die with this frame
        if (e == hipSuccess) e = waited;
        if (e == hipSuccess && on_device && *overflow != 0) {
            initial_state(*p, Q, Nc, dev);
            e = hipMemcpyAsync(d_state, dev.data(), dev.size(), hipMemcpyHostToDevice, h->stream);
            waited = hipStreamSynchronize(h->stream);
            if (e == hipSuccess) e = waited;
        }
        if (waited != hipSuccess) stage.abandon();
        if (e != hipSuccess) {
            h->magic = 0;
            return hip_fail(e, "lattice_create");
        }
        *out = made.release();
        return LAT_OK;
    });
}

int lattice_sweep(lattice *h, uint32_t sweeps)
{
    return guarded("lattice_sweep", [&]() -> int {
        if (!live(h)) return fail(LAT_ESTATE, "null or destroyed handle");
        return enqueue_sweeps(h, sweeps, h->stream);
    });
}

int lattice_sweep_batch(lattice *const *hs, int32_t count, uint32_t sweeps, void *hip_stream)
{
    return guarded("lattice_sweep_batch", [&]() -> int {
        if (count < 0 || (count > 0 && !hs)) return fail(LAT_EINVAL, "bad batch");
        for (int32_t i = 0; i < count; ++i)
            if (!live(hs[i])) return fail(LAT_ESTATE, "null or destroyed handle in batch");
        {
            std::vector<const lattice *> seen(hs, hs + count);
            std::sort(seen.begin(), seen.end());
            if (std::adjacent_find(seen.begin(), seen.end()) != seen.end())
                return fail(LAT_EINVAL, "a lattice appears twice in the batch");
        }
        if (sweeps == 0) return LAT_OK;
        std::vector<lattice *> small, big;
        for (int32_t i = 0; i < count; ++i) (hs[i]->path == kPathLds ? small : big).push_back(hs[i]);
        int rc = enqueue_small_sweeps(small.data(), (int32_t)small.size(), sweeps, (hipStream_t)hip_stream);
        if (rc == LAT_OK && !big.empty())
            rc = enqueue_offchip_sweeps(big.data(), (int32_t)big.size(), nullptr, sweeps, (hipStream_t)hip_stream);
        return rc;
    });
}

int lattice_observables_batch(lattice *const *hs, int32_t count, void *d_out, size_t out_bytes, lat_obs *out,
                              void *hip_stream)
{
    return guarded("lattice_observables_batch", [&]() -> int {
        if (count < 0 || (count > 0 && (!hs || !out || !d_out))) return fail(LAT_EINVAL, "bad batch");
        if (out_bytes < (size_t)count * 80u) return fail(LAT_ENOMEM, "output buffer smaller than 80 bytes per lattice");
        for (int32_t i = 0; i < count; ++i)
            if (!live(hs[i])) return fail(LAT_ESTATE, "null or destroyed handle in batch");
        hipStream_t stream = (hipStream_t)hip_stream;
        const int rc = enqueue_observables_batch(hs, count, (unsigned long long *)d_out, stream);
        if (rc) return rc;
        return read_records("lattice_observables_batch", d_out, 10, (size_t)count, hs, (size_t)count, false, stream,
                            [&](size_t at, const int64_t *v, size_t m) {
                                for (size_t i = 0; i < m; ++i) fill_obs(hs[at + i], v + 10 * i, &out[at + i]);
                            });
    });
}

int lattice_sweep_series(lattice *h, uint32_t intervals, uint32_t every, void *d_series, size_t series_bytes)
{
    return guarded("lattice_sweep_series", [&]() -> int {
        if (!live(h)) return fail(LAT_ESTATE, "null or destroyed handle");
        if (every == 0 || (intervals > 0 && !d_series)) return fail(LAT_EINVAL, "every must be > 0 and d_series set");
        if (series_bytes / kSeriesRecord < intervals)
            return fail(LAT_ENOMEM, "series buffer smaller than 88 bytes per interval");
        if (intervals == 0) return LAT_OK;
        lattice *one[1] = {h};
        hipStream_t st = h->stream;
        uint32_t *work = (uint32_t *)(h->d_scratch + kScrWork);
        // a packed int8 lattice stays on its 2-bit copy for the whole series
        if (h->packed) {
            const hipError_t e = launch_pack_int8((const int8_t *)h->d_state, work, h->L, st);
            if (e != hipSuccess) return hip_fail(e, "int8 pack launch");
        }
        // the whole series in persistent launches where they can run
        bool ran = false;
        const bool small = h->path == kPathLds, bytes = h->enc == LAT_ENC_INT8;
        // A series spread over the chip has a reduction more, but each of its records
        // costs less (L = 256, 20 intervals of one sweep 257 us and 500 on the chip, 1 of two
        // 50 and 60; L = 192, 4 of five 241 and 234).  Int8 lattices as they are take three
        // launches and a reduction an interval (L = 260, 4 of two 161 and 227; L = 208,
        // 4 of five 287 and 268), or launches per phase where that is one sweep.
        const bool wide = small && (bytes ? every > 1 && spreads(one, 1, every, 13000.0, st)
                                          : spreads(one, 1, (uint64_t)intervals * every, 10000.0 - 5000.0 * intervals, st));
        if (h->path == kPathWords || (wide && !bytes)) {
            const int rc = enqueue_words_persistent(one, 1, nullptr, intervals, every, (long long *)d_series, st,
                                                    /*bytes=*/false, &ran);
            if (rc) return rc;
        }
        if (small && !ran && !(wide && bytes)) {
            const ObsTarget obs{(unsigned long long *)d_series, intervals, kSeriesRecord / 8, kSeriesRecord / 8};
            const int rc = enqueue_lds_sweeps(one, 1, nullptr, every, st, &obs);
            if (rc) return rc;
            ran = true;
        }
        for (uint32_t k = 0; k < intervals && !ran; ++k) {
            const int rc = small ? enqueue_small_sweeps(one, 1, every, st)
                                 : enqueue_offchip_sweeps(one, 1, nullptr, every, st, /*convert=*/false);
            if (rc) return rc;
            long long *rec = (long long *)((uint8_t *)d_series + kSeriesRecord * (size_t)k);
            const hipError_t e = launch_observables(h->d_scratch, h->packed ? (const void *)work : h->d_state, h->L,
                                                    h->packed ? LAT_ENC_2BIT : h->enc, st, rec);
            if (e != hipSuccess) return hip_fail(e, "observables launch");
        }
        if (h->packed) {
            const hipError_t e = launch_unpack_int8(work, (int8_t *)h->d_state, h->L, st);
            if (e != hipSuccess) return hip_fail(e, "int8 unpack launch");
        }
        return LAT_OK;
    });
}

int lattice_series_read(lattice *h, const void *d_series, uint32_t intervals, lat_obs *out)
{
    return guarded("lattice_series_read", [&]() -> int {
        if (!live(h)) return fail(LAT_ESTATE, "null or destroyed handle");
        if (intervals > 0 && (!d_series || !out)) return fail(LAT_EINVAL, "null series or output");
        if (intervals == 0) return LAT_OK;
        lattice *one[1] = {h};
        return read_records("lattice_series_read", d_series, kSeriesRecord / 8, intervals, one, 1, true, h->stream,
                            [&](size_t at, const int64_t *v, size_t m) {
                                for (size_t k = at; k < at + m; ++k, v += kSeriesRecord / 8) {
                                    fill_obs(h, v, &out[k]);
                                    out[k].sweep = (uint64_t)v[10] - h->start_sweep;
                                }
                            });
    });
}

int lattice_observables(lattice *h, lat_obs *out)
{
    return guarded("lattice_observables", [&]() -> int {
        if (!live(h)) return fail(LAT_ESTATE, "null or destroyed handle");
        if (!out) return fail(LAT_EINVAL, "null output");
        // the reduction writes its record (tracker, 7 sums, next sweep) into
        // pinned memory where it can, else into the scratch, for a copy
        PinnedBlock stage;
        int64_t own[12];  // record, and the error flags after it
        int64_t *v = stage.p ? (int64_t *)stage.p : own;
        hipError_t e = launch_observables(h->d_scratch, h->d_state, h->L, h->enc, h->stream,
                                          stage.p ? (long long *)stage.p : nullptr);
        if (e == hipSuccess && !stage.p)
            e = hipMemcpyAsync(v, h->d_scratch + kScrTrack, 10 * sizeof(int64_t), hipMemcpyDeviceToHost, h->stream);
        v[11] = 0;
        if (e == hipSuccess && barrier_may_time_out(h))
            e = hipMemcpyAsync(&v[11], h->d_scratch + kScrErr, sizeof(uint32_t), hipMemcpyDeviceToHost, h->stream);
        const hipError_t waited = hipStreamSynchronize(h->stream);
        if (waited != hipSuccess) stage.abandon();
        if (e == hipSuccess) e = waited;
        if (e != hipSuccess) return hip_fail(e, "lattice_observables");
        if ((uint32_t)v[11] & 1u) return barrier_timed_out();
        fill_obs(h, v, out);
        return LAT_OK;
    });
}

int lattice_read_state(lattice *h, int8_t *host_codes)
{
    return guarded("lattice_read_state", [&]() -> int {
        if (!live(h)) return fail(LAT_ESTATE, "null or destroyed handle");
        if (!host_codes) return fail(LAT_EINVAL, "null output");
        // Through pinned memory where the state fits; else int8 codes go to the
        // caller's memory as they are, and packed ones through ordinary memory that
        // is not cleared first.  (Int8 codes to an array of the caller's, staged and
        // at once: L = 64 13 and 23 us, L = 1400 101 and 107; into memory that is new on
        // every call L = 320 33 and 74.)
        const size_t bytes = lattice_state_bytes(h->L, h->enc);
        const bool packed = h->enc == LAT_ENC_2BIT;
        std::unique_ptr<PinnedBlock> stage;
        if (bytes <= kPinnedLarge) stage = std::make_unique<PinnedBlock>(/*large=*/bytes > kPinnedBytes);
        std::unique_ptr<uint8_t[]> own;
        uint8_t *dev = stage ? (uint8_t *)stage->p : nullptr;
        if (!dev && packed) own.reset(dev = new uint8_t[bytes]);
        if (!dev) dev = (uint8_t *)host_codes;
        uint32_t err = 0;
        hipError_t e = hipMemcpyAsync(dev, h->d_state, bytes, hipMemcpyDeviceToHost, h->stream);
        if (e == hipSuccess && barrier_may_time_out(h))
            e = hipMemcpyAsync(&err, h->d_scratch + kScrErr, sizeof(err), hipMemcpyDeviceToHost, h->stream);
        const hipError_t waited = hipStreamSynchronize(h->stream);
        if (waited != hipSuccess && stage) stage->abandon();
        if (e == hipSuccess) e = waited;
        if (e != hipSuccess) return hip_fail(e, "lattice_read_state");
        if (err & 1u) return barrier_timed_out();
        if (packed)
            codes_from_words(h->L, (const uint32_t *)dev, host_codes);
        else if (dev != (uint8_t *)host_codes)
            std::memcpy(host_codes, dev, bytes);
        return LAT_OK;
    });
}

int lattice_destroy(lattice *h)
{
    return guarded("lattice_destroy", [&]() -> int {
        if (!live(h)) return fail(LAT_ESTATE, "null or destroyed handle");
        h->magic = 0;
        delete h;
        return LAT_OK;
    });
}

const char *lattice_last_error(void) { return g_err_fixed ? g_err_fixed : g_err.c_str(); }

}  // extern "C"
