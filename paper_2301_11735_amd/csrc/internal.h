// Library-internal declarations shared by the host sources (lattice_api.cpp,
// server.cpp).  Not part of the C-ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <exception>
#include <functional>
#include <new>
#include <string>

#include "../../include/lattice.h"
#include "kernels.h"

// How a lattice is swept (chosen at create from L and the encoding):
//   kPathLds    one block holds the whole lattice in LDS for all the sweeps of
//               a launch, or it is spread over many blocks where that is
//               faster (batch.hip, quad.hip); by default L <= 256 when
//               L % 64 == 0, else L <= 384;
//   kPathWords  many blocks per lattice, Q lanes per a-word, schedule
//               computed on the device (words.hip): one persistent launch
//               per call, or one launch per phase in graphs, in the server and
//               on other streams than the default one; L % 64 == 0, L <= 2048;
//   kPathPhase  one launch per phase (phase.hip): one thread per a-word, or two
//               pairs a thread for int8 lattices that are not packed;
//   kPathBytes  the latter for 384 < L <= 512, L % 64 != 0: batch graphs take
//               these sides and not those of kPathPhase, and many of them in one
//               call are swept as on kPathLds.
// Int8 lattices with L % 64 == 0 off the chip are swept on a 2-bit
// copy in their scratch (packed before the sweeps of a call, unpacked after).
enum : int { kPathLds = 0, kPathWords = 1, kPathPhase = 2, kPathBytes = 3 };

struct lattice {
    int L = 0, enc = 0;
    int64_t N = 0, Q = 0, Nc = 0;
    double n = 0, Delta = 0, V = 0, J = 0, T = 1;
    uint64_t seed = 0, start_sweep = 0, done = 0;
    void *d_state = nullptr;
    uint8_t *d_scratch = nullptr;
    hipStream_t stream = nullptr;
    lat::Tuning2Bit tuning{0, 0, 0, 0};
    int path = kPathLds;
    bool path_asked = false;  // by the environment
    bool packed = false;  // int8 swept on the 2-bit copy at scratch + kScrWork
    // set once a persistent launch has swept it, so that reads check the
    // device-wide barrier's time-out flag
    bool ran_persistent = false;
    uint32_t magic = 0;
};

namespace lat {
namespace detail {

int fail(int code, const std::string &msg);
int hip_fail(hipError_t e, const char *what);
// The error of every read of a lattice whose device-wide barrier timed out.
int barrier_timed_out();
// fail() for exception handlers: records "what: msg" without throwing (if
// even that string cannot be allocated, a fixed message is kept instead).
int fail_nothrow(int code, const char *what, const char *msg) noexcept;
bool live(const lattice *h);

// Runs the body of a C-ABI entry point so that no C++ exception crosses the
// ABI: host memory exhaustion (std::bad_alloc) becomes LAT_ENOMEM, anything
// else (a thread that cannot start, a container error) LAT_EHIP, each with a
// message for lattice_last_error().
template <class F>
int guarded(const char *what, F &&body) noexcept
{
    try {
        return body();
    } catch (const std::bad_alloc &) {
        return fail_nothrow(LAT_ENOMEM, what, "out of host memory");
    } catch (const std::exception &e) {
        return fail_nothrow(LAT_EHIP, what, e.what());
    } catch (...) {
        return fail_nothrow(LAT_EHIP, what, "unknown exception");
    }
}
// A pinned, device-visible block of host memory for one call's transfers
// (kernels may write results into it): kPinnedBytes for small ones (pageable
// copies of a few hundred bytes cost 5-10 us more each), or kPinnedLarge.  Taken
// from a pool of the process and given back by the destructor; the pool keeps at
// most kPinnedKeep small and kPinnedLargeKeep large blocks, others are freed.  The
// holder gives a block back only after it has waited for the device work that
// uses it; abandon() drops a block whose work may still run (a failed wait).  p is
// null when no pinned memory can be had: callers then use ordinary memory and
// copies.
constexpr size_t kPinnedBytes = 24576, kPinnedLarge = 2u << 20;
constexpr size_t kPinnedKeep = 8, kPinnedLargeKeep = 2;
class PinnedBlock {
  public:
    explicit PinnedBlock(bool large = false);
    ~PinnedBlock();
    PinnedBlock(const PinnedBlock &) = delete;
    PinnedBlock &operator=(const PinnedBlock &) = delete;
    void *p = nullptr;
    void abandon() { p = nullptr; }

  private:
    const bool large_;
};

// Advance lattices resident in LDS; lattice i by sweeps[i] (null: `uniform`).
// obs non-null: `intervals` times over, each
// time followed by the lattices' observables in obs->dev (obs->words int64 a
// lattice as enqueue_observables_batch, obs->stride int64 from one interval to
// the next), written from LDS by the sweep launch where its form does that.
struct ObsTarget {
    unsigned long long *dev;
    uint32_t intervals;
    uint32_t words;   // 10, or 11 with the next sweep index appended (series records)
    uint32_t stride;
};
int enqueue_lds_sweeps(lattice *const *hs, int32_t count, const uint32_t *sweeps, uint32_t uniform,
                       hipStream_t stream, const ObsTarget *obs = nullptr);
// One batched observables launch per 256 lattices into dev (10 int64 each).
int enqueue_observables_batch(lattice *const *hs, int32_t count, unsigned long long *dev, hipStream_t stream);
// Lattices on the off-chip paths (words, phase): lattice i by sweeps[i]
// (null: `uniform`); int8 ones are packed before and unpacked after.
// convert = false: packed lattices are already on (and stay on) their copy.
// persistent = false: the multi-block lattices take one launch per phase,
// never the persistent launch, whose blocks must all be resident
// at once (callers whose other streams run kernels at the same time, like
// the server, would otherwise leave it waiting for compute units).
int enqueue_offchip_sweeps(lattice *const *hs, int32_t count, const uint32_t *sweeps, uint32_t uniform,
                           hipStream_t stream, bool convert = true, bool persistent = true);
// Lattices as persistent multi-block launches (bytes: int8 ones as they are, at
// multiples of four bytes, without records; else on their two-bit state): lattice i by
// sweeps[i] (null: `every`) with intervals = 1 and no records, or, with
// records, an observation series of one lattice: intervals x every sweeps, a
// kSeriesRecord record after each interval.  *ran = false (nothing
// enqueued) when the persistent form is off (LATTICE_WORDS_PERSISTENT=0, a
// stream other than the default one) or cannot be launched here; the
// caller then uses the per-phase launches.  Packed int8 lattices must
// already be on their 2-bit copy.
int enqueue_words_persistent(lattice *const *hs, int32_t count, const uint32_t *sweeps, uint32_t intervals,
                             uint32_t every, long long *records, hipStream_t stream, bool bytes, bool *ran);
// Checks of lat_params (geometry, finite couplings, T > 0, the charge target
// of eq. 2); writes the target charge and the charged count.
int validate_params(const lat_params *p, int64_t *Q, int64_t *Nc);
// The lattice has run a persistent kernel, whose bounded device-wide barrier
// flags a time-out in its error word.
bool barrier_may_time_out(const lattice *h);
// Waits for the stream and hands the n records (`words` int64 each) at dev to
// fill(first, records, m) in order, m at once.  Also reads the error
// flags of those of the `count` lattices hs that ran a device-wide barrier
// (always: of all of them): a time-out is an error.  what: the entry point's name.
int read_records(const char *what, const void *dev, uint32_t words, size_t n, lattice *const *hs, size_t count,
                 bool always, hipStream_t stream, const std::function<void(size_t, const int64_t *, size_t)> &fill);
// v = (tracker nD, nV, nJ, sum S, sum S^2, bonds SS, bonds ss, M, M_st, C_st).
void fill_obs(const lattice *h, const int64_t *v, lat_obs *out);

}  // namespace detail
}  // namespace lat
