// gfx950 multi-block phase kernels of the coupled-pair Metropolis sweep
// (arXiv:2301.11735, section 3.1 update, section 3.2 parallel form) for
// lattices of medium size, and the int8 <-> 2-bit class-layout conversion.
//
// A phase of a lattice with L = 512..2048 has only 2k..33k a-words: one
// thread per word (16 pairs each, as in the large-lattice phase kernel)
// leaves most of the chip idle and puts 16 dependent pair steps on the
// critical path.  Here Q lanes share a word (word_task.h), a lattice spreads
// over many blocks, and one launch can hold several lattices, each at its own
// sweep.  What bounds these sizes is the chain of a phase: the loads of words
// that other compute units wrote, two dependent table gathers, the stores,
// and the meeting of all blocks.  The schedule of a
// sweep is computed on the device from the lattice's seed and sweep index,
// so a series of launches does not depend on host state and can be
// replayed from a HIP graph.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_common.h"
#include "word_task.h"

namespace lat {
namespace {

// One phase of every lattice of a batch, a row or more of the grid for each.  What
// bounds it: its chain, since a launch waits for the one before and memory that
// another kernel wrote is beyond the caches.  The rounds of that chain are the
// arguments (one wait), the lattice's descriptor with the tables behind it, and
// the state, whose loads and draws are issued before the tables go to LDS.  Ten
// lattices of L = 512 or one: 7.5 us a launch with the tables loaded entry by
// entry ahead of the state and the block's lattice looked up among the arguments,
// 5.6 with all loads at once, 5.0 with a row of the grid for each lattice, 4.4
// with the launch shape in the arguments' first line and a wave's sums added
// without a barrier.  The waves go first where they share a compute unit with
// other kernels (the server runs batches of small lattices beside them): the
// last block of a launch is waited for (served burst of 40 requests 173 ms
// without and 147 with priority; all of it 180 -> 126).
template <int Q, int N>
__global__ void __launch_bounds__(kWordsPhaseMaxThreads) k_phase_words(WordsArgsOf<N> a)
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
    uint32_t *st = (uint32_t *)(d.enc == 1 ? d.state : (void *)(scr + kScrWork));
    // after the descriptor's loads, which would not be scalar behind it
    __builtin_amdgcn_s_setprio(3);
    const uint64_t s = d.next_sweep + a.iter;
    int r, mm[4], kk[4];
    device_schedule(d.L, d.key0, d.key1, s, r, mm, kk);
    WordPhase f;
    word_phase_setup(f, d.L, d.key0, d.key1, s, a.p, r, mm, kk);
    const uint32_t csz = (uint32_t)f.H * (uint32_t)f.W;
    const uint32_t task = block * threads + threadIdx.x;
    // tasks = Q * csz is a multiple of Q, so a word's lanes are all in or all
    // out; those that are out load the first word's lanes again
    const int q = (int)(task & (uint32_t)(Q - 1));
    const bool mine = task < (uint32_t)Q * csz;
    const uint32_t at = mine ? task : (uint32_t)q;
    const WordRefs<Q> refs = word_refs<Q>(f, at);
    const WordVals<Q> v = word_fetch<Q, false>(st, refs);
    u32x4 draws[kTaskCalls<Q>];
    word_draws<Q>(task_call0<Q>(f, at), q, s, a.p, d.key0, d.key1, draws);
    tables.store(s_tab, s_slots, threads);
    __syncthreads();

    int tr[3] = {0, 0, 0};
    if (mine) unpack_tracker(word_apply<Q, false, false>(st, f, refs, v, q, draws, s_tab, (const uint8_t *)s_slots, nullptr), tr);
    wave_reduce_add3(tr, (unsigned long long *)(scr + kScrSlots) + 3 * (size_t)block);
}

// Block sums of m (per thread: tracker moves 0-2, spin, staggered spin and
// staggered charge moves 3-5 of an interval): thread i < 6 gets sum i.  Below
// kNarrowSweeps sweeps an interval a wave's sums fit 32 bits.
constexpr uint32_t kNarrowSweeps = 16384;  // 64 lanes x 4 phases x 16 pairs x at most 16 a pair
__device__ __forceinline__ long long block_moves(const int (&m)[6], bool narrow)
{
    __shared__ long long part[16][6];
    const int wave = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
    if (narrow) {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int v = dpp_step_sum(m[i]);
            if ((threadIdx.x & 63u) == 0) part[wave][i] = v;
        }
    } else {
        long long v[6] = {m[0], m[1], m[2], m[3], m[4], m[5]};
        wave_partials<6, long long>(v, part);
    }
    __syncthreads();
    long long sum = 0;
    if (threadIdx.x < 6)
        for (int w = 0; w < nw; ++w) sum += part[w][threadIdx.x];
    return sum;  // the barrier after it comes before part is written again
}
// Adds sum i (of block_moves) to its fields of a record (tracker 0-2, sums
// 3-9): the tracker moves to the tracker and to the charged-site count and
// the two bond sums, the others to the last three sums.
__device__ __forceinline__ void add_to_record(unsigned long long *rec, int i, long long sum)
{
    if (sum == 0) return;
    if (i < 3) atomicAdd(&rec[i], (unsigned long long)sum);
    atomicAdd(&rec[i + 4], (unsigned long long)sum);
}

// Persistent form: the sweeps of a whole call of up to kWordsBatch lattices,
// or a whole observation series of one lattice, in one launch of blocks that
// are all resident at once (GridBarrier: assemble); blocks first_block[i] ..
// first_block[i+1]-1 update lattice i.  Tables are staged once; every phase
// is one grid-stride pass over each lattice's a-word tasks by its own blocks,
// followed by a device-wide barrier of those blocks (the lattices do not
// wait for each other, and one with fewer sweeps ends earlier).  Sweep it of
// the launch (interval k, sweep e of it: it = k every + e) is sweep
// next_sweep + it.  All lattice words are read and written at device coherence, so
// the barrier needs no cache write-back or invalidation (measured on MI355X
// with 128 blocks: 2.3 us a barrier, against 6.9 us with one release/acquire
// fence pair per block and 12-14 us with a fence pair in every wave).
//
// Obs (a series with records, one lattice): the records start as the
// lattice's state before the launch (k_series_begin: tracker total and the
// seven sums), and at the end of interval k the moves of all blocks since the
// launch began are added to record k: the tracker sums (to the tracker and to
// the charged-site count and the two bond sums, which change by exactly them)
// and the spin, staggered spin and staggered charge moves of the words they
// wrote.  With one counter every block adds its own; with two levels the
// blocks of a group add up first (32 blocks at an address instead of 256),
// and the thread that completes the group adds its sums to the record while
// the others wait at the barrier.  The lattice is not read for the records, so
// no barrier beyond the phases' is needed; they are whole when the launch ends.
template <int Q, bool Obs>
__global__ void __launch_bounds__(Q >= 4 ? kWordsSeriesMaxThreads : kWordsThreads) k_words_series(WordsSeriesArgs a)
{
    __shared__ uint2 s_tab[kDevTabEntries];
    __shared__ __align__(16) uint2 s_slots[kSlotEntries];
    int li = 0;  // this block's lattice (uniform)
    while (li + 1 < a.count && blockIdx.x >= a.first_block[li + 1]) ++li;
    uint8_t *scr = a.scratch[li];
    // ahead of the meeting: its atomics would make the descriptor's loads vector loads
    const LatDesc d = *(const LatDesc *)(scr + kScrDesc);
    uint32_t *st = (uint32_t *)(d.enc == 1 ? d.state : (void *)(scr + kScrWork));
    const uint32_t b = blockIdx.x - a.first_block[li], nb = a.first_block[li + 1] - a.first_block[li];
    GridBarrier barrier{(unsigned *)(scr + kScrObsSlots), b, nb, 0u, false};
    unsigned *err = (unsigned *)(scr + kScrErr);
    if (a.alone ? !barrier.alone() : !barrier.first_arrive(a.assemble_ticks)) return;
    {
        const uint2 *g_tab = (const uint2 *)(scr + kScrDevTab);
        for (int i = threadIdx.x; i < kDevTabEntries; i += blockDim.x) s_tab[i] = g_tab[i];
        const uint2 *g_slots = (const uint2 *)kWordSlots.v;
        for (int i = threadIdx.x; i < kSlotEntries; i += blockDim.x) s_slots[i] = g_slots[i];
    }
    __syncthreads();
    const uint32_t my_sweeps = a.sweeps[li];
    const uint32_t csz = (uint32_t)(d.L >> 1) * (uint32_t)(d.L >> 6);
    const uint32_t n_tasks = (uint32_t)Q * csz, stride = nb * blockDim.x;
    const uint32_t first = b * blockDim.x + threadIdx.x;
    // At most one task a thread (uniform per lattice): its Philox draws for the
    // next phase and the places of its words are made while the block waits
    // at the barrier, where they depend on nothing the other blocks write.
    const bool one = stride >= n_tasks, mine = one && first < n_tasks;
    const int q = (int)(first & (uint32_t)(Q - 1));
    u32x4 pre[kTaskCalls<Q>];
    WordRefs<Q> refs{};
    WordPhase f;
    int r, mm[4], kk[4];
    device_schedule(d.L, d.key0, d.key1, d.next_sweep, r, mm, kk);
    word_phase_setup(f, d.L, d.key0, d.key1, d.next_sweep, 0, r, mm, kk);
    const uint32_t c0 = task_call0<Q>(f, mine ? first : 0u);
    // (behind the first draws a series at L=1024 took 14.5 us a sweep, not 14.3)
    if (!barrier.assemble(a.alone, a.assemble_ticks)) return;
    barrier.rounds = 1u;
    if (mine && my_sweeps > 0) {
        word_draws<Q>(c0, q, d.next_sweep, 0, d.key0, d.key1, pre);
        refs = word_refs<Q>(f, first);
    }
    int tr[3] = {0, 0, 0};
    int dv[3] = {0, 0, 0};  // Obs: spin, staggered spin, staggered charge moves of the interval
    long long moves = 0;    // Obs, thread i < 6: the block's sum i of the intervals before
    // one interval of the lattice's own number of sweeps, or (with records)
    // intervals of `every` sweeps, which make up that number
    const uint32_t every = a.records ? a.every : my_sweeps;
    for (uint32_t k = 0; k < a.intervals; ++k) {
        for (uint32_t e = 0; e < every; ++e) {
            const uint32_t it = k * every + e;
            const uint64_t s = d.next_sweep + it;
            for (int p = 0; p < 4; ++p) {
                uint32_t packed = 0u;
                {
                    const uint8_t *slots = (const uint8_t *)s_slots;
                    if (one) {
                        if (mine) {
                            const WordVals<Q> v = word_fetch<Q, true>(st, refs);
                            packed = word_apply<Q, true, Obs>(st, f, refs, v, q, pre, s_tab, slots, dv);
                        }
                    } else {
                        // stride is a multiple of Q: a word's lanes are all in or all out
                        for (uint32_t t = first; t < n_tasks; t += stride) {
                            const WordRefs<Q> at = word_refs<Q>(f, t);
                            const WordVals<Q> v = word_fetch<Q, true>(st, at);
                            word_draws<Q>(task_call0<Q>(f, t), q, s, p, d.key0, d.key1, pre);
                            unpack_tracker(word_apply<Q, true, Obs>(st, f, at, v, q, pre, s_tab, slots, dv), tr);
                        }
                    }
                }
                if (Obs) unpack_tracker(packed, tr);
                unsigned long long *rec = nullptr;  // Obs: the record that this phase completes
                if constexpr (Obs) {
                    if (p == 3 && e + 1 == every) {
                        rec = (unsigned long long *)(a.records + (kSeriesRecord / 8) * (size_t)k);
                        const int m[6] = {tr[0], tr[1], tr[2], dv[0], dv[1], dv[2]};
                        const long long sum = block_moves(m, every <= kNarrowSweeps);
                        if (threadIdx.x < 6) {
                            moves += sum;
                            if (barrier.flat())
                                add_to_record(rec, (int)threadIdx.x, moves);
                            else if (sum != 0)
                                atomicAdd(barrier.sums() + threadIdx.x, (unsigned long long)sum);
                        }
#pragma unroll
                        for (int i = 0; i < 3; ++i) tr[i] = dv[i] = 0;
                        if (b == 0 && threadIdx.x == 0)
                            rec[10] = (unsigned long long)(d.next_sweep + (uint64_t)(k + 1) * every);
                    }
                }
                const bool last = barrier.arrive();
                if (Obs && rec && last) {
                    long long g[6];
#pragma unroll
                    for (int i = 0; i < 6; ++i)
                        g[i] = (long long)__hip_atomic_load(barrier.sums() + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int i = 0; i < 6; ++i) add_to_record(rec, i, g[i]);
                }
                // the next phase's schedule, draws and places, while the others arrive
                if (!Obs) unpack_tracker(packed, tr);
                const uint32_t it_next = p < 3 ? it : it + 1;
                const uint64_t s_next = p < 3 ? s : s + 1;
                if (p == 3) device_schedule(d.L, d.key0, d.key1, s_next, r, mm, kk);
                word_phase_setup(f, d.L, d.key0, d.key1, s_next, p < 3 ? p + 1 : 0, r, mm, kk);
                if (mine && it_next < my_sweeps) {
                    word_draws<Q>(c0, q, s_next, p < 3 ? p + 1 : 0, d.key0, d.key1, pre);
                    refs = word_refs<Q>(f, first);
                }
                barrier.wait(err, a.barrier_ticks);
            }
        }
    }
    if (Obs && threadIdx.x < 3) atomicAdd((unsigned long long *)(scr + kScrSlots) + 3 * (size_t)b + threadIdx.x, (unsigned long long)moves);
    block_reduce_add<3>(tr, (unsigned long long *)(scr + kScrSlots) + 3 * (size_t)b);
    // every block read the descriptor before its first phase's barrier
    if (b == 0 && threadIdx.x == 0 && my_sweeps > 0)
        ((LatDesc *)(scr + kScrDesc))->next_sweep = d.next_sweep + my_sweeps;
}

// Before a persistent launch: clears every lattice's barrier words, which live in
// its scratch, in the observable slots (they hold nothing between calls), and
// copies a series' first record, the state before it, to the others.
static_assert(kScrObsSlots % 128 == 0 && kBarrierWords * 4u <= (size_t)kMaxObsSlots * 56u, "barrier words");
constexpr uint32_t kBeginThreads = 256;
__global__ void __launch_bounds__(kBeginThreads) k_series_begin(WordsSeriesArgs a)
{
    if ((int)blockIdx.x < a.count) {
        unsigned *w = (unsigned *)(a.scratch[blockIdx.x] + kScrObsSlots);
        for (unsigned i = threadIdx.x; i < kBarrierWords; i += kBeginThreads) w[i] = 0u;
    }
    constexpr uint32_t kFields = kSeriesRecord / 8;
    const uint64_t n = a.records ? (uint64_t)kFields * a.intervals : 0u;
    for (uint64_t i = kFields + blockIdx.x * kBeginThreads + threadIdx.x; i < n; i += gridDim.x * kBeginThreads)
        a.records[i] = a.records[i % kFields];
}

template <int N>
__global__ void k_advance_words(WordsArgsOf<N> a)
{
    if (blockIdx.x == 0 && (int)threadIdx.x < a.count)
        ((LatDesc *)(a.scratch[threadIdx.x] + kScrDesc))->next_sweep += a.sweeps[threadIdx.x];
}

// Thread (y, j): the 64 int8 codes of row y starting at x = 64j, i.e. word j
// of class row y/2 of the four classes 4(y mod 2) + cx (site x = 4X + cx,
// X = 16j + t at bits 2t).  Byte cx of 32-bit word t of the 64 codes is
// site 4(16j + t) + cx.
__global__ void __launch_bounds__(256) k_pack_int8(const int8_t *__restrict__ src, uint32_t *__restrict__ dst,
                                                   int L)
{
    const uint32_t W = (uint32_t)L >> 6, H = (uint32_t)L >> 1, csz = H * W;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint32_t)L * W) return;
    const uint32_t y = i / W, j = i - y * W;
    const uint4 *row = (const uint4 *)(src + (size_t)y * L + 64u * j);
    uint32_t w[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint4 v = row[k];
        w[4 * k] = v.x;
        w[4 * k + 1] = v.y;
        w[4 * k + 2] = v.z;
        w[4 * k + 3] = v.w;
    }
    const uint32_t c0 = 4u * (y & 1u), Y = y >> 1;
#pragma unroll
    for (uint32_t cx = 0; cx < 4; ++cx) {
        uint32_t cw = 0;
#pragma unroll
        for (int t = 0; t < 16; ++t) cw |= ((w[t] >> (8u * cx)) & 3u) << (2 * t);
        dst[(c0 + cx) * csz + Y * W + j] = cw;
    }
}

__global__ void __launch_bounds__(256) k_unpack_int8(const uint32_t *__restrict__ src, int8_t *__restrict__ dst,
                                                     int L)
{
    const uint32_t W = (uint32_t)L >> 6, H = (uint32_t)L >> 1, csz = H * W;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint32_t)L * W) return;
    const uint32_t y = i / W, j = i - y * W;
    const uint32_t c0 = 4u * (y & 1u), Y = y >> 1;
    uint32_t cw[4];
#pragma unroll
    for (uint32_t cx = 0; cx < 4; ++cx) cw[cx] = src[(c0 + cx) * csz + Y * W + j];
    uint4 *row = (uint4 *)(dst + (size_t)y * L + 64u * j);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = 4 * k + u;
            v[u] = ((cw[0] >> (2 * t)) & 3u) | (((cw[1] >> (2 * t)) & 3u) << 8) | (((cw[2] >> (2 * t)) & 3u) << 16) |
                   (((cw[3] >> (2 * t)) & 3u) << 24);
        }
        row[k] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

}  // namespace

// Lanes per a-word of the per-phase form.  Up to L = 1024: 4.  The form's
// main user below that size is the server's second stream, whose launches
// hold several lattices beside the on-chip kernel's blocks; there 4 lanes
// beat 8 (a 60 s served run: p99 0.224 s against 0.253-0.257 s, L = 512
// requests 0.246 against 0.277-0.280 s; 2 lanes: 0.232-0.236 s).
int words_lanes(int L)
{
    if (L <= 1024) return 4;
    if (L <= 2048) return 2;
    return 1;
}

namespace {
template <int N>
void phase_words(const WordsArgsOf<N> &a, int Q, int threads, hipStream_t s)
{
    const dim3 grid(a.max_blocks, (unsigned)a.count), block((unsigned)threads);
    switch (Q) {
    case 1: hipLaunchKernelGGL((k_phase_words<1, N>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_phase_words<2, N>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_phase_words<4, N>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((k_phase_words<8, N>), grid, block, 0, s, a); break;
    }
}
}  // namespace

hipError_t launch_phase_words(const WordsArgs &a, int Q, int threads, hipStream_t s)
{
    if (Q == 0) return launch_phase_bytes(a, threads, s);
    with_rows(a, [&](const auto &rows) { phase_words(rows, Q, threads, s); });
    return hipGetLastError();
}

namespace {
template <int Q>
const void *series_fn(bool obs)
{
    return obs ? (const void *)k_words_series<Q, true> : (const void *)k_words_series<Q, false>;
}
const void *series_fn_of(int Q, bool obs)
{
    switch (Q) {
    case 0: return bytes_series_kernel();
    case 1: return series_fn<1>(obs);
    case 2: return series_fn<2>(obs);
    case 4: return series_fn<4>(obs);
    default: return series_fn<8>(obs);
    }
}
}  // namespace

int words_persistent_capacity(int Q, int threads)
{
    int dev = 0, per_cu = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) return 0;
    // the smaller of the two forms' (with and without records) resident blocks
    for (const bool obs : {false, true}) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, series_fn_of(Q, obs), threads, 0) != hipSuccess ||
            n < 1)
            return 0;
        per_cu = obs ? std::min(per_cu, n) : n;
    }
    return per_cu * cus;
}

hipError_t launch_words_series(const WordsSeriesArgs &a, int Q, hipStream_t s)
{
    const uint32_t fields = a.records ? a.intervals * (uint32_t)(kSeriesRecord / 8) : 0u;
    const uint32_t blocks = std::max((uint32_t)a.count, std::min(256u, (fields + kBeginThreads - 1) / kBeginThreads));
    hipLaunchKernelGGL(k_series_begin, dim3(blocks), dim3(kBeginThreads), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // An ordinary launch: the blocks find out themselves whether they are all
    // there.  A cooperative one promises no more than the capacity that the
    // caller has checked, and costs a switch of queues.
    WordsSeriesArgs args = a;
    void *kargs[] = {&args};
    const void *fn = series_fn_of(Q, a.records != nullptr);
    args.alone = 0;
    const hipError_t ran = hipLaunchKernel(fn, dim3(a.first_block[a.count]), dim3((unsigned)a.threads), kargs, 0, s);
    if (ran != hipSuccess) return ran;
    args.alone = 1;
    for (int i = 0; i <= a.count; ++i) args.first_block[i] = (uint32_t)i;
    return hipLaunchKernel(fn, dim3((unsigned)a.count), dim3((unsigned)a.threads), kargs, 0, s);
}

namespace {
template <int N>
void advance_words(const WordsArgsOf<N> &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_advance_words<N>, dim3(1), dim3(kWordsBatch), 0, s, a);
}
}  // namespace

hipError_t launch_advance_words(const WordsArgs &a, hipStream_t s)
{
    with_rows(a, [&](const auto &rows) { advance_words(rows, s); });
    return hipGetLastError();
}

hipError_t launch_pack_int8(const int8_t *src, uint32_t *dst, int L, hipStream_t s)
{
    const uint32_t n = (uint32_t)L * ((uint32_t)L >> 6);
    hipLaunchKernelGGL(k_pack_int8, dim3((n + 255) / 256), dim3(256), 0, s, src, dst, L);
    return hipGetLastError();
}

hipError_t launch_unpack_int8(const uint32_t *src, int8_t *dst, int L, hipStream_t s)
{
    const uint32_t n = (uint32_t)L * ((uint32_t)L >> 6);
    hipLaunchKernelGGL(k_unpack_int8, dim3((n + 255) / 256), dim3(256), 0, s, src, dst, L);
    return hipGetLastError();
}

}  // namespace lat
