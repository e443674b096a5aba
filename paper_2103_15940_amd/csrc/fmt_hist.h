// Device-side pieces of the per-tensor statistics (Sec. V), shared by the stream kernels and the
// Linear-layer epilogue: the replicated exponent table in LDS, the per-lane class counters, and
// the fold of a workgroup's table into one of the partial records in global memory.
#pragma once

#include "fmt_internal.h"

namespace fmt {

constexpr int kHistRows = 256 + 24;      // exponent fields 0..255, then the 23 binades of fp32 denormals
constexpr int kSlots = 72;               // uint64 per partial record (8 class slots + 64 bins)
constexpr int kShards = 64;              // partial records in global memory (workgroup b adds into b % 64)
// slots of a partial record
enum { P_Z = 0, P_ZU, P_ZUD, P_TOP, P_INFNAN, P_NAN, P_BINS = 8 };

// Library scratch of a stream's statistics, in words of 8 bytes: kShards records for passes that are summed by a second kernel;
// for the passes of one launch, which take two sets in turn (see hist_clear), two sets of one record for launches of
// at most kFew workgroups, and two of kShards records and one of their sums for the others; and, where the stream has
// rounded groups of matrices, one set per matrix of a group (cleared by the group's first launch).
constexpr int kFew = 64;
constexpr int kSetWords = (kShards + 1) * kSlots;
constexpr size_t kHistScratchBytes = (size_t)(kShards * kSlots + 2 * kSlots + 2 * kSetWords) * sizeof(unsigned long long);

struct Counts {                          // per-lane counters, reduced once at the end
    uint32_t z = 0, zu = 0, zud = 0, top = 0, infnan = 0, nan = 0;
};

// Statistics of one element (a = pattern of |x|): one LDS increment and four compare-and-count
// steps (six when the wave holds an overflowing or non-finite element).  COPIES replicas of the
// table, lane l uses replica l % COPIES (with 32 replicas no two lanes share a bank).
template <bool DEEP, int COPIES>
__device__ __forceinline__ void account(uint32_t a, bool valid, const QuantParams &p, uint32_t *tbl, uint32_t copy,
                                        Counts &w)
{
    uint32_t row = a >> 23;
    if (DEEP) {
        // fp32-denormal inputs get a row per binade so that windows reaching below 2^-126 stay exact
        if (a - 1u < 0x007FFFFFu) row = 256u + (31u - (uint32_t)__builtin_clz(a));
    }
    if (valid) __hip_atomic_fetch_add(&tbl[row * COPIES + copy], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    w.z += (valid && a == 0u) ? 1u : 0u;
    w.zu += (valid && a <= p.t_zero) ? 1u : 0u;
    w.zud += (valid && a < p.t_den) ? 1u : 0u;
    const bool top = valid && a >= p.t_ovf;
    if (__ballot(top)) {                 // wave-uniform: rare for real tensors
        w.top += top ? 1u : 0u;
        w.infnan += (valid && a >= 0x7F800000u) ? 1u : 0u;
        w.nan += (valid && a > 0x7F800000u) ? 1u : 0u;
    }
}

// The same statistics for a run of elements that are all valid, in two parts.  account_run does the
// table increment and the three counters every element needs, and keeps the largest pattern seen in
// amax; after the run, account_run_top looks at amax once and recounts the run's elements for the
// overflow / infinity / NaN counters only if one of them can be non-zero anywhere in the wave.
template <bool DEEP, int COPIES>
__device__ __forceinline__ void account_run(uint32_t a, const QuantParams &p, uint32_t *tbl, uint32_t copy, Counts &w,
                                            uint32_t &amax)
{
    uint32_t row = a >> 23;
    if (DEEP) {
        if (a - 1u < 0x007FFFFFu) row = 256u + (31u - (uint32_t)__builtin_clz(a));
    }
    __hip_atomic_fetch_add(&tbl[row * COPIES + copy], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    w.z += a == 0u ? 1u : 0u;
    w.zu += a <= p.t_zero ? 1u : 0u;
    w.zud += a < p.t_den ? 1u : 0u;
    amax = a > amax ? a : amax;
}

template <int N>
__device__ __forceinline__ void account_run_top(const uint32_t (&u)[N], uint32_t amax, const QuantParams &p, Counts &w)
{
    if (__ballot(amax >= p.t_ovf)) {     // wave-uniform: rare for real tensors
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint32_t a = u[j] & 0x7FFFFFFFu;
            w.top += a >= p.t_ovf ? 1u : 0u;
            w.infnan += a >= 0x7F800000u ? 1u : 0u;
            w.nan += a > 0x7F800000u ? 1u : 0u;
        }
    }
}

// Statistics of one element below t_ovf, in the lanes that call it; not `valid`: it does not count.
template <int COPIES>
__device__ __forceinline__ void account_below(uint32_t a, bool valid, const QuantParams &p, uint32_t *tbl, uint32_t copy, Counts &w)
{
    __hip_atomic_fetch_add(&tbl[(a >> 23) * COPIES + copy], valid ? 1u : 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    a = valid ? a : 0xFFFFFFFFu;
    w.z += a == 0u ? 1u : 0u;
    w.zu += a <= p.t_zero ? 1u : 0u;
    w.zud += a < p.t_den ? 1u : 0u;
}

// Zeroes the table and the two small arrays; ends with a barrier.  tbl must be 16-byte aligned.
template <int COPIES, int BLOCK>
__device__ __forceinline__ void hist_begin(uint32_t *tbl, uint32_t *s_bins, uint32_t *s_cls, uint32_t tid)
{
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    for (int i = tid; i < kHistRows * COPIES / 4; i += BLOCK) reinterpret_cast<v4 *>(tbl)[i] = v4{0u, 0u, 0u, 0u};
    if (tid < FMT_NBINS) s_bins[tid] = 0;
    if (tid < 8) s_cls[tid] = 0;
    __syncthreads();
}

// Where a launch's counts go.
//   records only (hist == nullptr)   every workgroup adds into record (workgroup % shards); a kernel that follows
//                                    sums and clears the records (launch_hist_finalize)
//   one workgroup (records == nullptr)  it writes the caller's record itself
//   in one launch (otherwise)        as records only, and whoever adds last to a slot passes its sum on (see hist_end)
struct HistSink {
    unsigned long long *records;         // all zero between launches; the sums of the records go to record `shards`
    unsigned long long *hist;            // the caller's fmt_hist_t
    unsigned long long n;                // elements of the tensor
    uint32_t shards;                     // records in use
    uint32_t nclear;
    unsigned long long *clear;           // nclear words to set to zero meanwhile (hist_clear)
};

// Clears the set of records that the next pass on the stream takes.  A completed pass leaves its records zero by itself; passes
// that overlap on the same records (which the header forbids: replays of two graphs recorded on one stream, say) leave
// counts and arrivals behind that no later arrival would ever put right.  So passes take two sets in turn, each clearing the
// other's: what is left behind spoils at most the first pass that meets it.  At most one store per thread (37 KB cleared by
// three workgroups cost 0.4 us of 5.3: hence the small sets), called ahead of hist_end, whose additions take longer than the
// stores (ahead of the first tile's work it cost 0.2 us: 2^24 elements, statistics alone, 13.5 -> 13.7).  All BLOCK threads call it.
template <int BLOCK>
__device__ __forceinline__ void hist_clear(const HistSink &sink, uint32_t wg, uint32_t nwg, uint32_t tid)
{
    for (uint32_t i = wg * BLOCK + tid; i < sink.nclear; i += nwg * BLOCK)
        __hip_atomic_store(&sink.clear[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Slot `slot` of the caller's record from the 72 summed counts and the number of elements.
__device__ __forceinline__ unsigned long long hist_slot(const unsigned long long *tot, unsigned long long n, int slot)
{
    const unsigned long long z = tot[P_Z], zu = tot[P_ZU], zud = tot[P_ZUD], top = tot[P_TOP], infnan = tot[P_INFNAN],
                             nan = tot[P_NAN];
    switch (slot) {
        case 0: return n;                    // total
        case 1: return z;                    // zero
        case 2: return zu - z;               // underflow
        case 3: return zud - zu;             // denormal
        case 4: return n - zud - top;        // normal
        case 5: return top - infnan;         // overflow
        case 6: return infnan - nan;         // inf
        case 7: return nan;                  // nan
        default: return tot[slot];           // bins
    }
}

// Folds the workgroup's counters and table into 64 bins and hands the 72 counts to the sink: one 64-bit atomic per
// slot into a record, or (one workgroup) the caller's record itself.  All BLOCK threads call it.
//
// In one launch: the separate summing kernel costs a launch (3 us of host time, 3 - 4 us and a gap on the GPU: a third
// of a pass over 2^20 elements).  Here every slot is independent of the others: its word holds a count (bits 0 .. 47)
// and how many workgroups have added to it (bits 48 ..), both in one addition, so the lane whose addition returns
// the last number but one holds the slot's sum, clears the word for the next launch and passes the sum on -- to the
// sum of the records, in the same way, and from there to the caller's record.  Two additions that return, one after
// the other, are all a launch waits for (an arrival counter behind a wait for the additions, and exchanges that
// fetch the sums, are four such hops and cost as much as the summing kernel); device-scope atomics take effect where
// all XCDs meet, so no cache has to be written back.
template <int COPIES, int BLOCK>
__device__ __forceinline__ void hist_end(uint32_t *tbl, uint32_t *s_bins, uint32_t *s_cls, const Counts &w,
                                         const QuantParams &p, const HistSink &sink, uint32_t wg, uint32_t nwg, uint32_t tid)
{
    uint32_t c[6] = {w.z, w.zu, w.zud, w.top, w.infnan, w.nan};
#pragma unroll
    for (int q = 0; q < 6; ++q) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) c[q] += __shfl_xor(c[q], off, 64);
    }
    if ((tid & 63) == 0) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
            if (c[q]) atomicAdd(&s_cls[q], c[q]);
    }
    __syncthreads();
    for (int row = tid; row < kHistRows; row += BLOCK) {
        uint32_t sum = 0;
#pragma unroll 8
        for (int k = 0; k < COPIES; ++k) sum += tbl[row * COPIES + ((k + row) & (COPIES - 1))];
        int E;
        if (row < 256) {
            E = row - 127;
            if (row == 0) sum -= s_cls[P_Z];      // zeros are not binned; what is left are fp32 denormals
            if (row == 255) { sum -= s_cls[P_NAN]; E = 1 << 20; }   // infinities -> top bin, NaN not binned
        } else {
            E = row - 256 - 149;                  // binade of an fp32 denormal with leading bit row-256
        }
        int b = E - p.exp_lo;
        b = b < 0 ? 0 : (b > FMT_NBINS - 1 ? FMT_NBINS - 1 : b);
        if (sum) atomicAdd(&s_bins[b], sum);
    }
    __syncthreads();
    if (tid >= kSlots) return;
    if (sink.hist == nullptr) {
        const uint32_t v = tid < 8 ? s_cls[tid] : s_bins[tid - 8];
        if (v) atomicAdd(&sink.records[(size_t)(wg % sink.shards) * kSlots + tid], (unsigned long long)v);
        return;
    }
    // this slot's share of the workgroup: the classes are differences of the counters; `normal` counts what it is not
    uint32_t v = 0u;
    switch (tid) {
        case 0: break;                                                    // total: known
        case 1: v = s_cls[P_Z]; break;                                    // zero
        case 2: v = s_cls[P_ZU] - s_cls[P_Z]; break;                      // underflow
        case 3: v = s_cls[P_ZUD] - s_cls[P_ZU]; break;                    // denormal
        case 4: v = s_cls[P_ZUD] + s_cls[P_TOP]; break;                   // everything but normal
        case 5: v = s_cls[P_TOP] - s_cls[P_INFNAN]; break;                // overflow
        case 6: v = s_cls[P_INFNAN] - s_cls[P_NAN]; break;                // inf
        case 7: v = s_cls[P_NAN]; break;                                  // nan
        default: v = s_bins[tid - 8]; break;
    }
    unsigned long long sum = v;
    if (sink.records != nullptr) {
        constexpr unsigned long long kOne = 1ull << 48;
        auto pass = [&](uint32_t record, uint32_t adders) __attribute__((always_inline)) {
            unsigned long long *word = &sink.records[(size_t)record * kSlots + tid];
            const unsigned long long had = __hip_atomic_fetch_add(word, sum | kOne, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sum += had & (kOne - 1ull);
            if ((had >> 48) + 1ull != adders) return false;
            __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        };
        const uint32_t shard = wg % sink.shards, mine = nwg / sink.shards + (shard < nwg % sink.shards ? 1u : 0u);
        if (!pass(shard, mine)) return;
        if (sink.shards > 1u && !pass(sink.shards, nwg < sink.shards ? nwg : sink.shards)) return;
    }
    sink.hist[tid] = tid == 0 ? sink.n : tid == 4 ? sink.n - sum : sum;
}

// Sums the partial records into the caller's fmt_hist_t and clears them (fmt_stream.hip).
int launch_hist_finalize(unsigned long long *partials, size_t n, fmt_hist_t *hist, hipStream_t stream);

// The sink of a launch of nwg workgroups whose counts end in `hist` (n elements, below 2^48): one workgroup writes the
// record itself (no records needed); fewer than 2^21 (a record counts its additions in 16 bits) finish in the launch, at any
// size (stream passes, one launch against two: 2^20 elements 6.4 us against 8.7, 2^25 46.7 against 50.0, 2^28 alike; a layer's
// output pass of 4098 workgroups: 2 us less); more leave their records to launch_hist_finalize (then sink.hist is null),
// as do passes whose records nobody clears ahead (at.clear null: captured ones, and fmt_quantize_static).
// Records in use: additions to one address take about 12 ns each, so up to kFew workgroups share one record and
// one hop; beyond that the additions are spread and a second hop sums the records.
inline HistSink hist_sink(const HistRecords &at, unsigned long long n, fmt_hist_t *hist, uint64_t nwg)
{
    unsigned long long *out = reinterpret_cast<unsigned long long *>(hist);
    if (nwg == 1) return HistSink{nullptr, out, n, 1u, 0u, nullptr};
    if (at.clear != nullptr && nwg < ((uint64_t)1 << 21))
        return HistSink{at.records, out, n, nwg <= kFew ? 1u : nwg <= 1024 ? 16u : (uint32_t)kShards, at.nclear, at.clear};
    return HistSink{at.records, nullptr, n, (uint32_t)kShards, at.nclear, at.clear};
}

}  // namespace fmt
