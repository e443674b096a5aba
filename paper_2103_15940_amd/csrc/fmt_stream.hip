// Stream kernels of libfmt: the rounding kernel of Sec. IV-A (fp32 -> 1/e/m, result kept as
// fp32) and the per-tensor statistics of Sec. V, separately or fused in one pass over x.
//
// Both are HBM streams: 4 B read (+ 4 B written) per element, 128-bit non-temporal accesses.
// A workgroup walks over tiles of 16 KiB of consecutive input (tile b, b+grid, ...): contiguous
// tiles handed out in launch order measured faster on MI355X than a thread-granular grid stride.  The rounding works on the fp32 bit pattern:
//   * e < 8: the format's grid around |x| has spacing 2^(max(E,Emin)-m), E = floor(log2|x|), and
//     (|x| + C) - C with C = 2^(max(E,Emin)+23-m) lands on it with the hardware's own RNE --
//     exact, since the addition is one correctly rounded fp32 operation whose ulp is that
//     spacing and the subtraction is exact.  C comes from the exponent field of |x| with two
//     integer operations.  fp32-denormal inputs are far below minD/2 there, so a flush of
//     them could only give the same zero;
//   * e = 8: fp32's own denormal grid is the format's, so round-to-nearest-even is done on the
//     integer pattern (add "half minus one plus the last kept bit", clear the dropped bits; a
//     mantissa carry walks into the exponent by itself), fp32-denormal inputs included;
//   * overflow, zero and flush decisions are comparisons of |x|'s pattern with thresholds
//     computed on the host (the ties at minD/2, minN - minD/2 and maxN + ulp/2 all go to the
//     even neighbour).
// Statistics: each element adds one to an LDS table indexed by its 8-bit fp32 exponent field, replicated 8, 16 or 32 times
// (lane l uses replica l modulo that number); the class counts are per-lane compare-and-add counters.  Each workgroup folds its
// table into 64 bins and adds its 72 counts, with one 64-bit atomic per slot, into one of a few partial records in library
// scratch; the workgroup that adds last to a slot passes the sum on to the caller's fmt_hist_t (hist_end), so a pass is one
// launch.  fmt_quantize_static, whose records are shared by all streams, and passes recorded into a graph, whose records
// are the same at every replay, sum them in a second kernel.
#include <mutex>

#include "fmt_hist.h"
#include "fmt_internal.h"
#include "fmt_quant.h"

#ifndef FMT_STREAM_BLOCK
#define FMT_STREAM_BLOCK 256
#endif
#ifndef FMT_STREAM_UNROLL
#define FMT_STREAM_UNROLL 4
#endif
#ifndef FMT_STREAM_GRID_PER_CU
#define FMT_STREAM_GRID_PER_CU 16
#endif

namespace fmt {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kBlock = FMT_STREAM_BLOCK;  // threads per workgroup
// Replicas of the exponent table in LDS, lane l uses replica l % copies.  8: 9 KiB, so that registers and not LDS bound the
// resident workgroups, and little to clear and fold in a pass of one tile per workgroup (2^20 elements 6.4 us fused against 7.2
// with 32, one per bank; 2^24 24.8 against 25.9; codes 2^26 70.5 against 76.5, 16 alike).  The fused fp32 pass over the largest
// tensors, whose workgroups hold four tiles and more, is the faster with 32: 2^28 elements 351 against 355 us (2^26: alike).
// Statistics alone, with nothing to write beside them, show the lanes that meet on one address where all values are alike: 16
// from 2^26 elements up (all ones / normal: 2^26 44.4 / 42.9 us, with 8 45.4 / 43.8; 2^27 83.2 / 81.7, with 8 88.9 / 84.7; 2^28 160 /
// 158, with 8 167 / 162); below that ordinary values are up to 4 % faster with 8 (2^22 7.7 against 8.1; 2^25 22.3 against 22.8).
constexpr int kCopiesMost = 8;
constexpr int kCopiesAlone = 16;
constexpr int kCopiesLarge = 32;
constexpr size_t kAlone = (size_t)1 << 26;   // elements from which statistics alone take theirs,
constexpr size_t kLarge = (size_t)1 << 27;   // ... and the fused fp32 pass its
constexpr int kUnroll = FMT_STREAM_UNROLL;  // independent 128-bit loads in flight per thread
constexpr int kGridPerCU = FMT_STREAM_GRID_PER_CU;   // workgroups launched per compute unit (at most): statistics alone
constexpr int kGridFused = 64;           // ... fused with rounding, fp32 or codes out
constexpr int kGridStore = 256;          // ... quantize only

template <int MODE, bool STORE, bool FTZ, bool HIST, bool DEEP, int kCopies>
__device__ __forceinline__ u32x4 do_vec(u32x4 v, bool valid, const QuantParams &p, uint32_t *tbl, uint32_t lane32,
                                        Counts &w)
{
    u32x4 o = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t u = v[j];
        if (HIST) account<DEEP, kCopies>(u & 0x7FFFFFFFu, valid, p, tbl, lane32, w);
        if (STORE) o[j] = quantize_bits<MODE, FTZ>(u, p);
    }
    return o;
}

// x, y: element pointers.  The vector body covers elements [head, head + 4*nvec) and needs
// x + head (and y + head when STORE) 16-byte aligned; the at most 6 remaining elements at both
// ends are handled one per lane by the first wave of workgroup 0.  VEC = false is the fallback
// for x and y misaligned relative to each other: the whole range goes one dword per lane.
// PACK: y holds the format's 16-bit codes instead of fp32 values (two bytes written per element; the
// vector body then needs y + head 8-byte aligned).
template <int MODE, bool STORE, bool FTZ, bool HIST, bool DEEP, bool VEC, bool PACK, int kCopies>
__global__ __launch_bounds__(kBlock) void stream_kernel(const uint32_t *__restrict__ x, uint32_t *__restrict__ y,
                                                        size_t n, size_t head, size_t nvec, QuantParams p, HistSink sink)
{
    constexpr int EM = MODE == kModeInteger ? kModeInteger : kModeMagic;   // encode_bits' variant
    uint16_t *__restrict__ y16 = reinterpret_cast<uint16_t *>(y);
    auto put = [&](size_t vec_index, u32x4 o) {
        if (PACK) {
            u32x2 c;
            c[0] = encode_bits<EM>(o[0], p) | (encode_bits<EM>(o[1], p) << 16);
            c[1] = encode_bits<EM>(o[2], p) | (encode_bits<EM>(o[3], p) << 16);
            __builtin_nontemporal_store(c, reinterpret_cast<u32x2 *>(y16 + head) + vec_index);
        } else {
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4 *>(y + head) + vec_index);
        }
    };
    auto put_one = [&](size_t idx, uint32_t r) {
        if (PACK)
            y16[idx] = (uint16_t)encode_bits<EM>(r, p);
        else
            y[idx] = r;
    };
    __shared__ __attribute__((aligned(16))) uint32_t tbl[HIST ? kHistRows * kCopies : 4];
    __shared__ uint32_t s_bins[FMT_NBINS];
    __shared__ uint32_t s_cls[8];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane32 = tid & (kCopies - 1);
    Counts w;

    constexpr size_t kTileVec = (size_t)kBlock * kUnroll;
    // VEC: a tile is kBlock*kUnroll consecutive vectors; workgroup b takes tiles b, b+grid, ...  Every lane of the workgroup
    // runs the same trips, and all tiles but the last are full.
    if constexpr (VEC && (HIST || PACK)) {
        // leftovers around the vector body, [0, head) and [head + 4*nvec, n): one per lane of the first wave, loaded before
        // anything else so that the load is not a chain of its own at the end
        const bool edge = blockIdx.x == 0 && tid < 64 && tid < n - 4 * nvec;
        const size_t edge_at = tid < head ? tid : 4 * nvec + tid;
        uint32_t edge_u = 0u;
        if (edge) edge_u = x[edge_at];

        const u32x4 *xv = reinterpret_cast<const u32x4 *>(x + head);
        const size_t full_tiles = nvec / kTileVec;
        u32x4 v[kUnroll];
        auto load = [&](size_t t) __attribute__((always_inline)) {
            const size_t i = t * kTileVec + tid;
            if (t < full_tiles) {
#pragma unroll
                for (int k = 0; k < kUnroll; ++k) v[k] = __builtin_nontemporal_load(xv + i + k * kBlock);
            } else {
#pragma unroll
                for (int k = 0; k < kUnroll; ++k) {
                    v[k] = u32x4{0u, 0u, 0u, 0u};
                    if (i + k * kBlock < nvec) v[k] = __builtin_nontemporal_load(xv + i + k * kBlock);
                }
            }
        };
        // With statistics a tile's loads are issued ahead of the work on the tile before it, the first tile's ahead of the clearing
        // of the table (2^25 elements: statistics alone 27.3 -> 22.4 us, fused 50 -> 47).
        size_t t = blockIdx.x;
        if (HIST) {
            load(t);
            hist_begin<kCopies, kBlock>(tbl, s_bins, s_cls, tid);
        }
        while (t < full_tiles) {
            if (!HIST) load(t);
            const size_t i = t * kTileVec + tid;
            uint32_t amax = 0u;
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                u32x4 o = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t u = v[k][j];
                    if (HIST) account_run<DEEP, kCopies>(u & 0x7FFFFFFFu, p, tbl, lane32, w, amax);
                    if (STORE) o[j] = quantize_bits<MODE, FTZ>(u, p);
                }
                if (STORE) put(i + k * kBlock, o);
            }
            if (HIST) {
                uint32_t flat[4 * kUnroll];
#pragma unroll
                for (int k = 0; k < kUnroll; ++k)
#pragma unroll
                    for (int j = 0; j < 4; ++j) flat[4 * k + j] = v[k][j];
                account_run_top(flat, amax, p, w);
            }
            t += gridDim.x;
            if (HIST && t * kTileVec < nvec) load(t);
        }
        if (t == full_tiles && full_tiles * kTileVec < nvec) {
            // the ragged last tile, lane by lane
            if (!HIST) load(t);
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                const size_t i = full_tiles * kTileVec + k * kBlock + tid;
                const bool valid = i < nvec;
                u32x4 o = do_vec<MODE, STORE, FTZ, HIST, DEEP, kCopies>(v[k], valid, p, tbl, lane32, w);
                if (STORE && valid) put(i, o);
            }
        }
        if (blockIdx.x == 0 && tid < 64) {
            if (HIST) account<DEEP, kCopies>(edge_u & 0x7FFFFFFFu, edge, p, tbl, lane32, w);
            if (STORE && edge) put_one(edge_at, quantize_bits<MODE, FTZ>(edge_u, p));
        }
    } else if constexpr (VEC) {
        // Values without statistics: a workgroup has one tile, and what counts is a short kernel (2^23 elements: 11.1 us; 11.5 with
        // the other branch's loop and leftovers, where codes without statistics are the faster ones: 2^24 16.8 against 17.2).
        const u32x4 *xv = reinterpret_cast<const u32x4 *>(x + head);
        const size_t full_tiles = nvec / kTileVec;
        u32x4 v[kUnroll];
        size_t t = blockIdx.x;
        for (; t < full_tiles; t += gridDim.x) {
            const size_t i = t * kTileVec + tid;
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) v[k] = __builtin_nontemporal_load(xv + i + k * kBlock);
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                u32x4 o = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = quantize_bits<MODE, FTZ>(v[k][j], p);
                put(i + k * kBlock, o);
            }
        }
        if (t == full_tiles && full_tiles * kTileVec < nvec) {
            const size_t i = full_tiles * kTileVec + tid;
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                v[k] = u32x4{0u, 0u, 0u, 0u};
                if (i + k * kBlock < nvec) v[k] = __builtin_nontemporal_load(xv + i + k * kBlock);
            }
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                u32x4 o = do_vec<MODE, STORE, FTZ, HIST, DEEP, kCopies>(v[k], i + k * kBlock < nvec, p, tbl, lane32, w);
                if (i + k * kBlock < nvec) put(i + k * kBlock, o);
            }
        }
        if (blockIdx.x == 0 && tid < 64 && tid < n - 4 * nvec) {
            const size_t at = tid < head ? tid : 4 * nvec + tid;
            const uint32_t u = x[at];
            put_one(at, quantize_bits<MODE, FTZ>(u, p));
        }
    } else {
        if (HIST) {
            hist_begin<kCopies, kBlock>(tbl, s_bins, s_cls, tid);
        }
        const size_t stride = (size_t)gridDim.x * kBlock;
        // every lane runs the same number of trips
        const size_t trips = (n + stride - 1) / stride;
        size_t i = (size_t)blockIdx.x * kBlock + tid;
        for (size_t t = 0; t < trips; ++t, i += stride) {
            const bool valid = i < n;
            const uint32_t u = valid ? x[i] : 0u;
            if (HIST) account<DEEP, kCopies>(u & 0x7FFFFFFFu, valid, p, tbl, lane32, w);
            if (STORE && valid) put_one(i, quantize_bits<MODE, FTZ>(u, p));
        }
    }

    if (HIST) {
        hist_clear<kBlock>(sink, blockIdx.x, gridDim.x, tid);
        hist_end<kCopies, kBlock>(tbl, s_bins, s_cls, w, p, sink, blockIdx.x, gridDim.x, tid);
    }
}

// Sums the shard records into the caller's fmt_hist_t and clears them for the next call (one
// workgroup; the stream orders it after the kernel that filled them).
constexpr int kFinSplit = 14;
__device__ __forceinline__ void finalize_body(unsigned long long *__restrict__ partials, int nrec, unsigned long long n,
                                              unsigned long long *__restrict__ hist)
{
    __shared__ unsigned long long acc[kSlots * kFinSplit];
    __shared__ unsigned long long tot[kSlots];
    const int tid = threadIdx.x;
    const int slot = tid % kSlots, part = tid / kSlots;
    if (part < kFinSplit) {
        unsigned long long s = 0;
        for (int r = part; r < nrec; r += kFinSplit) {
            s += partials[(size_t)r * kSlots + slot];
            partials[(size_t)r * kSlots + slot] = 0;
        }
        acc[part * kSlots + slot] = s;
    }
    __syncthreads();
    if (tid < kSlots) {
        unsigned long long s = 0;
        for (int q = 0; q < kFinSplit; ++q) s += acc[q * kSlots + tid];
        tot[tid] = s;
    }
    __syncthreads();
    if (tid < kSlots) hist[tid] = hist_slot(tot, n, tid);
}

__global__ __launch_bounds__(1024) void finalize_kernel(unsigned long long *__restrict__ partials, int nrec,
                                                        unsigned long long n, unsigned long long *__restrict__ hist)
{
    finalize_body(partials, nrec, n, hist);
}

int launch_hist_finalize(unsigned long long *partials, size_t n, fmt_hist_t *hist, hipStream_t stream)
{
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(1024), 0, stream, partials, partials ? kShards : 0,
                       (unsigned long long)n, reinterpret_cast<unsigned long long *>(hist));
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

template <int MODE, bool STORE, bool FTZ, bool HIST, bool DEEP, bool VEC, bool PACK>
static int launch_variant(const float *x, void *y, size_t n, size_t head, size_t nvec, const QuantParams &p,
                          fmt_hist_t *hist, hipStream_t stream, unsigned long long *fixed_partials)
{
    auto kern = stream_kernel<MODE, STORE, FTZ, HIST, DEEP, VEC, PACK, kCopiesMost>;
    if constexpr (HIST && STORE && !PACK && VEC)
        if (n >= kLarge) kern = stream_kernel<MODE, STORE, FTZ, HIST, DEEP, VEC, PACK, kCopiesLarge>;
    if constexpr (HIST && !STORE && VEC)
        if (n >= kAlone) kern = stream_kernel<MODE, STORE, FTZ, HIST, DEEP, VEC, PACK, kCopiesAlone>;
    int cus = 0;
    int rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    const size_t per_block = (size_t)kBlock * (VEC ? 4 * kUnroll : 4);
    const size_t want = (n + per_block - 1) / per_block;
    // Workgroups per compute unit, measured on 2^28 elements: a pure stream likes one 16 KiB tile per
    // workgroup (6.4 TB/s against 5.9 with 16 per CU: the hardware balances the tail); every workgroup
    // of a statistics pass pays for clearing and folding its LDS table, so the read-only pass keeps 16 per CU (161 us; 168 with 32,
    // 171 with 64 and 128) and the passes that write take 64 (fp32 355 us, codes 264; with 16: 367 and 290; with 128: alike).
    const size_t cap = (size_t)cus * (HIST ? (STORE ? kGridFused : kGridPerCU) : kGridStore);
    size_t g = want;
    if (HIST) {
        // mid-size tensors: at least four tiles per workgroup (one tile does not pay for the table), but no fewer workgroups
        // than four per compute unit (1 to 12 tried on 4 M elements: 8 gain 8 % for statistics alone and lose 10 % fused)
        const size_t resident = (size_t)cus * 4;
        g = (want + 3) / 4;
        if (g < resident) g = want < resident ? want : resident;
    }
    int grid = (int)(g < cap ? g : cap);
    if (grid < 1) grid = 1;
    HistSink sink{};
    if (HIST) {
        HistRecords at{fixed_partials, nullptr, 0u};
        if (fixed_partials == nullptr) {
            rc = get_hist_records(stream, (uint64_t)grid, &at);
            if (rc != FMT_OK) return rc;
        }
        sink = hist_sink(at, n, hist, (uint64_t)grid);
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, stream, reinterpret_cast<const uint32_t *>(x),
                       reinterpret_cast<uint32_t *>(y), n, head, nvec, p, sink);
    FMT_HIP_CHECK(hipGetLastError());
    if (HIST && sink.hist == nullptr) return launch_hist_finalize(sink.records, n, hist, stream);
    return FMT_OK;
}

int launch_stream(const float *x, void *y, size_t n, const QuantParams &p, bool ftz, fmt_hist_t *hist,
                  hipStream_t stream, bool pack16, unsigned long long *fixed_partials)
{
    const bool store = y != nullptr;
    const bool do_hist = hist != nullptr;
    const bool deep = do_hist && p.exp_lo < -126;
    if (n == 0) {
        if (do_hist) return launch_hist_finalize(nullptr, 0, hist, stream);
        return FMT_OK;
    }
    // elements before the first 16-byte boundary of x, and before the first 16-byte (codes: 8-byte)
    // boundary of y: both must agree for the vector path
    const size_t hx = ((16 - (reinterpret_cast<uintptr_t>(x) & 15)) & 15) / 4;
    const size_t hy = !store ? hx
                      : pack16 ? ((8 - (reinterpret_cast<uintptr_t>(y) & 7)) & 7) / 2
                               : ((16 - (reinterpret_cast<uintptr_t>(y) & 15)) & 15) / 4;
    const bool vec = hx == hy;
    size_t head = hx < n ? hx : n;
    size_t nvec = vec ? (n - head) / 4 : 0;
    if (!vec) head = 0;

#define FMT_LAUNCH_M(MD, S, F, H, D, PK)                                                                     \
    (vec ? launch_variant<MD, S, F, H, D, true, PK>(x, y, n, head, nvec, p, hist, stream, fixed_partials)           \
         : launch_variant<MD, S, F, H, D, false, PK>(x, y, n, head, nvec, p, hist, stream, fixed_partials))
#define FMT_LAUNCH(S, F, H, D)                                                                               \
    (p.mode == kModeMagic ? FMT_LAUNCH_M(kModeMagic, S, F, H, D, false)                                      \
     : p.mode == kModeInteger ? FMT_LAUNCH_M(kModeInteger, S, F, H, D, false)                                \
                              : FMT_LAUNCH_M(kModeMixed, S, F, H, D, false))
    // formats with a 16-bit code have m <= 14: never the m == 23 variant
#define FMT_LAUNCH_PACK(F, H, D)                                                                             \
    (p.mode == kModeInteger ? FMT_LAUNCH_M(kModeInteger, true, F, H, D, true) : FMT_LAUNCH_M(kModeMagic, true, F, H, D, true))
    if (pack16) {
        if (!store || p.mode == kModeMixed) return FMT_ERR_FORMAT;
        if (!do_hist) return ftz ? FMT_LAUNCH_PACK(true, false, false) : FMT_LAUNCH_PACK(false, false, false);
        if (deep) return ftz ? FMT_LAUNCH_PACK(true, true, true) : FMT_LAUNCH_PACK(false, true, true);
        return ftz ? FMT_LAUNCH_PACK(true, true, false) : FMT_LAUNCH_PACK(false, true, false);
    }
    // the statistics do not depend on how the rounding is carried out: one instantiation serves all
    if (!store)
        return deep ? FMT_LAUNCH_M(kModeMagic, false, false, true, true, false)
                    : FMT_LAUNCH_M(kModeMagic, false, false, true, false, false);
    if (!do_hist) return ftz ? FMT_LAUNCH(true, true, false, false) : FMT_LAUNCH(true, false, false, false);
    if (deep) return ftz ? FMT_LAUNCH(true, true, true, true) : FMT_LAUNCH(true, false, true, true);
    return ftz ? FMT_LAUNCH(true, true, true, false) : FMT_LAUNCH(true, false, true, false);
#undef FMT_LAUNCH_PACK
#undef FMT_LAUNCH_M
#undef FMT_LAUNCH
}

// ---- fmt_quantize_static: the partial records in a file-scope device array instead of allocated scratch
//
// Every GPU that loads the library holds its own copy of this array (36 KiB) until the process ends.
// In host code the array's name is only a handle for hipGetSymbolAddress: the address kernels and
// fills use is looked up once per device, with that device current, and kept.
static __device__ __align__(256) unsigned long long scratch[kShards * kSlots];

constexpr int kMaxDevices = 64;
static std::mutex g_static_mu;
static unsigned long long *g_static_ptr[kMaxDevices];

static int static_partials(unsigned long long **out)
{
    int dev = 0;
    FMT_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return FMT_ERR_HIP;
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (g_static_ptr[dev] == nullptr) {
        void *ptr = nullptr;
        FMT_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (ptr == nullptr) return FMT_ERR_HIP;
        g_static_ptr[dev] = static_cast<unsigned long long *>(ptr);
    }
    *out = g_static_ptr[dev];
    return FMT_OK;
}

__global__ __launch_bounds__(256) void clear_records_kernel(unsigned long long *__restrict__ rec, int n)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) rec[i] = 0ull;
}

int launch_stream_static(const float *x, float *y, size_t n, const QuantParams &p, bool ftz, fmt_hist_t *hist,
                         hipStream_t stream)
{
    unsigned long long *rec = nullptr;
    if (hist != nullptr && n > 0) {
        int rc = static_partials(&rec);
        if (rc != FMT_OK) return rc;
        // The array keeps whatever the last call on this GPU left in it.  A completed call leaves zeros
        // (its last kernel clears what it has summed), a call that failed half-way may not have: start clean.
        // A kernel, not a memset, so that the call can be recorded into a graph.
        hipLaunchKernelGGL(clear_records_kernel, dim3(kShards * kSlots / 256), dim3(256), 0, stream, rec, kShards * kSlots);
        FMT_HIP_CHECK(hipGetLastError());
    }
    return launch_stream(x, y, n, p, ftz, hist, stream, false, rec);
}

// codes -> fp32: 2 bytes read, 4 written per element.  In the vector body a lane turns four codes (one
// 64-bit load) into four values (one 128-bit store), four such units per trip, consecutive lanes on
// consecutive units so that loads and stores of a wave are contiguous; the at most 6 elements around
// the body go one per lane.
template <bool INTEGER, bool VEC>
__global__ __launch_bounds__(kBlock) void unpack16_kernel(const uint16_t *__restrict__ codes, uint32_t *__restrict__ y,
                                                          size_t n, size_t head, size_t nvec, QuantParams p)
{
    const uint32_t tid = threadIdx.x;
    if (VEC) {
        const u32x2 *cv = reinterpret_cast<const u32x2 *>(codes + head);
        u32x4 *yv = reinterpret_cast<u32x4 *>(y + head);
        constexpr int kU = 4;
        for (size_t base = (size_t)blockIdx.x * kBlock * kU; base < nvec; base += (size_t)gridDim.x * kBlock * kU) {
            u32x2 c[kU];
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                const size_t i = base + (size_t)k * kBlock + tid;
                c[k] = u32x2{0u, 0u};
                if (i < nvec) c[k] = __builtin_nontemporal_load(cv + i);
            }
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                const size_t i = base + (size_t)k * kBlock + tid;
                u32x4 o;
                o[0] = decode_bits<INTEGER>(c[k][0] & 0xFFFFu, p);
                o[1] = decode_bits<INTEGER>(c[k][0] >> 16, p);
                o[2] = decode_bits<INTEGER>(c[k][1] & 0xFFFFu, p);
                o[3] = decode_bits<INTEGER>(c[k][1] >> 16, p);
                if (i < nvec) __builtin_nontemporal_store(o, yv + i);
            }
        }
        if (blockIdx.x == 0 && tid < 64) {
            const size_t body_end = head + 4 * nvec;
            const size_t ntail = n - body_end;
            const size_t idx = tid < head ? tid : body_end + (tid - head);
            if (tid < head + ntail) y[idx] = decode_bits<INTEGER>(codes[idx], p);
        }
    } else {
        for (size_t i = (size_t)blockIdx.x * kBlock + tid; i < n; i += (size_t)gridDim.x * kBlock)
            y[i] = decode_bits<INTEGER>(codes[i], p);
    }
}

int launch_unpack16(const uint16_t *codes, float *y, size_t n, const QuantParams &p, hipStream_t stream)
{
    if (n == 0) return FMT_OK;
    if (p.mode == kModeMixed) return FMT_ERR_FORMAT;
    int cus = 0;
    int rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    // codes before the first 8-byte boundary of the codes, values before the first 16-byte boundary of y:
    // both must agree for the vector body
    const size_t hc = ((8 - (reinterpret_cast<uintptr_t>(codes) & 7)) & 7) / 2;        // 0..3
    const size_t hy = ((16 - (reinterpret_cast<uintptr_t>(y) & 15)) & 15) / 4;         // 0..3
    const bool vec = hc == hy;
    const size_t head = vec ? (hc < n ? hc : n) : 0;
    const size_t nvec = vec ? (n - head) / 4 : 0;
    const size_t per_block = (size_t)kBlock * (vec ? 16 : 1);
    const size_t want = (n + per_block - 1) / per_block;
    const size_t cap = (size_t)cus * kGridStore;
    const int grid = (int)(want < cap ? (want ? want : 1) : cap);
    uint32_t *yo = reinterpret_cast<uint32_t *>(y);
    const bool integer = p.mode == kModeInteger;
    if (vec) {
        if (integer)
            hipLaunchKernelGGL((unpack16_kernel<true, true>), dim3(grid), dim3(kBlock), 0, stream, codes, yo, n, head, nvec, p);
        else
            hipLaunchKernelGGL((unpack16_kernel<false, true>), dim3(grid), dim3(kBlock), 0, stream, codes, yo, n, head, nvec, p);
    } else {
        if (integer)
            hipLaunchKernelGGL((unpack16_kernel<true, false>), dim3(grid), dim3(kBlock), 0, stream, codes, yo, n, head, nvec, p);
        else
            hipLaunchKernelGGL((unpack16_kernel<false, false>), dim3(grid), dim3(kBlock), 0, stream, codes, yo, n, head, nvec, p);
    }
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

}  // namespace fmt
