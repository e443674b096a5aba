// fmt_gemm_fmac8: matrix product with the FMAC-8 accumulation of Sec. IV-A, Algorithm 1.
//
// Every output element is a dot product taken in groups of 8 consecutive k: inside a group a 16-bit
// accumulator a (a value of the format, starting at zero) takes 8 fused multiply-adds,
// a = Q(a + w_k * x_k) with ONE rounding of the exact sum to the format (FMAC of Sec. III-B); after
// the group it is added into an fp32 master accumulator with one fp32 addition; the result is
// Q(master).  (Operands are zero-padded to whole groups: a + 0 * 0 = a is a value of the format, so a
// padded step changes nothing.)  The chain of roundings is sequential by definition, so this is plain
// ALU work (no matrix cores), bound by the rate at which the vector units issue instructions: one per
// lane and clock.
//
// Four forms of the fused step, all giving the one rounding of the exact sum:
//   half    (binary16, 1/5/10) the packed 16-bit fused multiply-add of the vector units: half an instruction (fmac8_half_kernel).
//   wide    (e <= 6, m <= 11, operands of ordinary size: the common case) fp64 around the hardware's fused
//           multiply-add, s = fma(w, x, a), and the rounding (C + s) - C with C = t * 2^(52 - m), t about as large as s:
//           4 vector instructions (6 with the flush), and the vector units issue fp64 adds and fused multiply-adds
//           at the rate of single fp32 ones.  See fmac_wide for why the rounding to 53 bits on the way does no harm
//           as long as |s| stays below `wide_limit`; a workgroup takes this form for a stage of 32 k when
//           the largest operand magnitudes of the stage say that no sum can get there.
//   single  (the same formats, a stage with larger, infinite or NaN operands) fp32 around the hardware FMA:
//           the exact sum rounded once to 24 bits, then to the format, which equals rounding the exact sum
//           unless the 24-bit sum lands exactly on a midpoint of the format's grid while the exact sum
//           does not; a wave that holds such a lane computes the exact error of the sum and puts that lane on the
//           side of the midpoint where the exact sum lies.  About 16 instructions.
//   odd     (other formats) fp64: the product of two <= 24-bit significands is exact; the sum a + w*x is rounded
//           to odd (TwoSum gives the exact error; if it is non-zero and the fp64 sum is the even neighbour, step
//           to the odd one), which makes the following rounding to the format (<= 24 significant bits) equal to a
//           single rounding of the exact sum.  That rounding uses (|s| + C) - C with C = 2^(max(E,Emin) - m + 52),
//           the fp64 adder's own round-to-nearest-even.  About 25 instructions.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "fmt_internal.h"
#include "fmt_quant.h"

namespace fmt {

struct Fmac8Params {
    double ovf;          // magnitudes >= ovf round to infinity: (2 - 2^-(m+1)) * 2^Emax
    double minn;         // 2^Emin
    int32_t emin_biased; // Emin + 1023 (fp64 exponent field of minN)
    int32_t m;
    int32_t ftz;
};

// Q_{e,m,d|n} of an fp64 value that is either exact or rounded to odd; result as fp64 (a value of the format).
__device__ __forceinline__ double quantize_f64(double s, const Fmac8Params &f)
{
    const double as = fabs(s);
    const uint64_t ebits = (uint64_t)(__double_as_longlong(as) >> 52);
    const uint64_t ce = (ebits > (uint64_t)f.emin_biased ? ebits : (uint64_t)f.emin_biased) + (uint64_t)(52 - f.m);
    const double c = __longlong_as_double((long long)(ce << 52));
    double r = (as + c) - c;                       // RNE on the format's grid; NaN stays NaN
    if (f.ftz && r < f.minn) r = 0.0;
    if (as >= f.ovf) r = __longlong_as_double(0x7FF0000000000000ll);   // overflow and infinities
    return copysign(r, s);
}

// a + p rounded to odd (p = w*x exact).
__device__ __forceinline__ double add_round_to_odd(double a, double p)
{
    double s = a + p;
    const double bb = s - a;
    const double err = (a - (s - bb)) + (p - bb);  // exact error of the fp64 addition (TwoSum)
    long long u = __double_as_longlong(s);
    // err != 0 (and finite): the exact sum lies strictly between s and its neighbour on err's side
    if (err != 0.0 && err == err && (u & 1ll) == 0) {
        const bool away = (err > 0.0) == (s > 0.0);  // neighbour further from zero <=> pattern + 1
        u += away ? 1ll : -1ll;
        s = __longlong_as_double(u);
    }
    return s;
}

// The fused step in single precision, for formats with e <= 6 and m <= 11: the product of two
// (m+1)-bit significands has at most 24 bits and, with Emin >= -30, lies in fp32's normal range, so
// w * x and the error term of TwoSum are exact in fp32.
// The step around the hardware FMA (see the top of the file), in two parts so that the rare exact
// correction costs one branch per 16 steps instead of one per step.
struct FmaConsts {
    float minn, tovf, inf2;     // 2^Emin; the input magnitude from which the result is infinite; 2^(Emax+1)
};

// Common path: returns Q(fma(w, x, a)) and, in `tie`, whether the 24-bit sum sits exactly on a midpoint
// of the format's grid (then fmac_fix decides).  FIRST: the step from a zero accumulator -- the sum is the
// product itself, exact in 24 bits, so its rounding needs no second look (a midpoint there is a true tie).
template <bool FTZ, bool FIRST = false>
__device__ __forceinline__ float fmac_try(float a, float w, float x, const QuantParams &qp, const FmaConsts &k, bool &tie)
{
    const float s = FIRST ? __fmul_rn(w, x) : __fmaf_rn(w, x, a);   // exact product, exact sum, one rounding to 24 bits
    // C = 2^(max(E, Emin) + 23 - m): (|s| + C) - C rounds |s| to the format's grid around it (RNE).  For an
    // infinite or NaN s the pattern of C is a NaN, so r is: the selection below restores the infinity.
    const uint32_t ce = max(__float_as_uint(s) & 0x7F800000u, qp.minn_bits) + qp.shift23;
    const float c = __uint_as_float(ce), fa = fabsf(s);
    float r = __fsub_rn(__fadd_rn(fa, c), c);
    tie = !FIRST && fabsf(__fsub_rn(fa, r)) == __uint_as_float(ce - (24u << 23));   // moved by exactly half a step, C * 2^-24
    if (FTZ) r = r < k.minn ? 0.0f : r;                   // the flush acts on the rounded value
    r = fa >= k.tovf ? __uint_as_float(0x7F800000u) : r;  // false for NaN, which stays NaN
    return copysignf(r, s);
}

// Exact correction for the lanes where fmac_try reported a midpoint: a + w*x = s + err exactly (TwoSum on
// the exact product); a non-zero err puts the exact sum off the midpoint, on err's side, and the result
// is the grid neighbour on that side.
template <bool FTZ>
__device__ __forceinline__ float fmac_fix(float tried, float a, float w, float x, const QuantParams &qp, const FmaConsts &k)
{
    const float p = __fmul_rn(w, x);                       // exact (two (m+1)-bit significands)
    const float s = __fadd_rn(a, p);                       // the same 24-bit sum the FMA gave
    const float bb = __fsub_rn(s, a);
    const float err = __fadd_rn(__fsub_rn(a, __fsub_rn(s, bb)), __fsub_rn(p, bb));
    const uint32_t ce = max(__float_as_uint(s) & 0x7F800000u, qp.minn_bits) + qp.shift23;
    const float c = __uint_as_float(ce), fa = fabsf(s), half = __uint_as_float(ce - (24u << 23));
    const float r0 = __fsub_rn(__fadd_rn(fa, c), c);
    const bool tie = fabsf(__fsub_rn(fa, r0)) == half;
    if (!tie || !(err != 0.0f)) return tried;              // a true tie keeps the even neighbour the adder chose
    float r = ((err > 0.0f) == (s > 0.0f)) ? __fadd_rn(fa, half) : __fsub_rn(fa, half);
    if (FTZ) r = r < k.minn ? 0.0f : r;
    r = r >= k.inf2 ? __uint_as_float(0x7F800000u) : r;
    return copysignf(r, s);
}

// Constants of the wide step.
struct WideConsts {
    uint32_t floor_hi;   // hi word of 1.5 * 2^Emin
    double scale;        // 2^(52 - m)
    uint32_t flush_hi;   // hi word of 2^Emin - 2^(Emin - m - 1), whose lo word is zero
    float limit;         // the form is used while max|w| * max|x| of a stage stays below this
};

// The larger of |s| and 1.5 * 2^Emin with the lo word cleared, in one instruction: the hi words of two non-negative doubles
// compare like the singles of the same pattern (a pattern that is a denormal single belongs to a double below 2^-1015,
// here zero, and loses either way; one that is an infinite or NaN single to a double from 2^1017, far above the limit).
// pair: the registers it comes in, the lower one zero from the kernel's start on (the compiler does not know that it is, and so does not
// set it to zero before every step or every few).
typedef float hi_lo __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double carrier(double s, const WideConsts &k, hi_lo &pair)
{
    float t;
    asm("v_max_f32 %0, |%1|, %2" : "=v"(t) : "v"(__int_as_float(__double2hiint(s))), "s"(k.floor_hi));
    pair.y = t;
    return __builtin_bit_cast(double, pair);
}

// The fused step in fp64, for |a + w*x| < wide_limit = 2^(Emin - m + 52): 4 instructions (6 with the flush).
//   * s = fma(w, x, a) is the exact sum rounded to 53 bits; r = (C + s) - C rounds s to the format's grid at s, whose step is
//     G = 2^(max(E(s), Emin) - m).  C = t * 2^(52 - m), with t in [2^max(E, Emin), 2^(max(E, Emin) + 1)) a value of at most
//     21 bits (carrier): the last place of C is G, and C is a multiple of 2^32 G, so that C + s, rounded to a multiple of G,
//     is C plus the multiple nearest to s, ties to the even one, and taking C off again is exact.  C + s stays in C's
//     binade at the upper end (t is at least 2^(max(E, Emin) - 20) below the next power of two, |s| far less than that times
//     2^(52 - m)); at the lower end it may leave it for s < 0 and t = 2^E exactly -- then |s| < 2^E (1 + 2^-20), the grid
//     is the finer G/2, and the nearest multiple is 2^E as on G.  C is formed inside the two additions, exactly.
//     (With |s| itself in place of its first 21 bits C could be an odd multiple of G, and a sum that crosses into the next
//     binade, where multiples of 2G are taken, would come out one G off.)
//   * r is the single rounding of the exact sum: with s exact there is nothing to show.  a is a multiple of
//     2^(Emin - m), which is at least the last place of s, so only bits of p = w*x can be lost.  p has at most
//     2m + 2 bits, so a p with bits below the last place of s is smaller than 2^(E(s) - 51 + 2m) <=
//     2^(E(s) - m - 18) (m <= 11): the exact sum and s then lie within a tiny fraction of a grid step of a,
//     which is itself a grid point, and both round to a.
//   * the sign of a zero is not kept (-0 may come out as +0).  Nothing in the result depends on it: a zero of
//     either sign adds the same to a non-zero sum, and the fp32 master starts from +0, which stays +0 when a
//     zero of either sign is added.
// Results do not overflow below the limit (the caller's bound is below the format's overflow threshold as well).
template <bool FTZ, bool FIRST>
__device__ __forceinline__ double fmac_wide(double a, double w, double x, const WideConsts &k, hi_lo &pair)
{
    const double s = FIRST ? __dmul_rn(w, x) : __fma_rn(w, x, a);
    const double t = carrier(s, k, pair);
    const double r = __fma_rn(t, -k.scale, __fma_rn(t, k.scale, s));
    if (!FTZ) return r;
    // The result is below minN exactly where |s| is below minN less half a step (that midpoint goes to minN, the even
    // multiple), which s's hi word decides while the additions run.  r has at most 12 significant bits: its lo word is zero,
    // clearing the hi word makes a zero of it.
    const bool below = fabsf(__int_as_float(__double2hiint(s))) < __uint_as_float(k.flush_hi);
    return __hiloint2double(below ? 0 : __double2hiint(r), __double2loint(r));
}

// A stage's operand: a double, or (LOW) a float in the low word.
template <class A, bool LOW>
__device__ __forceinline__ A operand(double v)
{
    if constexpr (LOW) return __int_as_float(__double2loint(v));
    else return (A)v;
}

// A thread's elements of an operand's stages of KS k x 16 T rows, element `it` a fixed step from the one before it: consecutive lanes
// walk whichever of k and row is contiguous in memory.  PITCH: of a stage in LDS, [k][row].
template <int T, int KS, int PITCH = 16 * T + 2>
struct StageOperand {
    static constexpr int kRows = 16 * T, kCount = kRows * KS / 256;
    const uint32_t *first;           // element 0 of the stage that begins at k = 0
    int64_t step, stage;             // from element to element, from k to k
    int row, k, row_step, k_step, rows;
    bool inside;                     // the tile's rows are inside the operand
    __device__ __forceinline__ StageOperand(const uint32_t *X, int64_t ld, bool kcontig, int row0, int rows_, int tid)
    {
        row = kcontig ? tid / KS : tid % kRows;
        k = kcontig ? tid % KS : tid / kRows;
        row_step = kcontig ? 256 / KS : 0;
        k_step = kcontig ? 0 : 256 / kRows;
        first = X + (kcontig ? (int64_t)(row0 + row) * ld + k : (int64_t)k * ld + row0 + row);
        step = kcontig ? (int64_t)row_step * ld : (int64_t)k_step * ld;
        stage = kcontig ? 1 : ld;
        rows = rows_ - row0;
        inside = row0 + kRows <= rows_;
    }
    __device__ __forceinline__ void load(uint32_t (&v)[kCount], int k0, int K) const
    {
        const uint32_t *src = first + (int64_t)k0 * stage;
        if (inside && k0 + KS <= K) {            // the same in the whole workgroup
#pragma unroll
            for (int it = 0; it < kCount; ++it) v[it] = src[it * step];
        } else {
#pragma unroll
            for (int it = 0; it < kCount; ++it) {
                v[it] = 0u;
                if (row + it * row_step < rows && k0 + k + it * k_step < K) v[it] = src[it * step];
            }
        }
    }
    __device__ __forceinline__ int place(int it) const { return (k + it * k_step) * PITCH + row + it * row_step; }
};

constexpr int kFK = 32;        // k per LDS stage (a multiple of 8: FMAC-8 groups never straddle stages)
enum { kStepSingle = 0, kStepOdd = 1 };     // the form besides the wide one that an instantiation holds

// One workgroup computes a tile of 16*T x 16*T outputs, T x T per thread.  The chains of an output are sequential, so
// what counts is that every SIMD has instructions to issue: for the wide step 16 chains per thread where there are tiles enough
// to fill the chip, 4 or 1 where there are not; the round-to-odd step, five times as long, fills it with one (see launch).  Operand stages are rounded on the way into LDS, as fp64 (a
// value converted once instead of once per use); the next stage's loads are in flight while a stage is computed.
// Bound by the vector units: the four instructions of the steps alone, in registers, take 0.46 to 0.49 ms of the 0.58 below (the chip answers
// fp64 with its clock), the rest is the rounding of the operands, the additions to the masters and LDS.  Four workgroups per compute
// unit (128 registers; the few that spill belong to the loads of tiles at an edge) are all of the 1024 tiles of 2048 x 2048: with
// three, the fourth ran alone.
// Measured in 1/6/9: 2048 x 2048 x 1024 takes 0.58 ms (7.4 T fused steps/s; 0.63 ms with three workgroups per compute unit, the general
// rounding of the operands and 64 registers of addresses, 0.74 ms with a step of 5 instructions, 1.97 ms with the
// single form alone; the single form at 2048 x 2048 x 256 0.39 ms, 0.49 before), 256 x 256 x 256 takes 12.5 us (17 us with a step of 5 instructions whose operands were read one by one).
template <int MODE, bool FTZ, int STEP, int T>
__global__ __launch_bounds__(256, T > 2 ? 4 : 1) void fmac8_kernel(const uint32_t *__restrict__ A, int64_t lda, int transA,
                                                    const uint32_t *__restrict__ B, int64_t ldb, int transB,
                                                    float *__restrict__ C, int64_t ldc, int M, int N, int K,
                                                    int tiles_n, QuantParams qp, Fmac8Params fp, WideConsts wc)
{
    constexpr int kTile = 16 * T;                  // outputs per workgroup edge
    constexpr int kLoads = kTile * kFK / 256;      // elements of one operand per thread and stage
    __shared__ __attribute__((aligned(16))) double sa[kFK][kTile + 2];   // rounded operand values, [k][row]
    __shared__ __attribute__((aligned(16))) double sb[kFK][kTile + 2];
    __shared__ uint32_t s_max[2][4];               // largest operand magnitude of the stage, per wave
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int row0 = (blockIdx.x / tiles_n) * kTile, col0 = (blockIdx.x % tiles_n) * kTile;

    float acc32[T][T];                             // the fp32 master accumulators
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc32[i][j] = 0.0f;
    const FmaConsts fk = {__uint_as_float(qp.minn_bits), __uint_as_float(qp.t_ovf),
                          __uint_as_float((qp.t_ovf & 0x7F800000u) + 0x00800000u)};   // t_ovf lies in the top binade

    uint32_t va[kLoads], vb[kLoads];
    const StageOperand<T, kFK> oa(A, lda, !transA, row0, M, tid), ob(B, ldb, transB != 0, col0, N, tid);
    auto load = [&](int k0) {
        oa.load(va, k0, K);
        ob.load(vb, k0, K);
    };

    // The largest tile, whose thread uses a value four times, stores a stage for the form that the stage before it took: as fp64,
    // or (the single form) as fp32 in the low words.  Converting at each use instead made the single form 4 % slower there
    // (2048 x 2048 x 256 in 1/6/9: 512 us against 496 with three workgroups per compute unit, 390 now); the smaller tiles, which gain nothing, are 2 us faster without the
    // code for it (1024 x 1024 x 256, wide form: 66 us against 68).
    constexpr bool kLow = STEP == kStepSingle && T > 2;
    hi_lo pair = {0.0f, 0.0f};
    asm("" : "+v"(pair));
    bool wide = true;
    load(0);
    for (int k0 = 0; k0 < K; k0 += kFK) {
        // Rounding in the short form unless a wave holds something near overflow or beyond (13 instructions per element otherwise, a sixth of
        // the steps').  The largest magnitudes are taken of the unrounded elements, two per instruction, and rounded where they are used: the
        // rounding is monotonic.  NaN come out as the largest pattern.
        uint32_t ma = 0u, mb = 0u;
        auto top = [](const uint32_t (&v)[kLoads]) {
            float m = fabsf(__uint_as_float(v[0]));
#pragma unroll
            for (int it = 1; it + 1 < kLoads; it += 2)
                m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(__uint_as_float(v[it])), fabsf(__uint_as_float(v[it + 1]))), m);
            if (kLoads % 2 == 0) m = __builtin_elementwise_maximum(fabsf(__uint_as_float(v[kLoads - 1])), m);
            return __float_as_uint(m) & 0x7FFFFFFFu;
        };
        ma = top(va), mb = top(vb);
        if (MODE != kModeMixed && __ballot(max(ma, mb) >= qp.t_ovf) == 0ull) {        // the same in the whole wave
            const RoundMasks masks = round_masks(qp);
#pragma unroll
            for (int it = 0; it < kLoads; ++it) {
                if constexpr (MODE != kModeMixed) {
                    va[it] = quantize_short<MODE, FTZ, false>(va[it], qp, masks);     // the sign of a zero changes nothing
                    vb[it] = quantize_short<MODE, FTZ, false>(vb[it], qp, masks);
                }
            }
        } else {
#pragma unroll
            for (int it = 0; it < kLoads; ++it) {
                va[it] = quantize_bits<MODE, FTZ>(va[it], qp);
                vb[it] = quantize_bits<MODE, FTZ>(vb[it], qp);
            }
        }
        auto store = [&](auto place) __attribute__((always_inline)) {
#pragma unroll
            for (int it = 0; it < kLoads; ++it) {
                (&sa[0][0])[oa.place(it)] = place(va[it]);
                (&sb[0][0])[ob.place(it)] = place(vb[it]);
            }
        };
        if (!kLow || wide) store([](uint32_t q) { return (double)__uint_as_float(q); });
        else store([](uint32_t q) { return __hiloint2double(0, (int)q); });
        if (STEP == kStepSingle) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                ma = max(ma, (uint32_t)__shfl_xor((int)ma, off, 64));
                mb = max(mb, (uint32_t)__shfl_xor((int)mb, off, 64));
            }
            if ((tid & 63) == 0) {
                s_max[0][tid >> 6] = ma;
                s_max[1][tid >> 6] = mb;
            }
        }
        __syncthreads();
        if (k0 + kFK < K) load(k0 + kFK);          // in flight while this stage is computed
        if (STEP == kStepSingle) {
            const uint32_t wa = quantize_bits<MODE, FTZ>(max(max(s_max[0][0], s_max[0][1]), max(s_max[0][2], s_max[0][3])), qp);
            const uint32_t wb = quantize_bits<MODE, FTZ>(max(max(s_max[1][0], s_max[1][1]), max(s_max[1][2], s_max[1][3])), qp);
            // infinities and NaN (patterns from 0x7F800000) are left to the other form
            const bool fits = wa < 0x7F800000u && wb < 0x7F800000u && __fmul_rn(__uint_as_float(wa), __uint_as_float(wb)) < wc.limit;
            const bool next = __builtin_amdgcn_readfirstlane(fits ? 1 : 0) != 0;      // the same in the whole workgroup
            if (kLow && next != wide) {            // stored for the other form: every thread converts what it stored
                auto other = [&](double v) {
                    return next ? (double)operand<float, true>(v) : __hiloint2double(0, __float_as_int((float)v));
                };
#pragma unroll
                for (int it = 0; it < kLoads; ++it) {
                    double &at = (&sa[0][0])[oa.place(it)], &bt = (&sb[0][0])[ob.place(it)];
                    at = other(at);
                    bt = other(bt);
                }
                __syncthreads();
            }
            wide = next;
        }
        // groups of 8 k (the stage is zero-padded beyond K): 8 fused steps from a = 0, then one fp32 addition
        if (STEP == kStepSingle && wide) {
#pragma unroll 1
            for (int g = 0; g < kFK / 8; ++g) {
                double a16[T][T];
                double w[8][T], x[8][T];
                auto read = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < T; ++i) {
                        w[kk][i] = sa[g * 8 + kk][ty * T + i];
                        x[kk][i] = sb[g * 8 + kk][tx * T + i];
                    }
                };
                // few chains per thread: operands are read ahead of the steps, which would wait for them one by one; with four chains half a
                // group's at a time (a whole group's take the registers of a fifth wave per SIMD, from the single form as well: 1500 x 1500 x
                // 256 in 1/6/9 240 us instead of 229; wide form 107 and 106)
                constexpr int kAhead = T == 1 ? 8 : T == 2 ? 4 : 1;
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    if (kk % kAhead == 0) {
#pragma unroll
                        for (int k2 = 0; k2 < kAhead; ++k2) read(kk + k2);
                        if (T <= 2) __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
                            a16[i][j] = kk == 0 ? fmac_wide<FTZ, true>(0.0, w[kk][i], x[kk][j], wc, pair)
                                                : fmac_wide<FTZ, false>(a16[i][j], w[kk][i], x[kk][j], wc, pair);
                }
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) acc32[i][j] = __fadd_rn(acc32[i][j], (float)a16[i][j]);
            }
        } else {
            typedef typename std::conditional<STEP == kStepSingle, float, double>::type acc_t;
            // four chains at a time: with sixteen the intermediates of a step take the registers of a third wave per SIMD, from
            // the wide form as well (T = 4: 222 registers; 164 now; 2048 x 2048 x 1024, wide form: 776 -> 741 us)
            constexpr int R = T > 2 ? 1 : T;
#pragma unroll 1
            for (int g = 0; g < kFK / 8; ++g) {
#pragma unroll
                for (int i0 = 0; i0 < T; i0 += R) {
                    acc_t a16[R][T];
#pragma unroll
                    for (int i = 0; i < R; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j) a16[i][j] = (acc_t)0;
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) {
                        acc_t w[R], x[T];
#pragma unroll
                        for (int i = 0; i < R; ++i) w[i] = operand<acc_t, kLow>(sa[g * 8 + kk][ty * T + i0 + i]);
#pragma unroll
                        for (int j = 0; j < T; ++j) x[j] = operand<acc_t, kLow>(sb[g * 8 + kk][tx * T + j]);
                        if constexpr (STEP == kStepSingle) {
                            // the chains take their step; which lanes met a midpoint is kept as wave masks
                            float nx[R][T];
                            unsigned long long met[R][T], any = 0ull;
#pragma unroll
                            for (int i = 0; i < R; ++i)
#pragma unroll
                                for (int j = 0; j < T; ++j) {
                                    bool tie;
                                    nx[i][j] = kk == 0 ? fmac_try<FTZ, true>(a16[i][j], w[i], x[j], qp, fk, tie)
                                                       : fmac_try<FTZ, false>(a16[i][j], w[i], x[j], qp, fk, tie);
                                    met[i][j] = __ballot(tie);
                                    any |= met[i][j];
                                }
                            if (any != 0ull) {                     // wave-uniform
#pragma unroll
                                for (int i = 0; i < R; ++i)
#pragma unroll
                                    for (int j = 0; j < T; ++j)
                                        if (met[i][j] != 0ull) nx[i][j] = fmac_fix<FTZ>(nx[i][j], a16[i][j], w[i], x[j], qp, fk);
                            }
#pragma unroll
                            for (int i = 0; i < R; ++i)
#pragma unroll
                                for (int j = 0; j < T; ++j) a16[i][j] = nx[i][j];
                        } else {
#pragma unroll
                            for (int i = 0; i < R; ++i)
#pragma unroll
                                for (int j = 0; j < T; ++j) a16[i][j] = quantize_f64(add_round_to_odd(a16[i][j], w[i] * x[j]), fp);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < R; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j) acc32[i0 + i][j] = acc32[i0 + i][j] + (float)a16[i][j];   // single-precision addition
                    if (R < T) __builtin_amdgcn_sched_barrier(0);  // the next rows' step stays behind this one's
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int r = row0 + ty * T + i;
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int c = col0 + tx * T + j;
            if (r < M && c < N)
                C[(size_t)r * ldc + c] = __uint_as_float(quantize_bits<MODE, FTZ>(__float_as_uint(acc32[i][j]), qp));
        }
    }
}

// binary16 (1/5/10), bound by the issue of vector instructions (about 1.2 per step with the conversions, the additions to the
// masters and the staging): 2048 x 2048 x 1024 takes 0.18 ms, 0.20 in 1/5/10/n (0.74 and 0.96 in the wide form of five
// instructions); a result of up to 512 x 512 x 256 11 us (17 - 29), bound by the latency of its stages.
// The vector units' own packed fused multiply-add takes two steps per instruction -- v_pk_fma_f16 rounds the
// exact w*x + a once to binary16, to nearest even, with denormal results and overflow to infinity, which is the step of 1/5/10/d.
// For 1/5/10/n the kernel runs with denormal inputs of 16-bit operations read as zero and denormal results kept (MODE.FP_DENORM
// of the 16- and 64-bit operations = 2): a step rounds first, and a result below minN is a zero to the step that follows, and to
// the end of the group by a selection.
template <bool FTZ, int T>
__global__ __launch_bounds__(256) void fmac8_half_kernel(const float *__restrict__ A, int64_t lda, int transA,
                                                         const float *__restrict__ B, int64_t ldb, int transB,
                                                         float *__restrict__ C, int64_t ldc, int M, int N, int K, int tiles_n,
                                                         QuantParams qp)
{
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    constexpr int kTile = 16 * T;
    constexpr int kHK = T == 2 ? 64 : 32;           // k per stage
    constexpr int kLoads = kTile * kHK / 256;      // elements of one operand per thread and stage
    __shared__ __attribute__((aligned(16))) _Float16 sa[2][kHK][kTile + 4];   // rounded operand values, [k][row]; two stages
    __shared__ __attribute__((aligned(16))) _Float16 sb[2][kHK][kTile + 4];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int row0 = (blockIdx.x / tiles_n) * kTile, col0 = (blockIdx.x % tiles_n) * kTile;
    if (FTZ) __builtin_amdgcn_s_setreg(1 | (6 << 6) | (1 << 11), 2);         // MODE[7:6]

    float acc32[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc32[i][j] = 0.0f;

    float va[kLoads], vb[kLoads];
    // element `it` of this thread, as in fmac8_kernel
    auto at = [&](int it, bool kcontig, int &r, int &k) {
        const int idx = it * 256 + tid;
        r = kcontig ? idx / kHK : idx % kTile;
        k = kcontig ? idx % kHK : idx / kTile;
    };
    auto load = [&](int k0) {
#pragma unroll
        for (int it = 0; it < kLoads; ++it) {
            int r, k;
            at(it, !transA, r, k);
            va[it] = 0.0f;
            if (row0 + r < M && k0 + k < K) va[it] = transA ? A[(size_t)(k0 + k) * lda + row0 + r] : A[(size_t)(row0 + r) * lda + k0 + k];
            at(it, transB != 0, r, k);
            vb[it] = 0.0f;
            if (col0 + r < N && k0 + k < K) vb[it] = transB ? B[(size_t)(col0 + r) * ldb + k0 + k] : B[(size_t)(k0 + k) * ldb + col0 + r];
        }
    };
    // the conversion to binary16 is the rounding of 1/5/10/d; 1/5/10/n reads its denormals as zeros
    auto store = [&](int buf) {
#pragma unroll
        for (int it = 0; it < kLoads; ++it) {
            int r, k;
            at(it, !transA, r, k);
            sa[buf][k][r] = static_cast<_Float16>(va[it]);
            at(it, transB != 0, r, k);
            sb[buf][k][r] = static_cast<_Float16>(vb[it]);
        }
    };

    load(0);
    store(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < K; k0 += kHK) {
        const bool more = k0 + kHK < K;
        if (more) load(k0 + kHK);                  // in flight while this stage is computed
#pragma unroll 1
        for (int g = 0; g < kHK / 8; ++g) {
            f16x2 a16[T][T / 2], w[8][T / 2], x[8][T / 2];
            auto read = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < T / 2; ++i) {
                    w[kk][i] = *reinterpret_cast<const f16x2 *>(&sa[buf][g * 8 + kk][ty * T + 2 * i]);
                    x[kk][i] = *reinterpret_cast<const f16x2 *>(&sb[buf][g * 8 + kk][tx * T + 2 * i]);
                }
            };
            if constexpr (T == 2) {
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) read(kk);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                if constexpr (T > 2) read(kk);
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    const f16x2 wi = {w[kk][i / 2][i & 1], w[kk][i / 2][i & 1]};
#pragma unroll
                    for (int j = 0; j < T / 2; ++j) a16[i][j] = kk == 0 ? wi * x[kk][j] : __builtin_elementwise_fma(wi, x[kk][j], a16[i][j]);
                }
            }
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    float a = static_cast<float>(a16[i][j / 2][j & 1]);
                    if (FTZ) a = fabsf(a) < 0x1p-14f ? 0.0f : a;
                    acc32[i][j] = __fadd_rn(acc32[i][j], a);
                }
        }
        buf ^= 1;
        if (more) store(buf);                      // the stage before this one was read before the last barrier
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int r = row0 + ty * T + i;
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int c = col0 + tx * T + j;
            if (r < M && c < N)
                C[(size_t)r * ldc + c] = __uint_as_float(quantize_bits<kModeMagic, FTZ>(__float_as_uint(acc32[i][j]), qp));
        }
    }
}

template <bool FTZ, int T>
static int launch_half_tile(int transA, int transB, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb,
                            float *C, int64_t ldc, const QuantParams &qp, hipStream_t stream)
{
    const int tiles_m = (M + 16 * T - 1) / (16 * T), tiles_n = (N + 16 * T - 1) / (16 * T);
    if ((int64_t)tiles_m * tiles_n >= ((int64_t)1 << 31)) return FMT_ERR_SHAPE;
    hipLaunchKernelGGL((fmac8_half_kernel<FTZ, T>), dim3(tiles_m * tiles_n), dim3(256), 0, stream, A, lda, transA, B, ldb, transB, C,
                       ldc, M, N, K, tiles_n, qp);
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

template <bool FTZ>
static int launch_half(int transA, int transB, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb,
                       float *C, int64_t ldc, const QuantParams &qp, hipStream_t stream)
{
#define FMT_TILE(T) launch_half_tile<FTZ, T>(transA, transB, M, N, K, A, lda, B, ldb, C, ldc, qp, stream)
    // Measured (us, N x N x 256, T = 2 / 4): N = 64 ... 512: 11 / 25; 768: 16 / 26; 1024: 20 / 26; 1500: 40 / 41; 2048: 66 / 51.
    int cus = 0;
    const int rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    auto estimate = [&](int t, double alone, double each) {
        const int64_t tiles = (((int64_t)M + 16 * t - 1) / (16 * t)) * (((int64_t)N + 16 * t - 1) / (16 * t));
        return std::max(alone, (double)((tiles + cus - 1) / cus) * each);
    };
    return estimate(2, 10.8, 4.2) <= estimate(4, 25.0, 13.2) ? FMT_TILE(2) : FMT_TILE(4);
#undef FMT_TILE
}

template <int MODE, bool FTZ, int STEP, int T>
static int launch_tile(int transA, int transB, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb,
                       float *C, int64_t ldc, const QuantParams &qp, const Fmac8Params &fp, const WideConsts &wc, hipStream_t stream)
{
    const int tiles_m = (M + 16 * T - 1) / (16 * T), tiles_n = (N + 16 * T - 1) / (16 * T);
    if ((int64_t)tiles_m * tiles_n >= ((int64_t)1 << 31)) return FMT_ERR_SHAPE;
    hipLaunchKernelGGL((fmac8_kernel<MODE, FTZ, STEP, T>), dim3(tiles_m * tiles_n), dim3(256), 0, stream,
                       reinterpret_cast<const uint32_t *>(A), lda, transA, reinterpret_cast<const uint32_t *>(B), ldb,
                       transB, C, ldc, M, N, K, tiles_n, qp, fp, wc);
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

template <int MODE, bool FTZ, int STEP>
static int launch(int transA, int transB, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb,
                  float *C, int64_t ldc, const QuantParams &qp, const Fmac8Params &fp, const WideConsts &wc, hipStream_t stream)
{
#define FMT_TILE(T) launch_tile<MODE, FTZ, STEP, T>(transA, transB, M, N, K, A, lda, B, ldb, C, ldc, qp, fp, wc, stream)
    // Which tile, from products of N x N x 256 on 256 compute units.
    if constexpr (STEP == kStepOdd) {
        // One output per thread at any size.  Measured in 1/8/7 (us, T = 1 / 2 / 4): N = 256: 36 / 103 / 376; 512: 69 / 106 / 378; 640:
        // 106 / 140 / 382; 768: 131 / 190 / 382; 1024: 221 / 242 / 382; 1500: 464 / 491 / 732; 2048: 837 / 844 / 933; 1/6/15 is alike.
        return FMT_TILE(1);
    } else {
        // `alone` is what one tile on a compute unit takes (the chains' latency with 1, 4 or 16 of them to interleave), `each` the
        // time per tile of a compute unit with work enough.  Measured in 1/6/9, wide form (us, T = 1 / 2 / 4): N = 64: 13.2 / 21.6 /
        // 53; 384: 22 / 23 / 54; 512: 28 / 23 / 55; 600: 38 / 32 / 63; 640: 42 / 31 / 55; 768: 52 / 39 / 56; 1024: 88 / 49 / 56; 1350: 154 / 88 /
        // 92; 1500: 184 / 98 / 125; 2048: 332 / 165 / 151.  The values decide which form a stage takes; at 448 and 512, where four chains per
        // thread would gain 5 us, the single form loses 29, so the line lies above them: the constants are a little above the wide form's
        // times (those are 13.4 / 5.2, 21.6 / 12.3 and 54 / 38).  Elsewhere the rule is within 4 % of the best tile in the wide form.  Where
        // all stages take the single form it is off by up to a third (640: 61 / 78 / 244; 768: 75 / 94 / 244; 1024: 122 / 115 / 246; 1350: 206 / 199 /
        // 267; 1500: 247 / 223 / 319; 1900: 386 / 345 / 391; 2048: 441 / 371 / 391).
        int cus = 0;
        const int rc = device_cu_count(&cus);
        if (rc != FMT_OK) return rc;
        auto estimate = [&](int t, double alone, double each) {
            const int64_t tiles = (((int64_t)M + 16 * t - 1) / (16 * t)) * (((int64_t)N + 16 * t - 1) / (16 * t));
            return std::max(alone, (double)((tiles + cus - 1) / cus) * each);
        };
        const double t1 = estimate(1, 16.8, 5.8), t2 = estimate(2, 28.7, 15.0), t4 = estimate(4, 62.7, 48.0);
        if (t4 <= t2 && t4 <= t1) return FMT_TILE(4);
        return t2 <= t1 ? FMT_TILE(2) : FMT_TILE(1);
    }
#undef FMT_TILE
}

// FMT_FMAC8_F64=1 keeps every format on the round-to-odd form (tests compare the two).
static bool fmac8_force_f64()
{
    const char *env = getenv("FMT_FMAC8_F64");
    return env != nullptr && env[0] == '1';
}

int launch_gemm_fmac8(int transA, int transB, int64_t M, int64_t N, int64_t K, const float *A, int64_t lda,
                      const float *B, int64_t ldb, float *C, int64_t ldc, fmt_format_t f, const QuantParams &qp,
                      hipStream_t stream)
{
    const int bias = (1 << (f.e - 1)) - 1;
    Fmac8Params fp;
    fp.ovf = ldexp(2.0 - ldexp(1.0, -(f.m + 1)), bias);
    fp.minn = ldexp(1.0, 1 - bias);
    fp.emin_biased = 1 - bias + 1023;
    fp.m = f.m;
    fp.ftz = f.denorm == 0;
    const bool ftz = f.denorm == 0;
    WideConsts wc;
    wc.floor_hi = ((uint32_t)(1 - bias + 1023) << 20) | 0x80000u;
    wc.scale = ldexp(1.0, 52 - f.m);
    const double flush = ldexp(1.0, 1 - bias) - ldexp(1.0, -bias - f.m);       // half a step below minN: m fractional ones, all in the hi word
    uint64_t flush_bits = 0;
    memcpy(&flush_bits, &flush, sizeof(flush_bits));
    wc.flush_hi = (uint32_t)(flush_bits >> 32);
    // Below 2^(Emin - m + 52) the wide step is exact (see fmac_wide), below 2^Emax nothing overflows.  Through the 8
    // steps of a group |a + w*x| grows to at most max|w*x| times the sum of (1 + 2^-(m+1))^i, i = 0..8 (each step's
    // rounding adds at most half a last place): that factor, and a little for the product of the maxima, comes off.
    double growth = 0.0;
    for (int i = 0; i <= 8; ++i) growth += pow(1.0 + ldexp(1.0, -(f.m + 1)), i);
    wc.limit = (float)(0.99 * ldexp(1.0, 1 - bias - f.m + 52 < bias ? 1 - bias - f.m + 52 : bias) / growth);
#define FMT_RUN(MD, STEP)                                                                                             \
    (ftz ? launch<MD, true, STEP>(transA, transB, (int)M, (int)N, (int)K, A, lda, B, ldb, C, ldc, qp, fp, wc, stream) \
         : launch<MD, false, STEP>(transA, transB, (int)M, (int)N, (int)K, A, lda, B, ldb, C, ldc, qp, fp, wc, stream))
    if (f.e == 5 && f.m == 10 && !fmac8_force_f64())
        return ftz ? launch_half<true>(transA, transB, (int)M, (int)N, (int)K, A, lda, B, ldb, C, ldc, qp, stream)
                   : launch_half<false>(transA, transB, (int)M, (int)N, (int)K, A, lda, B, ldb, C, ldc, qp, stream);
    // wide and single-precision fused steps where they are exact: 1/6/9 and its neighbours
    if (f.e <= 6 && f.m <= 11 && !fmac8_force_f64()) return FMT_RUN(kModeMagic, kStepSingle);
    if (qp.mode == kModeMagic) return FMT_RUN(kModeMagic, kStepOdd);
    if (qp.mode == kModeInteger) return FMT_RUN(kModeInteger, kStepOdd);
    return FMT_RUN(kModeMixed, kStepOdd);
#undef FMT_RUN
}

}  // namespace fmt
