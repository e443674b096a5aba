// The product kernels (see fmt_gemm.hip for what they multiply) and their launches, instantiated per piece scheme.
#pragma once

#include <cstdlib>
#include <type_traits>

#include "fmt_hist.h"
#include "fmt_internal.h"
#include "fmt_product.h"
#include "fmt_quant.h"
#include "fmt_split.h"
#include "fmt_tail.h"

namespace fmt {

// Epilogue of one wave.  The MFMAs are fed operand B's fragment first and A's second, so a 32 x 32 accumulator
// block holds the TRANSPOSE of the usual layout: register v of lane l holds row l % 32 and column
// 8*(v/4) + 4*(l/32) + v%4 of the block of C -- four consecutive columns per group of four registers, which
// leave in one 16-byte store per lane (64 store instructions per wave for a 256 x 256 tile instead of 256;
// nothing is assumed about alignment beyond 4 bytes).
// SCALED: out = acc * 2^-(S_row + S_col), exactly; the scale arrays are padded to the tile grid and 16-byte
// aligned, and all of a lane's scales are fetched together ahead of its stores.
// img > 0: column = (image, position), element (row, col) goes to out[image][row][position] (NCHW with `img`
// positions); the four columns of a group go out together when they fall into one image.
// A wave whose block of C lies inside the matrix (all but the last row and column of tiles) takes a path without
// per-lane tests, in two phases: first every accumulator is scaled in place, then the stores go out straight
// from the accumulator registers.  Measured on a 256 x 256 tile (one wave per SIMD): stores interleaved with
// the arithmetic that refills their data registers take 20 - 25 us per tile when every compute unit stores at
// once (a store holds its data registers until the memory pipeline has taken them), the two phases 8 us, of
// which the stores are 5.
template <int TM, int TN, bool SCALED>
__device__ __forceinline__ void store_tile(floatx16 (&acc)[TM][TN], float *__restrict__ out, int64_t ld, int M, int N, int img,
                                           int row_base, int col_base, int lane, const int *__restrict__ Sa,
                                           const int *__restrict__ Sb)
{
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const int r_in = lane & 31, c_half = (lane >> 5) * 4;
    int sa[TM];
    i32x4 sb[TN][4];
    if constexpr (SCALED) {
#pragma unroll
        for (int i = 0; i < TM; ++i) sa[i] = Sa[row_base + i * 32 + r_in];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) sb[j][g] = -*reinterpret_cast<const i32x4 *>(Sb + col_base + j * 32 + g * 8 + c_half);
    }
    // rows are `rs` elements apart in both output maps
    const size_t rs = img > 0 ? (size_t)img : (size_t)ld;
    float *rowp[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) rowp[i] = out + (size_t)(row_base + i * 32 + r_in) * rs;

    if (row_base + 32 * TM <= M && col_base + 32 * TN <= N && (img & 3) == 0) {      // the same in the whole wave
        if constexpr (SCALED) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = ldexpf(acc[i][j][v], sb[j][v >> 2][v & 3] - sa[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the four stores that complete the 128-byte lines of a block go out back to back
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            size_t coff[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col0 = col_base + j * 32 + g * 8 + c_half;
                coff[g] = (size_t)col0;
                if (img > 0) {                   // img is a multiple of 4 and so is col0: one image holds the four columns
                    const int image = col0 / img;
                    coff[g] = (size_t)image * M * img + (col0 - image * img);
                }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4u v;
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] = acc[i][j][g * 4 + c];
                    *reinterpret_cast<f32x4u *>(rowp[i] + coff[g]) = v;
                }
        }
        return;
    }
    // the last row or column of tiles, and NCHW maps whose images are not a multiple of 4 positions long
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col0 = col_base + j * 32 + g * 8 + c_half;
            if (col0 >= N) continue;
            // offset of column col0 within a row of the output map; whether its four columns are adjacent there
            size_t coff = (size_t)col0;
            bool together = col0 + 3 < N;
            if (img > 0) {
                const int image = col0 / img, pos = col0 - image * img;
                coff = (size_t)image * M * img + pos;
                together = together && pos + 3 < img;
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (row_base + i * 32 + r_in >= M) continue;
                f32x4u v;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    v[c] = acc[i][j][g * 4 + c];
                    if constexpr (SCALED) v[c] = ldexpf(v[c], sb[j][g][c] - sa[i]);
                }
                if (together) {
                    *reinterpret_cast<f32x4u *>(rowp[i] + coff) = v;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (col0 + c < N) {
                            size_t off = coff + c;
                            if (img > 0) {
                                const int image = (col0 + c) / img;
                                off = (size_t)image * M * img + (col0 + c - image * img);
                            }
                            rowp[i][off] = v[c];
                        }
                }
            }
        }
}

// The scales of exponent planes undone in place (see store_tile).
template <int TM, int TN>
__device__ __forceinline__ void unscale_tile(floatx16 (&acc)[TM][TN], int row_base, int col_base, int lane, const int *__restrict__ Sa,
                                             const int *__restrict__ Sb)
{
    typedef int i32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int sa = Sa[row_base + i * 32 + (lane & 31)];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const i32x4 sb = *reinterpret_cast<const i32x4 *>(Sb + col_base + j * 32 + g * 8 + (lane >> 5) * 4);
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[i][j][4 * g + c] = ldexpf(acc[i][j][4 * g + c], -(sb[c] + sa));
            }
    }
}

// replicas of the statistics table: as in the stream kernels, as many as fit a stage buffer of the smallest tile
constexpr int linear_copies(int tiles) { return tiles == 1 ? 4 : 8; }

// Outputs of a fully connected layer from a workgroup's accumulators, R(t) with t = R(acc) + R(b) (Sec. IV-A), HIST: and the statistics
// of t (Sec. V), to C or as 16-bit codes.  tbl: LDS that holds the statistics' table once every wave is done with its stages.
// The common case takes the short forms of the rounding on the accumulators: about 20 vector instructions per output, half
// of them the statistics, four neighbouring columns (a quad of registers) at a time.  A wave that holds sums or biases near the
// format's largest value or beyond leaves its sums in C and takes a loop over them: the code of the common case
// stays a few kilobytes (with both forms unrolled it is ten times that, and the workgroups wait for instructions).
// Formats without a short form never come here, nor do 128 x 128 tiles that cut a quad (product_of_views).
template <int PS, int TM, int TN, bool HIST>
__device__ __forceinline__ void linear_tile(floatx16 (&acc)[TM][TN], float *C, int64_t ldc, int M, int N, int row_base, int col_base, int lane,
                                            const uint32_t (&bias)[TN][16], const LinearOut &lin, const HistSink &sink, uint32_t *tbl,
                                            int tile, int ntiles)
{
    typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
    typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(2)));
    constexpr int kCopies = linear_copies(TM * TN);
    // quads that N cuts among the common ones: 40 % more code in a 128 x 128 tile (4096 x 3072 x 1024 in 1/6/9 with statistics and no such
    // quad 53 -> 69 us and more when it was measured, with 148 KB of code and spills; 77 KB without, and no spills, now), so not there
    constexpr bool kCut = TM * TN < 4;
    __shared__ uint32_t s_bins[HIST ? FMT_NBINS : 1], s_cls[HIST ? 8 : 1];
    const QuantParams &p = lin.p;
    const bool has_bias = lin.bias != nullptr;
    const uint32_t tid = threadIdx.x, copy = tid % kCopies;
    Counts w;

    // |acc| + |b| below half of the smallest magnitude that rounds to infinity keeps |t| below it: either rounding adds at most half a
    // step, an eighth of the largest power of two at that height (NaN is not below)
    float top = 0.0f, topb = 0.0f;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            topb = __builtin_elementwise_maximum(fabsf(__uint_as_float(bias[j][v])), topb);
#pragma unroll
            for (int i = 0; i < TM; ++i) top = __builtin_elementwise_maximum(fabsf(acc[i][j][v]), top);
        }
    const bool rare = __ballot(!(top + topb < 0.5f * __uint_as_float(p.t_ovf))) != 0ull;     // the same in the whole wave
    if constexpr (HIST) {
        __syncthreads();                         // every wave is done with the stage buffers
        hist_begin<kCopies, 256>(tbl, s_bins, s_cls, tid);
    }

    if (!rare) {
        const RoundMasks masks = round_masks(p);
        const int row_in = row_base + (lane & 31), col_in = col_base + (lane >> 5) * 4;
        auto run = [&](auto mode, auto flush) __attribute__((always_inline)) {
            constexpr int MODE = decltype(mode)::value;
            constexpr bool FTZ = decltype(flush)::value;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int col = col_in + j * 32 + g * 8;
                    const int left = kCut ? N - col : (col < N ? 4 : 0);     // columns of the quad inside the matrix
                    if (left <= 0) continue;
                    uint32_t rb[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) rb[c] = has_bias ? quantize_short<MODE, FTZ>(bias[j][4 * g + c], p, masks) : 0u;
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const int row = row_in + i * 32;
                        if (row >= M) continue;
                        uint32_t t[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            t[c] = quantize_short<MODE, FTZ>(__float_as_uint(acc[i][j][4 * g + c]), p, masks);
                            if (has_bias) t[c] = __float_as_uint(__fadd_rn(__uint_as_float(t[c]), __uint_as_float(rb[c])));
                            if constexpr (HIST) account_below<kCopies>(t[c] & 0x7FFFFFFFu, !kCut || c == 0 || c < left, p, tbl, copy, w);
                            if (has_bias) t[c] = quantize_short<MODE, FTZ>(t[c], p, masks);     // without one it changes nothing
                        }
                        // (kept in the accumulators for a store behind them all, under these tests, they would take twice the registers)
                        if (lin.codes == nullptr) {
                            float *dst = C + (size_t)row * ldc + col;
                            if (!kCut || left >= 4) {
                                *reinterpret_cast<u32x4u *>(dst) = u32x4u{t[0], t[1], t[2], t[3]};
                            } else {
                                dst[0] = __uint_as_float(t[0]);
                                if (left > 1) dst[1] = __uint_as_float(t[1]);
                                if (left > 2) dst[2] = __uint_as_float(t[2]);
                            }
                        } else {
#pragma unroll
                            for (int c = 0; c < 4; ++c) t[c] = MODE == kModeInteger ? t[c] >> p.shift : encode_bits<MODE>(t[c], p);     // e == 8: the upper bits
                            uint16_t *dst = lin.codes + (size_t)row * lin.ldcodes + col;
                            if (!kCut || left >= 4) {
                                *reinterpret_cast<u32x2u *>(dst) = u32x2u{t[0] | (t[1] << 16), t[2] | (t[3] << 16)};
                            } else {
                                dst[0] = (uint16_t)t[0];
                                if (left > 1) dst[1] = (uint16_t)t[1];
                                if (left > 2) dst[2] = (uint16_t)t[2];
                            }
                        }
                    }
                }
        };
        constexpr std::integral_constant<int, kModeMagic> magic{};
        constexpr std::integral_constant<int, kModeInteger> integer{};
        if (PS == 0 || p.mode == kModeMagic) {
            if (lin.ftz) run(magic, std::true_type{});
            else run(magic, std::false_type{});
        } else {
            if (lin.ftz) run(integer, std::true_type{});
            else run(integer, std::false_type{});
        }
    } else {
        // The wave's own block: a lane takes the same four columns of every kRows-th row, kAhead rows at a time.  A layer whose
        // outputs are all NaN, 4096 x 3072 x 1024 in 1/8/7: 47 us (others 40; 81 with one element and one load at a time).
        store_tile<TM, TN, false>(acc, C, ldc, M, N, 0, row_base, col_base, lane, nullptr, nullptr);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        constexpr int kRows = 64 / (8 * TN), kAhead = 4;
        const int col = col_base + lane % (8 * TN) * 4, left = N - col;
        auto run = [&](auto mode, auto flush) __attribute__((always_inline)) {
            constexpr int MODE = decltype(mode)::value;
            constexpr bool FTZ = decltype(flush)::value;
            uint32_t rb[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) rb[c] = has_bias && c < left ? quantize_bits<MODE, FTZ>(__float_as_uint(lin.bias[col + c]), p) : 0u;
#pragma unroll 1
            for (int r0 = row_base + lane / (8 * TN); r0 < row_base + 32 * TM; r0 += kRows * kAhead) {
                u32x4u u[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const uint32_t *src = reinterpret_cast<const uint32_t *>(C) + (size_t)(r0 + q * kRows) * ldc + col;
                    const bool in = r0 + q * kRows < M;
                    u[q] = u32x4u{0u, 0u, 0u, 0u};
                    if (in && left >= 4) {
                        u[q] = *reinterpret_cast<const u32x4u *>(src);
                    } else if (in) {
                        if (left > 0) u[q][0] = src[0];
                        if (left > 1) u[q][1] = src[1];
                        if (left > 2) u[q][2] = src[2];
                    }
                }
#pragma unroll 1
                for (int q = 0; q < kAhead; ++q) {
                    const int row = r0 + q * kRows;
                    uint32_t t[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        t[c] = quantize_bits<MODE, FTZ>(u[0][c], p);
                        if (has_bias) t[c] = __float_as_uint(__fadd_rn(__uint_as_float(t[c]), __uint_as_float(rb[c])));
                        if constexpr (HIST) account<false, kCopies>(t[c] & 0x7FFFFFFFu, row < M && c < left, p, tbl, copy, w);
                        if (has_bias) t[c] = quantize_bits<MODE, FTZ>(t[c], p);
                    }
                    u[0] = u[1], u[1] = u[2], u[2] = u[3];
                    if (row >= M) continue;
                    if (lin.codes == nullptr) {
                        uint32_t *dst = reinterpret_cast<uint32_t *>(C) + (size_t)row * ldc + col;
                        if (left >= 4) {
                            *reinterpret_cast<u32x4u *>(dst) = u32x4u{t[0], t[1], t[2], t[3]};
                        } else {
                            if (left > 0) dst[0] = t[0];
                            if (left > 1) dst[1] = t[1];
                            if (left > 2) dst[2] = t[2];
                        }
                    } else {
                        uint16_t *dst = lin.codes + (size_t)row * lin.ldcodes + col;
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (c < left) dst[c] = (uint16_t)encode_bits<MODE>(t[c], p);
                    }
                }
            }
        };
        constexpr std::integral_constant<int, kModeMagic> magic{};
        constexpr std::integral_constant<int, kModeInteger> integer{};
        if (PS == 0 || p.mode == kModeMagic) {
            if (lin.ftz) run(magic, std::true_type{});
            else run(magic, std::false_type{});
        } else {
            if (lin.ftz) run(integer, std::true_type{});
            else run(integer, std::false_type{});
        }
    }
    if constexpr (HIST) {
        hist_clear<256>(sink, (uint32_t)tile, (uint32_t)ntiles, tid);
        hist_end<kCopies, 256>(tbl, s_bins, s_cls, w, p, sink, (uint32_t)tile, (uint32_t)ntiles, tid);
    }
}

// Convolutions on exponent planes with one scale per tensor (formats with e == 6, m = 8 or 9): the products that meet an element outside
// plane 0 are added to the sums of plane 0, block of 32 k by block, by the wave that owns the results.  Which blocks those are is read
// from the operands' masks, a lane per block, for the first kWindowChunks * 64 blocks under the first stages' loads.  Of 3.2 M gradients with
// log2|x| ~ N(-20, 5^2) 43 lie outside, of activations and weights none, so the loops here are short and wait for memory: what bounds them
// is the wave that has most to do.  Each pair of planes has a scale of its own, 2^up, and a batch of blocks of one pair is summed apart and
// then added as 2^-up of it.  (The running sums cannot be brought to the pair's scale instead: up reaches 2 w = 64 with m = 8, and sums that
// another pair has raised to 2^64 and more in plane 0's units would overflow on the way.)  Nothing overflows or is lost on this one: a batch is a
// multiple of 2^-48 below 2^32 * 32 kAhead, so 2^-up of it lies between 2^-112 and 2^104, and the sums are at most 2^64 K in the values' own
// units, 2^94 K in plane 0's.  The order is fixed, so the results are the
// same on every run.  256 -> 256 channels of 14 x 14, 3 x 3 taps, batch 64: the
// dgrad kernel takes 30 us on gradients without such elements, 36 with one and 45 with 43 (the code is met for the first time then, so
// larger batches or fewer instructions on the common path did not help; reading the masks after the products cost 2 more).
constexpr int kWindowChunks = 2;
// Tiles of 128 x 128 and 64 x 64: with the tail the larger ones do not fit the registers.  256 x 256 spilled 2.5 KB per lane and took
// 2 to 5 times as long: 36 x 288 x 27 x 27 -> 480 channels, dgrad, 1 x 1, 170 us against 46, forward of 73 x 64 x 41 x 41 -> 160, 3 x 3, 443 against 90.
// Workgroups that a compute unit takes: LDS leaves room for two and four, and the tail's registers must not take it.
constexpr int window_workgroups(int tiles) { return tiles == 4 ? 2 : 4; }

// Bits 1 and 2: operand A has elements of the planes above / below in this wave's rows and block kb; bits 9 and 10: operand B.
template <int TM, int TN, bool GATHER>
__device__ __forceinline__ uint32_t window_masks(const Planes &pa, const Planes &pb, const Implicit &im, int kblocks, int kb, int kb1, int unit_a,
                                                 int unit_b)
{
    if (kb >= kb1) return 0u;
    uint32_t ma = 0u, mb = 0u;
#pragma unroll
    for (int i = 0; i < TM; ++i) ma |= pa.mask[(size_t)(unit_a + i) * kblocks + kb];
    if constexpr (GATHER) {
        if (unit_b * kUnitRows >= im.rows) return 0u;                // no positions: nothing is stored
        const unsigned long long *pixels = reinterpret_cast<const unsigned long long *>(pb.mask);
        int t, x, n0, n1, y0, y1, tap, cb, r, s2;
        divmod(im.r0, unit_b * kUnitRows, t, x);
        divmod(im.r1, t, n0, y0);
        divmod(im.r0, min((unit_b + TN) * kUnitRows, im.rows) - 1, t, x);
        divmod(im.r1, t, n1, y1);
        divmod(im.kc, kb, tap, cb);
        divmod(im.ks, tap, r, s2);
        y0 = y0 * im.mul_y + im.off_y + im.tap_sign * r;
        y1 = y1 * im.mul_y + im.off_y + im.tap_sign * r;
        // the pixels that the positions reach lie between the first of the first one's row and the last of the last one's
        const int lo = (n0 * im.th + min(max(y0, 0), im.th - 1)) * im.tw, hi = (n1 * im.th + min(max(y1, 0), im.th - 1)) * im.tw + im.tw - 1;
        for (int q0 = lo / 64; q0 <= hi / 64; q0 += 3) {
            unsigned long long w[3][2];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b) w[i][b] = pixels[((size_t)min(q0 + i, hi / 64) * (im.c8 / 4) + cb) * 2 + b];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int q = min(q0 + i, hi / 64);
                const unsigned long long within = (~0ull << max(lo - q * 64, 0)) & (~0ull >> max(q * 64 + 63 - hi, 0));
                mb |= ((w[i][0] & within) != 0ull ? 2u : 0u) | ((w[i][1] & within) != 0ull ? 4u : 0u);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) mb |= pb.mask[(size_t)(unit_b + j) * kblocks + kb];
    }
    return (ma & 6u) | ((mb & 6u) << 8);
}

template <int TM, int TN, bool GATHER>
__device__ __forceinline__ void window_tail(floatx16 (&acc)[TM][TN], const uint32_t (&early)[kWindowChunks], const u32x4 *__restrict__ Aw,
                                            const u32x4 *__restrict__ Bw, const Planes &pa, const Planes &pb, const Implicit &im, int kblocks,
                                            int kb0, int kb1, int unit_a, int unit_b, int lane)
{
    // blocks loaded together: an element outside plane 0 of a gathered tensor is met by every tap (as many as leave the
    // 64 x 64 and 128 x 128 tiles their four and two workgroups per compute unit)
    constexpr int kAhead = 4;
    const unsigned long long *pixels = reinterpret_cast<const unsigned long long *>(pb.mask);      // GATHER (see fmt_product.h)
#pragma unroll 1
    for (int first = kb0; first < kb1; first += 64) {
        const int mine = first + lane, chunk = (first - kb0) / 64;
        uint32_t masks = chunk == 0 ? early[0] : early[1];
        static_assert(kWindowChunks == 2, "early");
        if (chunk >= kWindowChunks) masks = window_masks<TM, TN, GATHER>(pa, pb, im, kblocks, mine, kb1, unit_a, unit_b);
        if (__ballot(masks != 0u) == 0ull) continue;
        const uint32_t ma = (masks & 255u) | 1u, mb = (masks >> 8) | 1u;
        int pn[TN], py[TN], px[TN];                                  // GATHER: corner pixels (columns beyond the matrix are not stored)
        if constexpr (GATHER) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                int t, x;
                divmod(im.r0, min((unit_b + j) * kUnitRows + (lane & 31), im.rows - 1), t, x);
                divmod(im.r1, t, pn[j], py[j]);
                py[j] = py[j] * im.mul_y + im.off_y;
                px[j] = x * im.mul_x + im.off_x;
            }
        }
#pragma unroll 1
        for (int pair = 1; pair < 9; ++pair) {                       // (0, 0) is in the sums
            const int qa = pair / 3, qb = pair % 3;                  // planes: 0, above, below
            unsigned long long todo = __ballot(mine < kb1 && ((ma >> qa) & (mb >> qb) & 1u) != 0u);
            if (todo == 0ull) continue;
            // scales above and below plane 0's: 2^-w, 2^w
            const int up = (qa == 0 ? 0 : qa == 1 ? -pa.w : pa.w) + (qb == 0 ? 0 : qb == 1 ? -pb.w : pb.w);
            const float down = ldexpf(1.0f, -up);
#pragma unroll 1
            while (todo != 0ull) {
                int block = 0;
                u32x4 fa[kAhead][2][TM], fb[kAhead][2][TN];
#pragma unroll
                for (int d = 0; d < kAhead; ++d) {
                    const bool some = d == 0 || todo != 0ull;        // the same in the whole wave; without: the block before again, times zero
                    if (some) block = first + __builtin_ctzll(todo);
                    todo &= todo - 1ull;
                    // what is not in the plane is loaded all the same, beside the mask, and left out
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const size_t unit = (size_t)(unit_a + i) * kblocks + block;
#pragma unroll
                        for (int kk = 0; kk < 2; ++kk) fa[d][kk][i] = Aw[qa * pa.plane + unit * kUnitVec + kk * 64 + lane];
                        if (qa != 0 && !((pa.mask[unit] >> qa) & 1u)) fa[d][0][i] = fa[d][1][i] = u32x4{0u, 0u, 0u, 0u};
                    }
                    int tap = 0, cb = 0, r = 0, s2 = 0;
                    if constexpr (GATHER) {
                        divmod(im.kc, block, tap, cb);
                        divmod(im.ks, tap, r, s2);
                    }
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        if constexpr (GATHER) {
                            const int iy = py[j] + im.tap_sign * r, ix = px[j] + im.tap_sign * s2, pix = (pn[j] * im.th + iy) * im.tw + ix;
                            const bool in = (unsigned)iy < (unsigned)im.th && (unsigned)ix < (unsigned)im.tw;
#pragma unroll
                            for (int kk = 0; kk < 2; ++kk)
                                fb[d][kk][j] = im.T[in ? qb * im.piece_vec + pix * im.c8 + cb * 4 + kk * 2 + (lane >> 5) : im.zero];
                            if (!some || (qb != 0 && in && !((pixels[((size_t)(pix / 64) * (im.c8 / 4) + cb) * 2 + (qb - 1)] >> (pix % 64)) & 1ull)))
                                fb[d][0][j] = fb[d][1][j] = u32x4{0u, 0u, 0u, 0u};
                        } else {
                            const size_t unit = (size_t)(unit_b + j) * kblocks + block;
#pragma unroll
                            for (int kk = 0; kk < 2; ++kk) fb[d][kk][j] = Bw[qb * pb.plane + unit * kUnitVec + kk * 64 + lane];
                            if (!some || (qb != 0 && !((pb.mask[unit] >> qb) & 1u))) fb[d][0][j] = fb[d][1][j] = u32x4{0u, 0u, 0u, 0u};
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        floatx16 t = {};
#pragma unroll
                        for (int d = 0; d < kAhead; ++d)
#pragma unroll
                            for (int kk = 0; kk < 2; ++kk)
                                t = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fb[d][kk][j]),
                                                                           __builtin_bit_cast(f16x8, fa[d][kk][i]), t, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[i][j][v] = fmaf(t[v], down, acc[i][j][v]);
                    }
            }
        }
    }
    const float unit = ldexpf(1.0f, -(pa.S[0] + pb.S[0]));
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] *= unit;
}

// A stage buffer, by its place in the ring, that the two bodies of a kernel that holds planes and pieces (product_kernel) have in common.
template <int PLACE, int VECTORS>
__device__ __forceinline__ auto stage_buffer() -> u32x4 (&)[VECTORS]
{
    __shared__ u32x4 vectors[VECTORS];
    return vectors;
}

// product: Aw / Bw are prepared operands (rows padded to a multiple of kRowPad, k to a multiple
// of 32).  A workgroup is 2 x 2 waves; each wave owns TM x TN MFMA tiles of 32 x 32, so the
// workgroup tile is (64*TM) x (64*TN).  Operand stages of KS*16 k go from global memory straight
// into LDS (global_load_lds, 16 bytes per lane) through a ring of NST stage buffers, one barrier
// per stage.  With SPLIT the k range is cut into parts and each part writes its own M x N slab
// of partial sums (summed by reduce_kernel).
// SCALED (single fp16 piece only): the operands are exponent planes with per-row power-of-two scales
// (pa.S / pb.S), undone on the way out; this kernel multiplies plane 0 by plane 0, planes_tail_kernel
// adds the products of the elements that live in the other planes.
// GATHER: operand B is not a prepared operand but a rounded convolution tensor in pixel-major order (`im`,
// Bw unused): a lane's 16-byte load of (position, 8 consecutive k) is 8 consecutive channels of one pixel,
// whose address is a per-lane base (the position's corner pixel) plus a per-stage term (the tap and the
// channel block), or the zero vector where the tap falls outside the tensor (a per-lane bit mask over
// the taps).  The stage image in LDS and everything after it are the same.
// The body is shared by the kernel of one product (bid = blockIdx.x) and the kernel of a group of products
// (bid = the workgroup's index within its product).
// WINDOW (single fp16 piece, plain or GATHER): exponent planes with one scale per operand (window_tail).
// LINEAR: the results are a fully connected layer's accumulators; they leave as R(R(acc) + R(b)) (lin), HIST: with the
// statistics of R(acc) + R(b) (sink).
template <int PS, int TM, int TN, int KS, int NST, bool SPLIT, bool SCHED, bool SCALED, bool GATHER = false, bool LINEAR = false,
          bool HIST = false, bool WINDOW = false, bool COMMON = WINDOW>
__device__ __forceinline__ void product_body(const u32x4 *__restrict__ Aw, const u32x4 *__restrict__ Bw,
                                             float *__restrict__ C, int M, int N, int64_t ldc, int img,
                                             int kblocks, int tiles_m, int tiles_n, int kb_per_split,
                                             const Planes &pa, const Planes &pb, const Implicit &im, const unsigned bid,
                                             const LinearOut &lin = LinearOut{}, const HistSink &sink = HistSink{})
{
    constexpr int P = pieces_of(PS);
    constexpr int UA = 2 * TM, UB = 2 * TN;              // 32-row units per operand in the workgroup tile
    constexpr int kHalf = 64;                            // vectors of one piece of one unit per 16 k
    constexpr int SV = kHalf * KS;                       // ... per stage
    constexpr int VA = UA * P * SV, VB = UB * P * SV;    // 16-byte vectors per operand per stage
    constexpr int LA = (VA + 255) / 256, LB = (VB + 255) / 256;   // loads per lane per stage
    // Loads of a wave that may still be in flight when a stage is read, which is the oldest of NST (the first) or NST - 1.  Where an
    // operand's stage is not a whole number of loads per wave (three pieces: 384 vectors of a 64-row operand), the upper waves issue
    // fewer than LA + LB; counting those of the last wave for every wave (j * 256 + 192 < VA), no wait ends before the wave's own loads
    // of the stage have landed.
    constexpr int kFewest = (VA + 63) / 256 + (VB + 63) / 256;
    constexpr int kWaitFirst = (NST - 1) * kFewest, kWaitLanded = (NST - 2) * kFewest;
    static_assert(kWaitFirst < 64 && (KS == 1 || KS == 2) && NST >= 2 && NST <= 4, "unsupported pipeline shape");
    // One LDS array per stage buffer, each addressed with a compile-time index: the compiler then knows
    // which loads-to-LDS an LDS read can depend on and leaves the younger stages in flight.
    constexpr int STV = VA + VB;
    // (References to these would cost registers: three pieces, 64 x 64, five workgroups per compute unit instead of six, 1 - 4 %.)
    __shared__ u32x4 st0[STV];
    __shared__ u32x4 st1[STV];
    __shared__ u32x4 st2[NST > 2 ? STV : 1];
    __shared__ u32x4 st3[NST > 3 ? STV : 1];
    auto stage = [&](int b) -> u32x4 * {
        if constexpr (COMMON)
            return b == 0 ? stage_buffer<0, STV>() : b == 1 ? stage_buffer<1, STV>() : b == 2 ? stage_buffer<2, (NST > 2 ? STV : 1)>() : stage_buffer<3, (NST > 3 ? STV : 1)>();
        else
            return b == 0 ? st0 : b == 1 ? st1 : b == 2 ? st2 : st3;
    };
    typedef __attribute__((address_space(3))) void lds_void;
    typedef const __attribute__((address_space(1))) void glb_void;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // Workgroup -> (tile, k part).  Consecutive workgroup ids go to different XCDs (8 of them,
    // each with its own L2), so ids are remapped to give every XCD a contiguous run of tiles.
    const int ntiles = tiles_m * tiles_n;
    const int per_xcd = (ntiles + 7) / 8;
    const int wg = (int)(bid % (unsigned)(per_xcd * 8));
    const int split = (int)(bid / (unsigned)(per_xcd * 8));
    const int tile = (wg % 8) * per_xcd + wg / 8;
    if (tile >= ntiles) return;
    // Within the run, tiles are walked in groups of kGroup tile rows, column by column, so that
    // the 32 tiles an XCD works on at a time cover few distinct operand panels.
    constexpr int kGroup = 16 / TM;                      // 1024 rows of op(A) per group
    const int per_group = kGroup * tiles_n;
    const int group = tile / per_group, in_group = tile % per_group;
    const int rows_here = min(kGroup, tiles_m - group * kGroup);
    const int tm = group * kGroup + in_group % rows_here, tn = in_group / rows_here;
    const int kb0 = SPLIT ? split * kb_per_split : 0;
    const int kb1 = SPLIT ? min(kblocks, kb0 + kb_per_split) : kblocks;
    const int steps = (kb1 - kb0) * (2 / KS);            // stages to consume

    // Stage image per operand = [unit row-block][piece][SV vectors]; in the workspace a unit's
    // piece is 128 vectors (two 16-k halves) and row-blocks are kblocks*P*128 vectors apart.
    const size_t rb_stride = (size_t)kblocks * P * kUnitVec;
    const u32x4 *ga[LA], *gb[LB];
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        const int q = min(j * 256 + tid, VA - 1);
        const int rbl = q / (P * SV), piece = (q % (P * SV)) / SV, v = q % SV;
        ga[j] = Aw + ((size_t)tm * UA + rbl) * rb_stride + (size_t)kb0 * P * kUnitVec + piece * kUnitVec + v;
    }
    int gbase[GATHER ? LB : 1];          // GATHER: vector index of the position's corner pixel (+ piece, + k chunk)
    uint32_t gmask[GATHER ? LB : 1];     // ... and the taps that fall inside the tensor
#pragma unroll
    for (int j = 0; j < LB; ++j) {
        const int q = min(j * 256 + tid, VB - 1);
        const int rbl = q / (P * SV), piece = (q % (P * SV)) / SV, v = q % SV;
        if constexpr (GATHER) {
            const int row = (tn * UB + rbl) * kUnitRows + v % kUnitRows;
            int x, t, y, n;
            divmod(im.r0, min(row, im.rows - 1), t, x);
            divmod(im.r1, t, n, y);
            const int by = y * im.mul_y + im.off_y, bx = x * im.mul_x + im.off_x;
            uint32_t mq = 0u;
            int tap = 0;
            for (int r = 0; r < im.R; ++r)
                for (int s2 = 0; s2 < im.S; ++s2, ++tap) {
                    const int iy = by + im.tap_sign * r, ix = bx + im.tap_sign * s2;
                    if ((unsigned)iy < (unsigned)im.th && (unsigned)ix < (unsigned)im.tw) mq |= 1u << tap;
                }
            gmask[j] = row < im.rows ? mq : 0u;
            gbase[j] = piece * im.piece_vec + ((n * im.th + by) * im.tw + bx) * im.c8 + v / kUnitRows;
            gb[j] = im.T;
        } else {
            gb[j] = Bw + ((size_t)tn * UB + rbl) * rb_stride + (size_t)kb0 * P * kUnitVec + piece * kUnitVec + v;
        }
    }

    // a layer's bias, loaded ahead of the products: register v of a lane holds column 8*(v/4) + 4*(l/32) + v%4 (see store_tile)
    uint32_t bias[LINEAR ? TN : 1][LINEAR ? 16 : 1];
    auto load_bias = [&]() __attribute__((always_inline)) {
        if constexpr (LINEAR) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    bias[j][v] = linear_bias(lin, (tn * 2 + wn) * (32 * TN) + j * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3), N);
        }
    };
    load_bias();

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // Loads of stage t (clamped to the last one, so that the number of loads in flight is the
    // same in every trip; a clamped load lands in a buffer nobody reads any more).
    auto issue = [&](int t, int buf) {
        const int tc = min(t, steps - 1);
        u32x4 *sa = stage(buf), *sb = sa + VA;
        const size_t off = KS == 2 ? (size_t)tc * P * kUnitVec : (size_t)(tc >> 1) * P * kUnitVec + (tc & 1) * kHalf;
#pragma unroll
        for (int j = 0; j < LA; ++j)
            if (VA % 256 == 0 || j * 256 + wave * 64 < VA)
                __builtin_amdgcn_global_load_lds((glb_void *)(ga[j] + off), (lds_void *)(sa + j * 256 + wave * 64), 16, 0, 0);
        if constexpr (GATHER) {
            // stage number (in stages of 16*KS k) -> tap and channel block: the same in the whole workgroup
            int tap, cb, r, s2;
            divmod(im.kc, kb0 * (2 / KS) + tc, tap, cb);
            divmod(im.ks, tap, r, s2);
            const int toff = im.tap_sign * (r * im.tw + s2) * im.c8 + cb * (2 * KS);
#pragma unroll
            for (int j = 0; j < LB; ++j)
                if (VB % 256 == 0 || j * 256 + wave * 64 < VB) {
                    const int at = ((gmask[j] >> tap) & 1u) ? gbase[j] + toff : im.zero;
                    __builtin_amdgcn_global_load_lds((glb_void *)(im.T + at), (lds_void *)(sb + j * 256 + wave * 64), 16, 0, 0);
                }
        } else {
#pragma unroll
            for (int j = 0; j < LB; ++j)
                if (VB % 256 == 0 || j * 256 + wave * 64 < VB)
                    __builtin_amdgcn_global_load_lds((glb_void *)(gb[j] + off), (lds_void *)(sb + j * 256 + wave * 64), 16, 0, 0);
        }
    };

    // Operand fragments live in two register sets: while the MFMAs of stage t run on one, the LDS
    // reads of stage t + 1 fill the other, so that no MFMA waits for LDS latency (a workgroup tile
    // of 128 x 128 has one wave per SIMD and nothing else to run meanwhile).
    bf16x8 fa[2][KS][TM][P], fb[2][KS][TN][P];
    auto read_frags = [&](int buf, int set) __attribute__((always_inline)) {
        const u32x4 *sa = stage(buf), *sb = sa + VA;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < P; ++q)
                    fa[set][kk][i][q] = __builtin_bit_cast(bf16x8, sa[((wm * TM + i) * P + q) * SV + kk * kHalf + lane]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < P; ++q)
                    fb[set][kk][j][q] = __builtin_bit_cast(bf16x8, sb[((wn * TN + j) * P + q) * SV + kk * kHalf + lane]);
        }
    };
    // The barrier is the bare instruction behind the waits it needs (this wave's LDS reads retired,
    // its stage landed): __syncthreads() would also wait for every load-to-LDS still in flight.
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    [[maybe_unused]] uint32_t early[kWindowChunks] = {0u, 0u};
    // Tensors that span more than a plane have been prepared as two bf16 pieces (window_pair).  The first stages' loads are issued before
    // that is known: S comes out of the memory behind another XCD's L2.
    [[maybe_unused]] int in_pieces = 0;
    if constexpr (WINDOW) in_pieces = pa.S[1];
    if (steps > 0) {
#pragma unroll
        for (int t = 0; t < NST; ++t) issue(t, t);
        if constexpr (WINDOW) {
#pragma unroll
            for (int c = 0; c < kWindowChunks; ++c)
                early[c] = window_masks<TM, TN, GATHER>(pa, pb, im, kblocks, kb0 + c * 64 + lane, kb1, tm * UA + wm * TM, tn * UB + wn * TN);
            if (__builtin_amdgcn_readfirstlane(in_pieces) != 0) {    // the same in the whole launch
                // twice the bytes per k, so the same stages in half as many k; the buffers are the same
                typedef Pipe<2, TM, TN> Pieces;
                static_assert(Pieces::nst == NST && 2 * Pieces::ks == KS, "stages of the same bytes");
                __builtin_amdgcn_s_waitcnt(0x0F70);
                barrier();
                Implicit imp = im;
                imp.kc = fastdiv_twice(im.kc);
                product_body<2, TM, TN, Pieces::ks, Pieces::nst, SPLIT, SCHED, false, GATHER, false, false, false, true>(
                    Aw, Bw, C, M, N, ldc, img, kblocks, tiles_m, tiles_n, kb_per_split, pa, pb, imp, bid);
                return;
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70 | (kWaitFirst & 0xF) | ((kWaitFirst >> 4) << 14));
        barrier();
        read_frags(0, 0);
    }
    // Trip t: stage t is in register set `cur`; stage t + 1 (buffer b + 1) is read into the other set
    // and stage t + NST is loaded into buffer b, which every wave has finished reading once it is past
    // the barrier.  The trips are unrolled over the ring and the two register sets, so that buffer and
    // set are compile-time constants, and the loop over whole turns has a single exit (with early
    // exits the compiler falls back to waiting for all loads at the loop head); the remaining trips
    // follow it.
    auto trip = [&](int t, int b, int cur) __attribute__((always_inline)) {
        // stage t + 1 has landed once at most the loads of the NST-2 younger stages are in flight
        __builtin_amdgcn_sched_barrier(0);       // MFMAs are not memory operations: without this they drift across the barrier
        __builtin_amdgcn_s_waitcnt(0x0F70 | (kWaitLanded & 0xF) | ((kWaitLanded >> 4) << 14));
        barrier();                               // ... for every wave; and every wave holds stage t in registers
        read_frags((b + 1) % NST, cur ^ 1);
        issue(t + NST, b);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int qa = 0; qa < P; ++qa)
#pragma unroll
                        for (int qb = 0; qb < P; ++qb)
                            // B's fragment first: the block comes out transposed (see store_tile)
                            acc[i][j] = PS == 0 ? __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fb[cur][kk][j][qb]),
                                                                                         __builtin_bit_cast(f16x8, fa[cur][kk][i][qa]),
                                                                                         acc[i][j], 0, 0, 0)
                                                : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][kk][j][qb], fa[cur][kk][i][qa], acc[i][j], 0, 0, 0);
        }
        // Issue order inside one trip: the next stage's LDS reads, then its global loads, threaded
        // between the MFMAs so that they issue in the MFMAs' shadow.
        if constexpr (SCHED) {
            constexpr int kMfma = TM * TN * P * P * KS, kReads = (TM + TN) * P * KS, kLoads = LA + LB;
            constexpr int kDsEach = (kReads + kMfma - 1) / kMfma;            // LDS reads behind each of the first MFMAs
            constexpr int kPairs = (kReads + kDsEach - 1) / kDsEach;
#pragma unroll
            for (int r = 0; r < kPairs; ++r) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, kDsEach, 0);
            }
            constexpr int kLeft = kMfma - kPairs;                            // MFMAs left for the global loads
            if constexpr (kLeft > kLoads) {
                constexpr int kPer = kLeft / (kLoads + 1);
#pragma unroll
                for (int r = 0; r < kLoads; ++r) {
                    __builtin_amdgcn_sched_group_barrier(0x008, kPer, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
            } else if constexpr (kLeft > 0) {
                constexpr int kEach = (kLoads + kLeft - 1) / kLeft;
#pragma unroll
                for (int r = 0; r < kLeft; ++r) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, kEach, 0);
                }
            } else {
                __builtin_amdgcn_sched_group_barrier(0x020, kLoads, 0);
            }
        }
    };
    constexpr int kTurn = NST % 2 == 0 ? NST : 2 * NST;      // trips after which buffer and register set repeat
    int t0 = 0;
    for (; t0 + kTurn <= steps; t0 += kTurn) {
#pragma unroll
        for (int u = 0; u < kTurn; ++u) trip(t0 + u, u % NST, u & 1);
    }
#pragma unroll
    for (int u = 0; u < kTurn - 1; ++u)
        if (t0 + u < steps) trip(t0 + u, u % NST, u & 1);
    // every load-to-LDS of this wave must have landed before the workgroup's LDS is handed back
    __builtin_amdgcn_s_waitcnt(0x0F70);

    if constexpr (LINEAR) {
        static_assert(sizeof(st0) >= kHistRows * linear_copies(TM * TN) * 4, "room for the statistics' table");
        const int row_base = (tm * 2 + wm) * (32 * TM), col_base = (tn * 2 + wn) * (32 * TN);
        if constexpr (SCALED) {
            unscale_tile<TM, TN>(acc, row_base, col_base, lane, pa.S, pb.S);
            // Elements outside plane 0 in the rows or columns of the tile: their products are added ahead of the roundings.
            uint32_t any = 0u;
#pragma unroll
            for (int u = 0; u < UA; ++u) any |= pa.rec_cnt[tm * UA + u];
#pragma unroll
            for (int u = 0; u < UB; ++u) any |= pb.rec_cnt[tn * UB + u];
            if (__builtin_amdgcn_readfirstlane((int)any) != 0) {
                // The stage buffers serve again: the sums take the last ones, kRows rows each; the records take the first where it is
                // left and holds them.
                constexpr int kRows = STV * 16 / (64 * TN * 4), kUsed = (64 * TM + kRows - 1) / kRows;
                static_assert(kUsed <= NST && NST > 2, "room for the sums");
                constexpr bool kFits = kUsed < NST && sizeof(st0) >= sizeof(TailLds);
                __shared__ __attribute__((aligned(16))) char s_tail[kFits ? 16 : sizeof(TailLds)];
                typedef float f32x4 __attribute__((ext_vector_type(4)));
                TailTile<TM, TN, kRows> tile_sums;
#pragma unroll
                for (int q = 0; q < 4; ++q) tile_sums.s[q] = (lds_ptr<float>)reinterpret_cast<char *>(stage(q < kUsed ? NST - kUsed + q : 0));
                auto quads = [&](auto &&move) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
#pragma unroll
                            for (int g = 0; g < 4; ++g)
                                move(i, j, g, (lds_ptr<f32x4>)tile_sums.at((wm * TM + i) * 32 + (lane & 31), (wn * TN + j) * 32 + g * 8 + (lane >> 5) * 4));
                };
                __syncthreads();                 // every wave is done with the stage buffers
                quads([&](int i, int j, int g, lds_ptr<f32x4> at) __attribute__((always_inline)) {
                    *at = f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                });
                __syncthreads();
                tail_tile<TM, TN, kRows>(Aw, Bw, pa, pb, kblocks, tm, tn, tile_sums, (lds_ptr<TailLds>)(kFits ? reinterpret_cast<char *>(st0) : s_tail));
                quads([&](int i, int j, int g, lds_ptr<f32x4> at) __attribute__((always_inline)) {
                    const f32x4 v = *at;
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[i][j][4 * g + c] = v[c];
                });
                load_bias();                     // again: nothing is kept in registers over the call
            }
        }
        linear_tile<PS, TM, TN, HIST>(acc, C, ldc, M, N, row_base, col_base, lane, bias, lin, sink, reinterpret_cast<uint32_t *>(st0), tile, ntiles);
        return;
    }
    if constexpr (WINDOW) {
        static_assert(PS == 0 && KS == 2 && !SCALED, "one fp16 plane, a block of 32 k per stage");
        window_tail<TM, TN, GATHER>(acc, early, Aw, Bw, pa, pb, im, kblocks, kb0, kb1, tm * UA + wm * TM, tn * UB + wn * TN, lane);
    }
    // plain: C[row][col] with leading dimension ldc; a part of a split k: its own M x N slab; img > 0: NCHW
    float *out = SPLIT ? C + (size_t)split * M * ldc : C;
    store_tile<TM, TN, SCALED>(acc, out, ldc, M, N, SPLIT ? 0 : img, (tm * 2 + wm) * (32 * TM), (tn * 2 + wn) * (32 * TN), lane, pa.S,
                               pb.S);
}

template <int PS, int TM, int TN, int KS, int NST, bool SPLIT, bool SCHED, bool SCALED, bool GATHER = false, bool WINDOW = false>
__global__ __launch_bounds__(256, WINDOW ? window_workgroups(TM * TN) : 1) void product_kernel(const u32x4 *__restrict__ Aw, const u32x4 *__restrict__ Bw,
                                                      float *__restrict__ C, int M, int N, int64_t ldc, int img,
                                                      int kblocks, int tiles_m, int tiles_n, int kb_per_split,
                                                      Planes pa, Planes pb, Implicit im)
{
    product_body<PS, TM, TN, KS, NST, SPLIT, SCHED, SCALED, GATHER, false, false, WINDOW>(Aw, Bw, C, M, N, ldc, img, kblocks, tiles_m, tiles_n,
                                                                                        kb_per_split, pa, pb, im, blockIdx.x);
}

template <int PS, int TM, int TN, int KS, int NST, bool SCALED, bool HIST>
__global__ __launch_bounds__(256, SCALED ? (TM * TN == 4 ? 2 : 3) : 1) void product_linear_kernel(const u32x4 *__restrict__ Aw, const u32x4 *__restrict__ Bw,
                                                             float *C, int M, int N, int64_t ldc, int kblocks,
                                                             int tiles_m, int tiles_n, Planes pa, Planes pb, LinearOut lin, HistSink sink)
{
    product_body<PS, TM, TN, KS, NST, false, true, SCALED, false, true, HIST>(Aw, Bw, C, M, N, ldc, 0, kblocks, tiles_m, tiles_n, kblocks, pa,
                                                                            pb, Implicit{}, blockIdx.x, lin, sink);
}

template <int PS, int TM, int TN, int KS, int NST, bool SCHED, bool SCALED>
__global__ __launch_bounds__(256) void product_group_kernel(Group grp)
{
    const GroupItem &it = grp.p[group_member(grp.first, blockIdx.x)];      // the same in the whole workgroup
    product_body<PS, TM, TN, KS, NST, true, SCHED, SCALED, false>(it.Aw, it.Bw, it.C, it.M, it.N, it.ldc, 0, it.kblocks, it.tiles_m,
                                                                it.tiles_n, it.kb_per_part, it.pa, it.pb, Implicit{},
                                                                blockIdx.x - it.first);
}

template <int PS, int TM, int TN, bool SPLIT, bool SCHED, bool SCALED, bool GATHER = false, bool WINDOW = false>
static int launch_product_v2(const u32x4 *Aw, const u32x4 *Bw, float *out, int M, int N, int64_t ld, int img, int kblocks,
                            int nsplit, hipStream_t stream, const Planes &pa, const Planes &pb, const Implicit &im = Implicit{})
{
    constexpr int KS = Pipe<PS, TM, TN>::ks, NST = Pipe<PS, TM, TN>::nst;
    if constexpr (lds_bytes(TM, TN, pieces_of(PS), KS, NST) > 160 * 1024) {
        return FMT_ERR_SHAPE;                            // never planned (make_plan skips such tiles)
    } else {
        const int tiles_m = (M + 64 * TM - 1) / (64 * TM), tiles_n = (N + 64 * TN - 1) / (64 * TN);
        const int64_t per_xcd = ((int64_t)tiles_m * tiles_n + 7) / 8;
        if (per_xcd * 8 * nsplit >= ((int64_t)1 << 31)) return FMT_ERR_SHAPE;
        const int kb_per = (kblocks + nsplit - 1) / nsplit;
        auto kern = product_kernel<PS, TM, TN, KS, NST, SPLIT, SCHED, SCALED, GATHER, WINDOW>;
        Implicit imk = im;
        if (GATHER) imk.kc = make_fastdiv(im.c8 * 8 / (16 * KS));   // stages of 16*KS k per tap
        hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8 * nsplit)), dim3(256), 0, stream, Aw, Bw, out, M, N, ld, img,
                           kblocks, tiles_m, tiles_n, kb_per, pa, pb, imk);
        FMT_HIP_CHECK(hipGetLastError());
        return FMT_OK;
    }
}

template <int PS, int TM, int TN, bool SPLIT, bool SCHED>
static int launch_product_v(const u32x4 *Aw, const u32x4 *Bw, float *out, int M, int N, int64_t ld, int img, int kblocks,
                            int nsplit, hipStream_t stream, const Planes &pa, const Planes &pb)
{
    if constexpr (PS == 0) {
        if (pa.S != nullptr)
            return launch_product_v2<PS, TM, TN, SPLIT, SCHED, true>(Aw, Bw, out, M, N, ld, img, kblocks, nsplit, stream, pa, pb);
    }
    return launch_product_v2<PS, TM, TN, SPLIT, SCHED, false>(Aw, Bw, out, M, N, ld, img, kblocks, nsplit, stream, pa, pb);
}

template <int PS, int TM, int TN>
static int launch_product(const u32x4 *Aw, const u32x4 *Bw, float *C, int M, int N, int64_t ldc, int img, int kblocks,
                          const Plan &plan, float *part, hipStream_t stream, const Planes &pa, const Planes &pb,
                          const Implicit *im = nullptr)
{
    if (im != nullptr) {
        // operand B gathered inside the product kernel (convolutions); no planes, pinned issue order only
        if (plan.nsplit == 1)
            return launch_product_v2<PS, TM, TN, false, true, false, true>(Aw, nullptr, C, M, N, ldc, img, kblocks, 1, stream, pa,
                                                                          pb, *im);
        int rcg = launch_product_v2<PS, TM, TN, true, true, false, true>(Aw, nullptr, part, M, N, (int64_t)N, 0, kblocks,
                                                                        plan.nsplit, stream, pa, pb, *im);
        if (rcg != FMT_OK) return rcg;
        return launch_reduce(part, plan.nsplit, C, M, N, ldc, img, stream);
    }
    // the elements outside plane 0 of exponent-plane operands follow the product (plain row-major results only)
    auto tail = [&]() -> int {
        if (PS != 0 || pa.S == nullptr) return FMT_OK;
        if (img != 0) return FMT_ERR_SHAPE;
        return launch_planes_tail(Aw, Bw, pa, pb, C, ldc, M, N, kblocks, stream);
    };
    if (plan.nsplit == 1) {
        int rc1 = plan.sched ? launch_product_v<PS, TM, TN, false, true>(Aw, Bw, C, M, N, ldc, img, kblocks, 1, stream, pa, pb)
                             : launch_product_v<PS, TM, TN, false, false>(Aw, Bw, C, M, N, ldc, img, kblocks, 1, stream, pa, pb);
        return rc1 != FMT_OK ? rc1 : tail();
    }
    int rc = plan.sched
                 ? launch_product_v<PS, TM, TN, true, true>(Aw, Bw, part, M, N, (int64_t)N, 0, kblocks, plan.nsplit, stream, pa, pb)
                 : launch_product_v<PS, TM, TN, true, false>(Aw, Bw, part, M, N, (int64_t)N, 0, kblocks, plan.nsplit, stream, pa, pb);
    if (rc != FMT_OK) return rc;
    rc = launch_reduce(part, plan.nsplit, C, M, N, ldc, img, stream);
    return rc != FMT_OK ? rc : tail();
}

template <int PS, int TM, int TN, bool SCALED, bool HIST>
static int launch_product_linear(const OperandView &va, const OperandView &vb, const OutSpec &out, int M, int N, int kblocks, hipStream_t stream)
{
    constexpr int KS = Pipe<PS, TM, TN>::ks, NST = Pipe<PS, TM, TN>::nst;
    const int tiles_m = (M + 64 * TM - 1) / (64 * TM), tiles_n = (N + 64 * TN - 1) / (64 * TN);
    const int64_t ntiles = (int64_t)tiles_m * tiles_n, per_xcd = (ntiles + 7) / 8;
    if (per_xcd * 8 >= ((int64_t)1 << 31)) return FMT_ERR_SHAPE;
    HistSink sink{};
    if (HIST) {
        HistRecords at;
        const int rc = get_hist_records(stream, (uint64_t)ntiles, &at);
        if (rc != FMT_OK) return rc;
        sink = hist_sink(at, (unsigned long long)M * (unsigned long long)N, out.lin->hist, (uint64_t)ntiles);
    }
    hipLaunchKernelGGL((product_linear_kernel<PS, TM, TN, KS, NST, SCALED, HIST>), dim3((unsigned)(per_xcd * 8)), dim3(256), 0, stream, va.W,
                       vb.W, out.C, M, N, out.ldc, kblocks, tiles_m, tiles_n, va.pl, vb.pl, *out.lin, sink);
    FMT_HIP_CHECK(hipGetLastError());
    if (HIST && sink.hist == nullptr) return launch_hist_finalize(sink.records, (size_t)M * (size_t)N, out.lin->hist, stream);
    return FMT_OK;
}

template <int PS, int TM, int TN>
static int launch_product_linear_t(const OperandView &va, const OperandView &vb, const OutSpec &out, int M, int N, int kblocks,
                                   hipStream_t stream)
{
    const bool hist = out.lin->hist != nullptr;
    if constexpr (PS == 0)
        if (va.pl.S != nullptr)
            return hist ? launch_product_linear<PS, TM, TN, true, true>(va, vb, out, M, N, kblocks, stream)
                        : launch_product_linear<PS, TM, TN, true, false>(va, vb, out, M, N, kblocks, stream);
    return hist ? launch_product_linear<PS, TM, TN, false, true>(va, vb, out, M, N, kblocks, stream)
                : launch_product_linear<PS, TM, TN, false, false>(va, vb, out, M, N, kblocks, stream);
}

// Whether a layer's roundings have the short forms and statistics that the product's kernel knows: not where statistics reach below
// 2^-126 (rows for fp32 denormals), and not with 23 and more bits of significand in formats with e < 8.
template <int PS>
static bool layer_in_product(const LinearOut &lin)
{
    if (lin.hist != nullptr && lin.p.exp_lo < -126) return false;
    return PS < 3 || lin.p.mode == kModeInteger || (lin.p.mode == kModeMagic && lin.p.shift >= 2u);
}

// The tile of a layer that ends in the product's kernel, from the plan of its product.  The roundings behind the sums gain by
// company on the compute unit, the sums by large tiles, so the line goes by k.  (Tiles per compute unit: of 128 x 128.)
template <int PS>
static Plan layer_plan(const Plan &plan, const LinearOut &lin, int M, int N, int kblocks)
{
    Plan p = plan;
    if (p.forced || PS == 3) return p;               // three pieces: 128 x 128 is the best of the tiles that round (9 products per value)
    const bool hist = lin.hist != nullptr;
    const int64_t tiles_m = ((int64_t)M + 127) / 128, tiles_n = ((int64_t)N + 127) / 128, tiles = tiles_m * tiles_n, cus = plan.cus;
    const int64_t outputs = (int64_t)M * N;
    if (p.tm * p.tn > 4 && kblocks <= 48) {
        // 128 x 128 instead of 256 x 256 (or 128 x 256) and a pass, up to k = 1536 (us, with statistics, 1/6/9: 4096 x 4096 x 1024 71 / 61;
        // 8192 x 4096 x 1536 154 / 143; k = 2048: alike, 4096: 256 x 256 is better).  From 2^26 outputs the chip's reads and stores
        // count as well.  Where the XCDs' runs of tiles are whole groups of tile rows, or whole groups whole runs, they walk in step,
        // a power of two of bytes apart, and 128 x 128 loses from k = 512 with 8192 columns and more (8192 x 8192 x 1024 in 1/5/10
        // 266 / 299, x 512 218 / 222; 8320 x 8192 x 1024, not in step, 287 / 254), from k = 1024 with fewer (32768 x 2048 x 1024
        // 258 / 261, x 1536 309 / 342; 33000 x 2048 x 1536 349 / 341).  From 2^27 outputs k = 1536 is too long in any case, from 2^28
        // being in step counts no more (16384 x 16384 x 512 1050 / 846, x 1024 1205 / 1113).
        const int64_t per_xcd = tiles / 8, group = 8 * tiles_n;
        const bool in_step = tiles % 8 == 0 && (per_xcd % group == 0 || group % per_xcd == 0);
        const int most = outputs < ((int64_t)1 << 26)              ? 48
                         : in_step && outputs < ((int64_t)1 << 28) ? (N > 4096 ? (hist ? 8 : 16) : 32)
                         : outputs < ((int64_t)1 << 27)            ? 48
                                                                   : 32;
        if (kblocks <= most) p.tm = p.tn = 2;
    } else if (p.tm == 2 && p.tn == 2) {
        // 128 x 64 instead of 128 x 128: three workgroups per compute unit instead of two share the roundings.  Times of 128 x 64 over
        // 128 x 128 with one piece, with statistics / without:
        //   k up to 256    0.86 - 0.97 / 0.78 - 0.90 at 0.75 to 9 tiles per compute unit, 1 at 24
        //   k = 512        0.88 - 1.02 / 0.83 - 0.98 at 0.75 to 9, 1.05 / 1.1 at 24
        //   k = 1024       0.92 - 0.99 / 0.90 - 1.0 up to 1.5 tiles, 0.92 / 0.94 at 2.25, 1.03 / 1.02 at 3, 1.07 / 1.06 at 9
        //   k = 1536       0.96 - 1.01 / 0.95 - 1.06 up to 1.5 tiles, 1.08 / 1.1 at 3
        // and two pieces as half as long a k.  Between 1.5 and 2 tiles, which 128 x 128 takes in one round, with statistics 1.01 - 1.07.
        const int one = PS == 2 ? kblocks * 2 : kblocks;     // as if of one piece
        const bool few = 2 * tiles < 5 * cus, one_round = hist && tiles <= 2 * cus && 2 * tiles > 3 * cus;
        if (!one_round && (one <= 8 || (one <= 16 && tiles <= 12 * cus) || (few && one <= (hist ? 48 : 32)))) p.tn = 1;
    }
    // a quad that N cuts is in the common case of the smaller tiles only (as 128 x 128 / 128 x 64, with statistics, us:
    // 4096 x 3003 x 1024 in 1/6/9 86 / 59; 1001 x 3003 x 2500 62 / 33)
    if (p.tm == 2 && p.tn == 2 && (N & 3) != 0) p.tn = 1;
    return p;
}

template <int PS>
int product_of_views(const OperandView &va, const OperandView &vb, int M, int N, int kblocks, const OutSpec &out,
                            const Plan &plan, float *part, hipStream_t stream)
{
    // A layer's output roundings, statistics and codes in the product's kernel: where the product leaves whole sums in one launch, and for
    // tiles of up to 128 x 128 (two workgroups and more per compute unit, so that the roundings of one run beside the products of
    // another; a 256 x 256 tile has neither the registers nor the company).  Measured, product (with planes: and the launch that adds
    // the elements outside plane 0) and pass against one kernel, us: 4096 x 3072 x 1024 in 1/6/9 with statistics 59 -> 49, without 54 -> 40,
    // in 1/8/7 55 -> 46 and 46 -> 39, in 1/7/20 179 -> 166 and 173 -> 158; 333 x 4096 x 1024 in 1/6/9 22.0 -> 13.5 and 15.6 -> 9.7.
    if (out.lin != nullptr && out.img == 0 && plan.nsplit == 1 && layer_in_product<PS>(*out.lin)) {
        const Plan p = layer_plan<PS>(plan, *out.lin, M, N, kblocks);
        if (p.tm <= 2 && p.tn <= 2 && (p.tn == 1 || (N & 3) == 0)) {
            const int rc = p.tm == 2 ? (p.tn == 2 ? launch_product_linear_t<PS, 2, 2>(va, vb, out, M, N, kblocks, stream)
                                                  : launch_product_linear_t<PS, 2, 1>(va, vb, out, M, N, kblocks, stream))
                                     : launch_product_linear_t<PS, 1, 1>(va, vb, out, M, N, kblocks, stream);
            if (rc == FMT_OK) *out.rounded = true;
            return rc;
        }
    }
#define FMT_PRODUCT(TMV, TNV) \
    launch_product<PS, TMV, TNV>(va.W, vb.W, out.C, M, N, out.ldc, out.img, kblocks, plan, part, stream, va.pl, vb.pl)
    if (plan.tm == 4 && plan.tn == 4) return FMT_PRODUCT(4, 4);
    if (plan.tm == 4 && plan.tn == 2) return FMT_PRODUCT(4, 2);
    if (plan.tm == 2 && plan.tn == 4) return FMT_PRODUCT(2, 4);
    if (plan.tm == 2 && plan.tn == 2) return FMT_PRODUCT(2, 2);
    return FMT_PRODUCT(1, 1);
#undef FMT_PRODUCT
}

// Convolutions: operand B gathered by the product kernel.
template <int PS>
int product_gathered(const OperandView &va, const Implicit &im, int M, int N, int kblocks, const OutSpec &out, const Plan &plan,
                     float *part, hipStream_t stream)
{
    const Planes none{nullptr, nullptr, 0, 0, nullptr, nullptr};
#define FMT_PRODUCT(TMV, TNV) \
    launch_product<PS, TMV, TNV>(va.W, nullptr, out.C, M, N, out.ldc, out.img, kblocks, plan, part, stream, none, none, &im)
    if (plan.tm == 4 && plan.tn == 4) return FMT_PRODUCT(4, 4);
    if (plan.tm == 4 && plan.tn == 2) return FMT_PRODUCT(4, 2);
    if (plan.tm == 2 && plan.tn == 4) return FMT_PRODUCT(2, 4);
    if (plan.tm == 2 && plan.tn == 2) return FMT_PRODUCT(2, 2);
    return FMT_PRODUCT(1, 1);
#undef FMT_PRODUCT
}

// Convolutions on exponent planes with one scale per operand: operand B prepared or gathered (im; vb.pl has
// its scale and masks).
template <int TM, int TN, bool GATHER>
static int launch_window(const OperandView &va, const OperandView &vb, const Implicit &im, int M, int N, int kblocks, const OutSpec &out,
                         const Plan &plan, float *part, hipStream_t stream)
{
    if (plan.nsplit == 1)
        return launch_product_v2<0, TM, TN, false, true, false, GATHER, true>(va.W, vb.W, out.C, M, N, out.ldc, out.img, kblocks, 1, stream, va.pl,
                                                                             vb.pl, im);
    const int rc = launch_product_v2<0, TM, TN, true, true, false, GATHER, true>(va.W, vb.W, part, M, N, (int64_t)N, 0, kblocks, plan.nsplit,
                                                                               stream, va.pl, vb.pl, im);
    return rc != FMT_OK ? rc : launch_reduce(part, plan.nsplit, out.C, M, N, out.ldc, out.img, stream);
}

template <bool GATHER>
int product_window(const OperandView &va, const OperandView &vb, const Implicit &im, int M, int N, int kblocks, const OutSpec &out,
                   const Plan &plan, float *part, hipStream_t stream)
{
    if (plan.tm > 1 && plan.tn > 1) return launch_window<2, 2, GATHER>(va, vb, im, M, N, kblocks, out, plan, part, stream);
    return launch_window<1, 1, GATHER>(va, vb, im, M, N, kblocks, out, plan, part, stream);
}

template <int PS, bool SCALED, int T>
static int launch_group_t(const Group &grp, unsigned grid, hipStream_t stream)
{
    constexpr int KS = Pipe<PS, T, T>::ks, NST = Pipe<PS, T, T>::nst;
    if constexpr (lds_bytes(T, T, pieces_of(PS), KS, NST) > 160 * 1024) {
        return FMT_ERR_SHAPE;                            // never chosen (group_tile checks the same bound)
    } else {
        hipLaunchKernelGGL((product_group_kernel<PS, T, T, KS, NST, true, SCALED>), dim3(grid), dim3(256), 0, stream, grp);
        FMT_HIP_CHECK(hipGetLastError());
        return FMT_OK;
    }
}

template <int PS, bool SCALED>
int launch_group(const Group &grp, unsigned grid, int t, hipStream_t stream)
{
    return t == 4 ? launch_group_t<PS, SCALED, 4>(grp, grid, stream) : launch_group_t<PS, SCALED, 2>(grp, grid, stream);
}

#define FMT_PRODUCT_INSTANCES(PS)                                                                                            \
    template int product_of_views<PS>(const OperandView &, const OperandView &, int, int, int, const OutSpec &, const Plan &, \
                                      float *, hipStream_t);                                                                  \
    template int product_gathered<PS>(const OperandView &, const Implicit &, int, int, int, const OutSpec &, const Plan &,    \
                                      float *, hipStream_t);                                                                  \
    template int launch_group<PS, false>(const Group &, unsigned, int, hipStream_t);

}  // namespace fmt
