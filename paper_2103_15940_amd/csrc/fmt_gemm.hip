// fmt_gemm: C = Q(op(A)) * Q(op(B)) with exact products and fp32 accumulation -- the FMACS
// instruction of Sec. III-B applied to the matrix products of Sec. IV-A.
//
// The matrix cores have no 1/6/9 (or general 1/e/m) operand type, so each rounded operand
// value r is split exactly into P bf16 pieces r = p0 + p1 (+ p2): p0 is r truncated to bf16's
// 8 significant bits, p1 the (exactly representable) remainder, and so on.  bf16 has fp32's
// exponent range, so every piece of a format with e <= 8 fits.  A product r*s is then the sum
// of the P*P piece products, each exact inside the bf16 MFMA, accumulated in its fp32
// accumulator: exact products, fp32 accumulation -- FMACS.  P = 1 for m <= 7 (bfloat16),
// P = 2 for m <= 15 (1/6/9), P = 3 up to m = 23.  Formats whose values are all binary16 values
// (e <= 5, m <= 10: binary16 itself) need no split: one fp16 piece on the fp16 MFMA.
//
// Two kernels:
//   prepare  reads one fp32 operand (either layout), rounds it to the format, splits it and
//            writes the pieces into a library-owned workspace, zero-padded and already in the
//            order the product kernel consumes: units of 32 rows x 32 k per piece, each unit
//            stored as [k-chunk of 8][row][8 x bf16] so that a wave's MFMA operand fetch is one
//            contiguous 1 KiB read.
//   product  workgroup tiles of 64x64 up to 256x256, 4 waves of MFMA 32x32x16 tiles each, operand
//            stages loaded from global memory straight into LDS (a ring of stage buffers, 32 k per
//            stage), optional split of the k range with a deterministic reduction.
//
// Formats with a 6-bit exponent and at most 10 significant bits (1/6/9, 1/6/8) take a cheaper exact
// route, "exponent planes": their significands fit binary16, only their exponent range does not.
// Every row of an operand gets a power-of-two scale 2^S that moves the binades where the row lives
// into binary16's exactly representable range (plane 0, the only one the main loop reads: ONE fp16
// MFMA product per multiply).  A value that does not fit there -- too large, or with bits below
// binary16's last denormal bit -- fits exactly under the scale 2^(S-w) (plane "above") or 2^(S+w)
// (plane "below"), w = 40 - m binades being what one plane holds; three planes cover the whole range
// of the format whatever S is.  A per-(32 rows x 32 k) mask says which planes hold anything, and every 32
// rows carry a short list of their elements outside plane 0 (with a count that says when the list did
// not hold them all: then the masks lead to them); a small kernel after the product kernel adds the
// products of those few elements, one fp32 fused multiply-add each, in a fixed order.  Exact products,
// fp32 accumulation, nothing that can overflow into a wrong result, no fallback product: the result is
// reproducible bit for bit.
//
// Several products on prepared operands can share launches (launch_gemm_prepared_batch): the product and the
// tail kernel exist in a form that takes a table of products and finds a workgroup's product from its id.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <vector>

#include "fmt_hist.h"
#include "fmt_internal.h"
#include "fmt_product.h"
#include "fmt_quant.h"
#include "fmt_split.h"
#include "fmt_tail.h"

namespace fmt {

// Workspace address (in 16-byte vectors) of chunk c (8 consecutive k) of row `row` in unit
// (rb, kb), piece `piece`.
__device__ __forceinline__ size_t unit_vec_index(int rb, int kb, int kblocks, int P, int piece, int c, int row)
{
    return (((size_t)rb * kblocks + kb) * P + piece) * kUnitVec + c * kUnitRows + row;
}


constexpr int kWinTmin = 0, kWinTmax = 31;              // range of plane 0's top binade T (S = 15 - T): with
                                                        // three planes every value of a 1/6/m format, m <= 9, fits

constexpr int kNoBinade = -1000;

// The binades of a sample of elements (fp32 patterns): the largest, and the smallest of a value that is normal in the format, emin - 1
// standing for one in its denormal range.  Zeros, what rounds to zero, infinities and NaN do not count.
__device__ __forceinline__ void window_look(uint32_t u, int emin, int m, int &hi, int &lo)
{
    const uint32_t ab = u & 0x7FFFFFFFu;
    const int E = (int)(ab >> 23) - 127;
    if (ab < 0x7F800000u && E >= emin - m - 1) {
        hi = max(hi, E);
        lo = min(lo, max(E, emin - 1));
    }
}

// The scale exponent S of exponent planes that suits what a sample showed (the rule and its reasons: window_stats_block).
__device__ __forceinline__ int window_scale(int hi, int lo, int emin, int m)
{
    const int wid = 39 - m;                       // binades below the top one that a plane holds with m + 1 significant bits
    int T = 0;
    if (hi != kNoBinade) {
        const int top = hi + 1, room = lo + wid;
        T = lo < emin ? 9 - m : (top >= room ? room : top + min(4, (room - top) / 2));
    }
    return 15 - max(kWinTmin, min(kWinTmax, T));
}

// What a pass that makes such planes knows of a tensor of n > 0 elements.
struct WindowTensor {
    const uint32_t *x;
    uint32_t n;
    int emin, m;
};

// Whether a tensor is to be expected to have more elements outside plane 0 than the products of planes are worth, from a sample's binades
// lo .. hi (as window_look has them).  Where plane 0 holds all small values, the sample shows one above it; elsewhere both ends are near, and
// the sample is to leave three binades to spare in all.  log2|x| ~ N(mean, deviation^2), the share outside and how often the answer is
// yes with 2048 elements: N(-20, 5^2), the gradients of a convolution, 1e-5, 0.02; N(-17, 5^2) 2e-4, 0.3; N(-15, 5^2) 7e-4, 0.7;
// N(-14, 5^2) 1e-3, 0.95; N(-12, 3.5^2) 2e-5, 0.1; N(-12, 4^2) 2e-4, 0.8; N(-12, 4.5^2) 8e-4, 1.  (4096, and two elements above: 0.00,
// 0.15, 0.8, 0.97 for the first four, but 1 - 2 us more per call for the lines.)
__device__ __forceinline__ bool window_wide(int hi, int lo, int S, int emin, int m)
{
    const int T = 15 - S, low = T - (39 - m);
    if (T <= 9 - m) return hi > T;
    return low > lo || (T - min(hi + 1, 1 - emin)) + (lo - low) < 3;             // 1 - emin: the largest binade
}

// The scales of a product's two tensors, one per tensor, by a workgroup of 256: 32 runs of 32 elements spread over the one, 64 over the
// other (the tensor whose patches are gathered, and the gradient).  Every workgroup of the pass that needs them does this for itself, beside its own
// loads, and all come to the same: a launch less than with a kernel ahead.  All workgroups read the same lines, which is what it costs
// (128 runs of 16 elements of each, in two lines mostly, were 2 us more in a launch of 10), so a run is a whole line of 128 bytes.
// wide: one of the two spans more than a plane (only if adapt).  Both then take two bf16 pieces instead, which hold any value: 256 -> 256
// channels of 14 x 14, 3 x 3 taps, batch 64, us for dgrad and wgrad in planes / pieces, gradients with log2|x| ~ N(mean, deviation^2)
// and their share outside plane 0: N(-20, 5^2) 1e-5 58 / 77 and 75 / 102, N(-17, 5^2) 3e-4 80 / 77 and 101 / 103, N(-15, 5^2) 1e-3
// 150 / 78 and 194 / 104, N(-14, 8^2) 4e-2 101 / 77 and 153 / 104.
struct WindowPair {
    int S[2];
    bool wide;
};

// The largest of a wave's values: four steps inside rows of 16 lanes, then row to row and half to half, into the wave's last lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    auto with = [&](auto ctrl) __attribute__((always_inline)) {
        v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, false));
    };
    with(std::integral_constant<int, 0x111>{});      // row_shr:1
    with(std::integral_constant<int, 0x112>{});
    with(std::integral_constant<int, 0x114>{});
    with(std::integral_constant<int, 0x118>{});
    with(std::integral_constant<int, 0x142>{});      // row_bcast:15
    with(std::integral_constant<int, 0x143>{});      // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// A thread's 4 * LOADS elements of the 1024 * LOADS (of fewer: all, some of them twice).  Runs start an odd number of lines
// apart, so that they do not all meet the same pixels of images of a power of two, the first with the tensor: the same elements, and the same results,
// wherever the tensor lies (of one that starts inside a line a run touches two).
template <uint32_t LOADS>
__device__ __forceinline__ void window_sample(const WindowTensor &t, uint32_t wave, uint32_t lane, uint32_t *v)
{
    constexpr uint32_t kRuns = 32u * LOADS;
    typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
    if (t.n >= kRuns * 32u + 32u) {               // the same in the whole launch
        const uint32_t step = (((t.n - 32u) / (kRuns - 1u) / 32u - 1u) | 1u) * 32u;
#pragma unroll
        for (uint32_t i = 0; i < LOADS; ++i) {
            const uint32_t *first = t.x + (size_t)((i * 4u + wave) * 8u) * step;
            const u32x4u w = *reinterpret_cast<const u32x4u *>(first + (lane / 8u * step + lane % 8u * 4u));
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) v[4 * i + j] = w[j];
        }
    } else {
#pragma unroll
        for (uint32_t i = 0; i < 4u * LOADS; ++i) v[i] = t.x[min((wave * 4u * LOADS + i) * 64u + lane, t.n - 1u)];
    }
}

// The binades are those of the largest magnitude and of the smallest that counts: two elements per instruction for the one (infinities
// and NaN in a wave's sample send it through the patterns), one and a half per element for the other, the smallest of
// twice the pattern less twice the least that counts (what lies below wraps round and comes last).
__device__ __forceinline__ WindowPair window_pair(const WindowTensor &a, const WindowTensor &b, int adapt)
{
    __shared__ uint32_t s_top[2][4], s_low[2][4];
    constexpr uint32_t kInf = 0x7F800000u;
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t least = (uint32_t)(a.emin - a.m - 1 + 127) << 23;
    uint32_t u[12];
    window_sample<1>(a, wave, lane, u);
    window_sample<2>(b, wave, lane, u + 4);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const int from = o == 0 ? 0 : 4, to = o == 0 ? 4 : 12;
        float most = 0.0f;
        uint32_t low = 0xFFFFFFFFu;
#pragma unroll
        for (int i = from; i < to; i += 2) {
            most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(__uint_as_float(u[i])), fabsf(__uint_as_float(u[i + 1]))), most);
            low = min(min(low, (u[i] << 1) - 2u * least), (u[i + 1] << 1) - 2u * least);
        }
        uint32_t top = __float_as_uint(most);
        if (__ballot(top >= kInf) != 0ull) {
            top = 0u;
#pragma unroll
            for (int i = from; i < to; ++i) {
                const uint32_t ab = u[i] & 0x7FFFFFFFu;
                top = max(top, ab < kInf ? ab : 0u);
            }
        }
        top = wave_max(top);
        low = ~wave_max(~low);
        if (lane == 0u) {
            s_top[o][wave] = top;
            s_low[o][wave] = low;
        }
    }
    __syncthreads();
    WindowPair w{{0, 0}, false};
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        uint32_t top = 0u, low = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            top = max(top, s_top[o][i]);
            low = min(low, s_low[o][i]);
        }
        top = (uint32_t)__builtin_amdgcn_readfirstlane((int)top);
        low = ((uint32_t)__builtin_amdgcn_readfirstlane((int)low) >> 1) + least;
        const int hi = top < least ? kNoBinade : (int)(top >> 23) - 127, lo = max((int)(low >> 23) - 127, a.emin - 1);
        w.S[o] = window_scale(hi, lo, a.emin, a.m);
        w.wide = w.wide || (adapt != 0 && hi != kNoBinade && window_wide(hi, lo, w.S[o], a.emin, a.m));
    }
    return w;
}

// How element (row, k) of an operand is found in memory.
enum {
    kSrcMatrix = 0,     // X[row*ld + k] (kcontig) or X[k*ld + row]
    kSrcPatchRows = 1,  // convolution patches: row = (n, y, x) on a grid gy x gx, k = (ch, r, s)
    kSrcPatchK = 2,     // the same patches transposed: row = (ch, r, s), k = (n, y, x)
    kSrcChannelRows = 3,  // NCHW tensor as a matrix: row = channel, k = (n, position)
    kSrcFilterT = 4,    // filter [K][C][R][S] with row = c, k = (kout, r, s)
    kSrcFilterTap = 5   // filter [K][C][R][S] with k = (tap, channel): element (row, k) sits at
                        // row*th + (k % D)*tw + k / D, D = k0.d channels (th, tw hold the two strides)
};

// Geometry of a gathered operand.  Patches read T[n][ch][iy][ix] of an NCHW tensor with tc
// channels of th x tw, where iy = (y*mul_y + off_y + tap*r) / den_y must divide exactly and lie in
// [0, th) (else the element is zero), likewise ix.  Forward and wgrad: mul = stride, off = -pad,
// tap = +1, den = 1; dgrad (patches of dY seen from an input position): mul = 1, off = +pad,
// tap = -1, den = stride.
struct Gather {
    int kind;
    int tc, th, tw;
    int gy, gx;
    int R, S;
    int mul_y, mul_x, off_y, off_x, tap, den_y, den_x;
    // pre != 0: the tensor was rounded and split beforehand (round_split_kernel); X then points to
    // the piece patterns, two per 32-bit word, in (P+1)/2 planes of `plane` elements each (a patch
    // element is reused R*S times, so rounding it once pays)
    int pre, plane;
    // fast != 0 (patch rows, den == 1, R*S <= 32, pre): the taps inside the tensor are kept as a
    // per-lane bit mask and the element offset splits into a per-lane and a per-k (scalar) part;
    // element plane-1 of the rounded tensor is a zero that out-of-range taps read
    int fast;
    // fast == 2: the same for the transposed patches (rows = taps, k = positions; see gather_taps)
    // divisors of the index decompositions: rows by (r0 inner, r1 outer), k by (k0 inner, k1 outer)
    FastDiv r0, r1, k0, k1;
};

// One operand of a prepare launch: X is fp32, `rows` x K after op(); for a plain matrix element
// (r, k) sits at X[r*ld + k] (kcontig) or X[k*ld + r]; vec4: base 16-byte aligned and ld a
// multiple of 4.  kcontig also selects the lane mapping (8 lanes along k per row, or lanes
// along rows) for the gathered kinds.
struct PrepOperand {
    const uint32_t *X;
    u32x4 *W;
    int64_t ld;
    int rows;
    int kcontig;
    int vec4;
    unsigned nblocks;   // workgroups of this operand: slabs * row groups
    Gather g;
    Planes pl;          // pl.S != nullptr: scaled fp16 exponent planes (PS == 0, plain matrices only)
};

// Offset of tap (r, s) seen from the spatial base (by, bx) = (y*mul + off) inside one h x w plane,
// or -1 when the tap falls outside the tensor (or, for dgrad, between the strides).  All tensors
// have fewer than 2^31 elements, so 32-bit offsets suffice.
template <bool DIV>
__device__ __forceinline__ int tap_offset(const Gather &g, int by, int bx, int r, int s)
{
    int iy = by + g.tap * r, ix = bx + g.tap * s;
    if (DIV) {
        if (iy < 0 || ix < 0) return -1;
        const int qy = iy / g.den_y, qx = ix / g.den_x;
        if (qy * g.den_y != iy || qx * g.den_x != ix) return -1;
        iy = qy;
        ix = qx;
    }
    return ((unsigned)iy < (unsigned)g.th && (unsigned)ix < (unsigned)g.tw) ? iy * g.tw + ix : -1;
}

template <bool DIV>
__device__ __forceinline__ void gather_patches(const PrepOperand &o, int row, int k0, int K, int (&idx)[8])
{
    const Gather &g = o.g;
    const int hw = g.th * g.tw;
    if (g.kind == kSrcPatchRows) {
        // fixed position (n, y, x); k runs over (ch, r, s).  Lanes run along rows in this layout, so
        // k0 is the same in the whole wave and its decomposition and the walk over the taps are
        // scalar work.
        int x, t, y, n;
        divmod(g.r0, row, t, x);
        divmod(g.r1, t, n, y);
        const int by = y * g.mul_y + g.off_y, bx = x * g.mul_x + g.off_x;
        const int ku = __builtin_amdgcn_readfirstlane(k0);
        int s, t2, r, ch;
        divmod(g.k0, ku, t2, s);
        divmod(g.k1, t2, ch, r);
        const int nplane = n * g.tc * hw;
        int cplane = ch * hw;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int off = tap_offset<DIV>(g, by, bx, r, s);
            if (ku + j < K && off >= 0) idx[j] = nplane + cplane + off;
            if (++s == g.S) {
                s = 0;
                if (++r == g.R) {
                    r = 0;
                    cplane += hw;
                }
            }
        }
    } else {
        // fixed tap (ch, r, s); k runs over the positions (n, y, x)
        int s, t, r, ch;
        divmod(g.r0, row, t, s);
        divmod(g.r1, t, ch, r);
        int x, t2, y, n;
        divmod(g.k0, k0, t2, x);
        divmod(g.k1, t2, n, y);
        int plane = (n * g.tc + ch) * hw;
        const int step = g.tc * hw;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int off = tap_offset<DIV>(g, y * g.mul_y + g.off_y, x * g.mul_x + g.off_x, r, s);
            if (k0 + j < K && off >= 0) idx[j] = plane + off;
            if (++x == g.gx) {
                x = 0;
                if (++y == g.gy) {
                    y = 0;
                    plane += step;
                }
            }
        }
    }
}

// Element offsets of (row, k0 .. k0+7) of a gathered operand in its tensor; -1 = a zero (padding,
// a tap between the strides, beyond rows / K).
__device__ __forceinline__ void gather8(const PrepOperand &o, int row, int k0, int K, int (&idx)[8])
{
    const Gather &g = o.g;
#pragma unroll
    for (int j = 0; j < 8; ++j) idx[j] = -1;
    if (row >= o.rows || k0 >= K) return;
    if (g.kind == kSrcPatchRows || g.kind == kSrcPatchK) {
        if (g.den_y == 1 && g.den_x == 1)
            gather_patches<false>(o, row, k0, K, idx);
        else
            gather_patches<true>(o, row, k0, K, idx);
    } else if (g.kind == kSrcFilterTap) {
        int ch, tap;
        divmod(g.k0, k0, tap, ch);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (k0 + j < K) idx[j] = row * g.th + ch * g.tw + tap;
            if (++ch == g.k0.d) {
                ch = 0;
                ++tap;
            }
        }
    } else {
        // kSrcChannelRows: k = (image, position), L = g.k0.d positions; kSrcFilterT: k = (filter, tap),
        // L = R*S taps; element (row, k) sits at ((k / L) * tc + row) * L + k % L in both
        const int L = g.k0.d;
        int pos, q;
        divmod(g.k0, k0, q, pos);
        int base = (q * g.tc + row) * L;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (k0 + j < K) idx[j] = base + pos;
            if (++pos == L) {
                pos = 0;
                base += g.tc * L;
            }
        }
    }
}

// Rounds a tensor to the format and splits it once, elementwise, for operands that are gathered
// many times: word plane w (n + 1 words, the last one zero) holds piece 2w in its low half and
// piece 2w+1 in its high half.
template <int MODE, bool FTZ, int PS>
__global__ __launch_bounds__(256) void round_split_kernel(const uint32_t *__restrict__ x, uint32_t *__restrict__ out,
                                                          int n, QuantParams p)
{
    constexpr int P = pieces_of(PS);
    const size_t plane = (size_t)n + 1;          // one extra element per plane, always zero
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        uint32_t pc[P];
        round_and_split<MODE, FTZ, PS>(x[i], p, pc);
        out[i] = pc[0] | (P >= 2 ? pc[P >= 2 ? 1 : 0] << 16 : 0u);
        if (P >= 3) out[plane + i] = pc[P >= 3 ? 2 : 0];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        out[n] = 0u;
        if (P >= 3) out[plane + n] = 0u;
    }
}

constexpr int kRoundEach = 8;      // elements per thread: the sample is as much work as 4 of them
// The same for the weight gradient on exponent planes: a word holds the element's binary16 pattern and, in its upper half, the plane that it
// belongs to (0, 1 above, 2 below).  Wide tensors (window_pair, with the gradient's): two bf16 pieces as above.  What was found is left for the
// launches behind: S_out[0] and S_grad[0] the scales, S_grad[1] whether there are pieces.
template <int MODE, bool FTZ>
__global__ __launch_bounds__(256) void round_window_kernel(WindowTensor t, WindowTensor grad, int adapt, uint32_t *__restrict__ out, int w,
                                                           int *__restrict__ S_out, int *__restrict__ S_grad, QuantParams p)
{
    constexpr int kEach = kRoundEach;
    uint32_t u[kEach];
    auto load = [&](uint32_t first) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t j = 0; j < kEach; ++j) u[j] = t.x[min(first + threadIdx.x + j * 256u, t.n - 1u)];
    };
    uint32_t first = blockIdx.x * (256u * kEach);
    load(first);
    const WindowPair pair = window_pair(t, grad, adapt);
    const int S = pair.S[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        out[t.n] = 0u;
        S_out[0] = S;
        S_grad[0] = pair.S[1];
        S_grad[1] = pair.wide ? 1 : 0;
    }
    const float f = __uint_as_float((uint32_t)(127 + S) << 23);
    for (;;) {
        uint32_t r[kEach];
        if (!pair.wide) quantize_run<MODE, FTZ>(u, run_is_rare(u, p), p, round_masks(p), r);
#pragma unroll
        for (uint32_t j = 0; j < kEach; ++j) {
            const uint32_t i = first + threadIdx.x + j * 256u;
            if (pair.wide) {                      // the same in the whole launch
                uint32_t pc[2];
                round_and_split<MODE, FTZ, 2>(u[j], p, pc);
                if (i < t.n) out[i] = pc[0] | (pc[1] << 16);
                continue;
            }
            const float sc = __uint_as_float(r[j]) * f;
            _Float16 h = static_cast<_Float16>(sc);
            const float back = static_cast<float>(h);
            uint32_t plane = 0u;
            if (back < sc || back > sc) {         // as split_planes has it
                const bool up = fabsf(sc) >= 65536.0f;
                h = static_cast<_Float16>(ldexpf(__uint_as_float(r[j]), up ? S - w : S + w));
                plane = up ? 1u : 2u;
            }
            if (i < t.n) out[i] = (uint32_t)__builtin_bit_cast(uint16_t, h) | (plane << 16);
        }
        if (t.n - first <= gridDim.x * (256u * kEach)) break;
        first += gridDim.x * (256u * kEach);
        load(first);
    }
}

// Rounds an NCHW tensor (C a multiple of 32) to the format, splits it, and writes the pieces in
// pixel-major order out[piece][pixel][channel] (16 bits per element) -- the operand the product kernel
// gathers convolution patches from.  A workgroup takes 64 consecutive pixels (of the flattened n*h*w)
// by 32 channels: reads run along pixels, the transposition goes through LDS, and a lane writes 8
// consecutive channels of one pixel as one 16-byte vector.  One vector of zeros follows the last piece.
template <int MODE, bool FTZ, int PS>
__device__ __forceinline__ void nhwc_split_block(const uint32_t *__restrict__ x, u32x4 *__restrict__ out, int C, int HW, int npix,
                                                 const QuantParams &p, int bx, int cb)
{
    constexpr int P = pieces_of(PS);
    constexpr int kPitch = 18;                                  // 32-bit words per pixel row (16 + 2: odd multiple of 2)
    __shared__ uint32_t tile[P][64][kPitch];
    const int tid = threadIdx.x;
    const int pix = tid % 64, cg = tid / 64;
    const int gp = bx * 64 + pix;
    const bool valid = gp < npix;
    const int n = valid ? gp / HW : 0, hw = valid ? gp - n * HW : 0;
    const uint32_t *src = x + ((size_t)n * C + cb * 32 + cg * 8) * HW + hw;
    uint32_t u[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) u[i] = valid ? src[(size_t)i * HW] : 0u;
    u32x4 pc[P];
    split8<MODE, FTZ, PS>(u, p, pc);
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[q][pix][cg * 4 + i] = pc[q][i];
    __syncthreads();
    const int opix = tid / 4, part = tid % 4;
    const int ogp = bx * 64 + opix;
    const size_t piece_vec = (size_t)npix * (C / 8);
    if (ogp < npix) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = tile[q][opix][part * 4 + i];
            out[q * piece_vec + (size_t)ogp * (C / 8) + cb * 4 + part] = w;
        }
    }
    if (bx == 0 && cb == 0 && tid == 0) out[P * piece_vec] = u32x4{0u, 0u, 0u, 0u};
}

// Transposed patches (wgrad: rows = taps (ch, r, s), k = positions (n, y, x)), pre-rounded tensor.
// A workgroup takes one unit of 32 taps and 256 positions, one position per lane: which taps fall
// inside the tensor is a per-lane bit mask and the walk over the taps is scalar work, exactly as in
// the forward gather; what differs is the output, which wants 8 consecutive positions of ONE tap in
// a lane.  Each wave therefore passes its 8 taps x 64 positions through a tile of its own in LDS and
// reads them back transposed (rows padded to 72 words against bank conflicts).
// WINDOW: the words are round_window_kernel's.  Plane 0 is written in a first turn over the taps, and only if the workgroup met elements of
// the other planes are these written, in a second, for the units that hold any.  pieces: the words are two bf16 pieces (wide tensors).
template <int P, bool WINDOW = false>
__device__ __forceinline__ void gather_taps(const PrepOperand &o, unsigned bid, int K, int kblocks, bool pieces = false)
{
    static_assert(!WINDOW || P == 1, "one piece");
    constexpr int NW = (P + 1) / 2;                    // 32-bit word planes per element
    __shared__ uint32_t tile[4][NW][8][72];
    const Gather &g = o.g;
    const uint32_t *__restrict__ X = o.X;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ngroups = (kblocks + 7) / 8;
    const int pg = (int)(bid % (unsigned)ngroups), rb = (int)(bid / (unsigned)ngroups);
    const int hw = g.th * g.tw;
    const int pos = pg * 256 + tid;
    int x, t, y, n;
    divmod(g.k0, pos, t, x);
    divmod(g.k1, t, n, y);
    const int by = y * g.mul_y + g.off_y, bx = x * g.mul_x + g.off_x;
    const int lo_r = max(0, -by), hi_r = min(g.R, g.th - by);
    const int lo_s = max(0, -bx), hi_s = min(g.S, g.tw - bx);
    const int ns = hi_s - lo_s;
    const uint32_t mx = ns <= 0 ? 0u : ((ns >= 32 ? 0xFFFFFFFFu : (1u << ns) - 1u) << lo_s);
    uint32_t mask = 0u;
    for (int r = 0; r < g.R; ++r)
        if (r >= lo_r && r < hi_r) mask |= mx << (r * g.S);
    if (pos >= K) mask = 0u;
    const int lane_base = n * g.tc * hw + by * g.tw + bx;
    const int zero = g.plane - 1;
    const int gi = lane >> 3, li = lane & 7;           // after the transpose: positions gi*8 .. gi*8+7 of tap li
    const int pb = pg * 256 + wave * 64 + gi * 8;       // first of this lane's 8 positions
    const int kb = pb / kUnitK, c = (pb % kUnitK) / 8;
    uint32_t have = 1u;                                // WINDOW: planes met
#pragma unroll 1
    for (int turn = 0; turn < (WINDOW ? 2 : 1); ++turn) {
    if constexpr (WINDOW) {
        if (turn == 1) {
            if (pieces) break;                         // the same in the whole launch
            // of the unit: the lanes of one half of the wave
#pragma unroll
            for (int off = 1; off < 32; off <<= 1) have |= (uint32_t)__shfl_xor((int)have, off, 64);
            if (kb < kblocks && (lane & 31) == 0) o.pl.mask[(size_t)rb * kblocks + kb] = (uint8_t)have;
            if (!__syncthreads_or((have & 6u) != 0u)) break;
        }
    }
    for (int pass = 0; pass < 4; ++pass) {
        const int tap0 = rb * 32 + pass * 8;           // the same in the whole workgroup
        int s, t2, r, ch;
        divmod(g.r0, tap0, t2, s);
        divmod(g.r1, t2, ch, r);
        int rs = r * g.S + s;
        int delta = ch * hw + r * g.tw + s;
        uint32_t w[NW][8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool ok = tap0 + j < o.rows && ((mask >> rs) & 1u);
            const uint32_t idx = (uint32_t)(ok ? lane_base + delta : zero);
#pragma unroll
            for (int q = 0; q < NW; ++q) w[q][j] = X[(size_t)q * g.plane + idx];
            ++rs;
            ++delta;
            if (++s == g.S) {
                s = 0;
                delta += g.tw - g.S;
                if (++r == g.R) {
                    r = 0;
                    rs = 0;
                    delta += hw - g.R * g.tw;
                }
            }
        }
        __syncthreads();                               // the previous pass's tile has been read
#pragma unroll
        for (int q = 0; q < NW; ++q)
#pragma unroll
            for (int j = 0; j < 8; ++j) tile[wave][q][j][lane] = w[q][j];
        __syncthreads();
        uint32_t v[NW][8];
#pragma unroll
        for (int q = 0; q < NW; ++q)
#pragma unroll
            for (int m = 0; m < 8; ++m) v[q][m] = tile[wave][q][li][gi * 8 + m];
        const int rr = pass * 8 + li;
        if constexpr (WINDOW) {
            if (pieces) {
                if (kb < kblocks) {
                    u32x4 hi, lo;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        hi[i] = __builtin_amdgcn_perm(v[0][2 * i + 1], v[0][2 * i], 0x05040100u);
                        lo[i] = __builtin_amdgcn_perm(v[0][2 * i + 1], v[0][2 * i], 0x07060302u);
                    }
                    o.W[unit_vec_index(rb, kb, kblocks, 2, 0, c, rr)] = hi;
                    o.W[unit_vec_index(rb, kb, kblocks, 2, 1, c, rr)] = lo;
                }
                continue;
            }
            uint32_t planes = 0u;
#pragma unroll
            for (int m = 0; m < 8; ++m) planes |= v[0][m] >> 16;             // 1 above, 2 below, 3 both
            if (turn == 0) {
                have |= planes << 1;
                if (__ballot(planes != 0u) != 0ull) {                        // the same in the whole wave
#pragma unroll
                    for (int m = 0; m < 8; ++m) v[0][m] = v[0][m] < 0x10000u ? v[0][m] : 0u;
                }
                if (kb < kblocks) {
                    u32x4 out;
#pragma unroll
                    for (int i = 0; i < 4; ++i) out[i] = __builtin_amdgcn_perm(v[0][2 * i + 1], v[0][2 * i], 0x05040100u);
                    o.W[unit_vec_index(rb, kb, kblocks, 1, 0, c, rr)] = out;
                }
            } else if (kb < kblocks) {
#pragma unroll
                for (uint32_t q = 1; q < 3; ++q)
                    if ((have >> q) & 1u) {
                        u32x4 out;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            out[i] = (v[0][2 * i] >> 16 == q ? v[0][2 * i] & 0xFFFFu : 0u) | (v[0][2 * i + 1] >> 16 == q ? v[0][2 * i + 1] << 16 : 0u);
                        o.W[q * o.pl.plane + unit_vec_index(rb, kb, kblocks, 1, 0, c, rr)] = out;
                    }
            }
        } else if (kb < kblocks) {
#pragma unroll
            for (int pc = 0; pc < P; ++pc) {
                u32x4 out;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t hi = v[pc / 2][2 * i + 1], lo = v[pc / 2][2 * i];
                    out[i] = __builtin_amdgcn_perm(hi, lo, (pc & 1) ? 0x07060302u : 0x05040100u);
                }
                o.W[unit_vec_index(rb, kb, kblocks, P, pc, c, rr)] = out;
            }
        }
    }
    }
}

// prepare: both operands of a product in one launch (workgroups [0, a.nblocks) take op(A), the
// rest op(B)).  k-contiguous input: a workgroup takes 32 rows x 64 k, 8 neighbouring lanes read
// 256 contiguous bytes of a row; transposed input: 64 rows x 32 k, a wave reads 256 contiguous
// bytes for each k.
// TAPS: one of the operands may take gather_taps (whose LDS tile and barriers the other launches do
// not pay for).
template <int MODE, bool FTZ, int PS, bool TAPS = false>
__device__ __forceinline__ void prepare_block(const PrepOperand &a, const PrepOperand &b, int K, int kblocks,
                                              const QuantParams &p, unsigned block)
{
    constexpr int P = pieces_of(PS);
    const int tid = threadIdx.x;
    // Each operand owns a run of workgroup ids padded to a multiple of 8.  Consecutive ids go to
    // different XCDs (each with its own L2), so the ids are remapped to give every XCD a contiguous
    // range of rows: a gathered tensor is then read into each L2 once, not eight times.
    const unsigned a_ids = (a.nblocks + 7u) / 8u * 8u;
    const bool second = block >= a_ids;
    const PrepOperand &o = second ? b : a;
    const unsigned lid = block - (second ? a_ids : 0u);
    const unsigned per_xcd = (o.nblocks + 7u) / 8u;
    const unsigned bid = (lid % 8u) * per_xcd + lid / 8u;
    if (bid >= o.nblocks) return;
    if constexpr (TAPS) {
        if (o.g.fast == 2) {                 // block-uniform: every thread takes part in its barriers
            gather_taps<P>(o, bid, K, kblocks);
            return;
        }
    }
    const uint32_t *__restrict__ X = o.X;
    const int64_t ld = o.ld;
    const int rows = o.rows;
    const bool kcontig = o.kcontig != 0;
    const int nslabs = kcontig ? (kblocks + 1) / 2 : kblocks;
    const int bx = bid % nslabs, by = bid / nslabs;
    int row, k0;
    if (kcontig) {
        row = by * 32 + tid / 8;
        k0 = bx * 64 + (tid % 8) * 8;
    } else {
        // the fast gather takes kFastRows groups of 64 rows per workgroup, the other paths one
        row = by * 64 * (o.g.fast == 1 ? kFastRows : 1) + tid % 64;
        k0 = bx * 32 + (tid / 64) * 8;
    }
    if (k0 >= kblocks * kUnitK) return;      // k-contiguous slabs cover two k-blocks; the last may be half
    uint32_t v[8];
    uint32_t w01[8], w2[P >= 3 ? 8 : 1];     // pre-rounded source: pieces 0|1 packed per element, piece 2
    bool packed = false;
    if (o.g.fast == 1) {
        // Patches, lanes along positions: which taps (r, s) fall inside the tensor is a per-lane bit
        // mask, the offset of a tap is per-lane base + a term that depends on k alone, and k is
        // the same in the whole wave, so walking the 8 taps is scalar work.
        // The walk is shared by kFastRows groups of 64 positions (the scalar unit, not the vector unit
        // or memory, bounds this path), each lane owning one position per group.
        const Gather &g = o.g;
        const int hw = g.th * g.tw;
        uint32_t mask[kFastRows];
        int lane_base[kFastRows];
#pragma unroll
        for (int q = 0; q < kFastRows; ++q) {
            const int rq = row + 64 * q;
            int x, t, y, n;
            divmod(g.r0, rq, t, x);
            divmod(g.r1, t, n, y);
            const int by = y * g.mul_y + g.off_y, bx = x * g.mul_x + g.off_x;
            const int lo_r = g.tap > 0 ? max(0, -by) : max(0, by - g.th + 1), hi_r = g.tap > 0 ? min(g.R, g.th - by) : min(g.R, by + 1);
            const int lo_s = g.tap > 0 ? max(0, -bx) : max(0, bx - g.tw + 1), hi_s = g.tap > 0 ? min(g.S, g.tw - bx) : min(g.S, bx + 1);
            const int ns = hi_s - lo_s;
            const uint32_t mx = ns <= 0 ? 0u : ((ns >= 32 ? 0xFFFFFFFFu : (1u << ns) - 1u) << lo_s);
            uint32_t mq = 0u;
            for (int r = 0; r < g.R; ++r)
                if (r >= lo_r && r < hi_r) mq |= mx << (r * g.S);
            mask[q] = rq < rows ? mq : 0u;
            lane_base[q] = n * g.tc * hw + by * g.tw + bx;
        }
        const int ku = __builtin_amdgcn_readfirstlane(k0);
        int s, t2, r, ch;
        divmod(g.k0, ku, t2, s);
        divmod(g.k1, t2, ch, r);
        int rs = r * g.S + s;
        int delta = ch * hw + g.tap * (r * g.tw + s);
        const int zero = g.plane - 1;
        const uint32_t *__restrict__ X2 = X + g.plane;
        uint32_t f01[kFastRows][8], f2[kFastRows][P >= 3 ? 8 : 1];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool kin = ku + j < K;
#pragma unroll
            for (int q = 0; q < kFastRows; ++q) {
                const bool ok = kin && ((mask[q] >> rs) & 1u);
                const uint32_t idx = (uint32_t)(ok ? lane_base[q] + delta : zero);
                f01[q][j] = X[idx];
                if (P >= 3) f2[q][j] = X2[idx];
            }
            ++rs;
            delta += g.tap;
            if (++s == g.S) {
                s = 0;
                delta += g.tap * (g.tw - g.S);
                if (++r == g.R) {
                    r = 0;
                    rs = 0;
                    delta += hw - g.tap * g.R * g.tw;
                }
            }
        }
        // two elements' 16-bit halves into one word with a byte permute
        const int kb = k0 / kUnitK, c = (k0 % kUnitK) / 8;
#pragma unroll
        for (int q = 0; q < kFastRows; ++q) {
            const int rq = row + 64 * q;
            const int rb = rq / kUnitRows, rr = rq % kUnitRows;
#pragma unroll
            for (int pc = 0; pc < P; ++pc) {
                u32x4 w;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (pc == 0) w[i] = __builtin_amdgcn_perm(f01[q][2 * i + 1], f01[q][2 * i], 0x05040100u);
                    if (pc == 1) w[i] = __builtin_amdgcn_perm(f01[q][2 * i + 1], f01[q][2 * i], 0x07060302u);
                    if (pc == 2) w[i] = __builtin_amdgcn_perm(f2[q][P >= 3 ? 2 * i + 1 : 0], f2[q][P >= 3 ? 2 * i : 0], 0x05040100u);
                }
                o.W[unit_vec_index(rb, kb, kblocks, P, pc, c, rr)] = w;
            }
        }
        return;
    } else if (o.g.kind != kSrcMatrix) {
        int idx[8];
        gather8(o, row, k0, K, idx);
        if (o.g.pre) {
            // pieces were made beforehand: pure data movement (element plane-1 is a zero)
            const uint32_t *__restrict__ X2 = X + o.g.plane;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t at = (uint32_t)(idx[j] >= 0 ? idx[j] : o.g.plane - 1);
                w01[j] = X[at];
                if (P >= 3) w2[j] = X2[at];
            }
            packed = true;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = idx[j] >= 0 ? X[(uint32_t)idx[j]] : 0u;
        }
    } else if (kcontig && o.vec4 && row < rows && k0 + 8 <= K) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(X + (size_t)row * ld + k0);
        const u32x4 lo = __builtin_nontemporal_load(src), hi = __builtin_nontemporal_load(src + 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = lo[j];
            v[4 + j] = hi[j];
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = k0 + j;
            const bool ok = row < rows && k < K;
            const size_t idx = kcontig ? (size_t)row * ld + k : (size_t)k * ld + row;
            v[j] = ok ? X[idx] : 0u;
        }
    }
    const int rb = row / kUnitRows, rr = row % kUnitRows;
    const int kb = k0 / kUnitK, c = (k0 % kUnitK) / 8;
    if (packed) {
        // two elements' 16-bit halves into one word with a byte permute
#pragma unroll
        for (int q = 0; q < P; ++q) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (q == 0) w[i] = __builtin_amdgcn_perm(w01[2 * i + 1], w01[2 * i], 0x05040100u);
                if (q == 1) w[i] = __builtin_amdgcn_perm(w01[2 * i + 1], w01[2 * i], 0x07060302u);
                if (q == 2) w[i] = __builtin_amdgcn_perm(w2[P >= 3 ? 2 * i + 1 : 0], w2[P >= 3 ? 2 * i : 0], 0x05040100u);
            }
            o.W[unit_vec_index(rb, kb, kblocks, P, q, c, rr)] = w;
        }
        return;
    }
    u32x4 w[P];
    split8<MODE, FTZ, PS>(v, p, w);
#pragma unroll
    for (int q = 0; q < P; ++q) o.W[unit_vec_index(rb, kb, kblocks, P, q, c, rr)] = w[q];
}

// Eight rounded values of one thread (fp32 patterns r[], elements k0 .. k0 + 7 of row `row` of operand o) as
// binary16 patterns, two per word: p0 = plane 0, pa / pb = the planes above / below (zero where an element
// does not belong to the plane).  Elements outside plane 0 also leave a record in the list of their row of
// units for the kernel that adds their products (not where one scale S serves the whole tensor: RECORDS false, and row and k0 unused).
// Returns 2 / 4 if any element went above / below.
template <bool RECORDS = true>
__device__ __forceinline__ uint32_t split_planes(const Planes &pl, int S, int row, int k0, const uint32_t (&r)[8], u32x4 &p0, u32x4 &pa,
                                                 u32x4 &pb)
{
    const float f = __uint_as_float((uint32_t)(127 + S) << 23);     // 2^S: -16 <= S <= 15
    pa = pb = u32x4{0u, 0u, 0u, 0u};
    uint32_t mine = 0u;
    // All eight lie in plane 0 if their magnitudes, scaled (exactly), are below 2^16 and the smallest that is not zero has its last
    // bit at or above binary16's, 2^-24: is at least 2^-15 or, where the plane reaches down to the format's denormals (S >= 6 + m), whatever
    // it is.  Then the conversion is exact: 2 vector instructions per element (3.5 for the higher planes), where a conversion there
    // and back and two comparisons per element take 8.
    float sc[8], top = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) sc[j] = __uint_as_float(r[j]) * f;
#pragma unroll
    for (int j = 0; j < 8; j += 2) top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(sc[j]), fabsf(sc[j + 1])), top);
    bool inside = top < 65536.0f;
    const bool bottom = S >= 46 - pl.w;
    if (__ballot(!bottom) != 0ull) {             // the same in the whole wave
        uint32_t least = 0xFFFFFFFFu;            // twice a pattern less one: zeros come last
#pragma unroll
        for (int j = 0; j < 8; ++j) least = min(least, (__float_as_uint(sc[j]) << 1) - 1u);
        inside = inside && (bottom || least >= 2u * 0x38000000u - 1u);
    }
    if (inside) {
#pragma unroll
        for (int i = 0; i < 4; ++i) p0[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(sc[2 * i], sc[2 * i + 1]));
        return mine;
    }
    uint32_t hb[8];
    bool other[8], any = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        // r * 2^S converts to binary16 and back unchanged <=> it is a binary16
        // value -- zeros, the normal and the denormal range, infinities.  NaN (neither below nor above its
        // own conversion) stays in plane 0 as well.
        const _Float16 h = static_cast<_Float16>(sc[j]);            // round to nearest even
        const float back = static_cast<float>(h);
        other[j] = back < sc[j] || back > sc[j];
        any |= other[j];
        hb[j] = (uint32_t)__builtin_bit_cast(uint16_t, h);
    }
    if (any) {  
        const int w = pl.w;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (other[j]) {
                // too large for plane 0 -> the plane above; bits below 2^-24 -> the plane below (exact there)
                const float rf = __uint_as_float(r[j]);
                const bool up = fabsf(ldexpf(rf, S)) >= 65536.0f;
                const _Float16 g = static_cast<_Float16>(ldexpf(rf, up ? S - w : S + w));
                const uint32_t gb = (uint32_t)__builtin_bit_cast(uint16_t, g) << (16 * (j & 1));
                pa[j / 2] |= up ? gb : 0u;
                pb[j / 2] |= up ? 0u : gb;
                mine |= up ? 2u : 4u;
                hb[j] = 0u;
                if constexpr (RECORDS) {
                    const uint32_t slot = atomicAdd(&pl.rec_cnt[row / kUnitRows], 1u);
                    if (slot < (uint32_t)kRecCap) {
                        uint32_t *rec = pl.recs + ((size_t)(row / kUnitRows) * kRecCap + slot) * 2;
                        rec[0] = ((uint32_t)(k0 + j) << 5) | (uint32_t)(row % kUnitRows);
                        rec[1] = r[j];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) p0[i] = hb[2 * i] | (hb[2 * i + 1] << 16);
    return mine;
}

// Stores what split_planes made: plane 0 always, the planes in `have` (bit 1 above, bit 2 below; agreed on by
// the threads of the unit); the unit's leader writes the mask.
template <class OP>
__device__ __forceinline__ void store_planes(const OP &o, int row, int k0, int kblocks, const u32x4 &p0, const u32x4 &pa,
                                             const u32x4 &pb, uint32_t have, bool leader)
{
    const int rb = row / kUnitRows, rr = row % kUnitRows;
    const int kb = k0 / kUnitK, c = (k0 % kUnitK) / 8;
    const size_t at = unit_vec_index(rb, kb, kblocks, 1, 0, c, rr);
    o.W[at] = p0;
    if (have & 2u) o.W[o.pl.plane + at] = pa;
    if (have & 4u) o.W[2 * o.pl.plane + at] = pb;
    if (leader) o.pl.mask[(size_t)rb * kblocks + kb] = (uint8_t)(1u | have);
}

// Scaled exponent planes of a plain matrix operand (see the top of this file).  Same element-to-thread
// mapping as prepare_block, so a workgroup covers exactly two units; which of them has elements
// outside plane 0 is agreed on through two words of LDS, and only then are the other planes of that
// unit written (the elements that do not belong to a plane are zero there).
template <int MODE, bool FTZ, class OP>
__device__ __forceinline__ void prepare_scaled_block(const OP &o, int K, int kblocks, const QuantParams &p,
                                                     unsigned bid)
{
    __shared__ uint32_t s_planes[2];
    const int tid = threadIdx.x;
    if (tid < 2) s_planes[tid] = 0u;
    const uint32_t *__restrict__ X = o.X;
    const int64_t ld = o.ld;
    const int rows = o.rows;
    const bool kcontig = o.kcontig != 0;
    const int nslabs = kcontig ? (kblocks + 1) / 2 : kblocks;
    const int bx = bid % nslabs, by = bid / nslabs;
    int row, k0, u;                              // u: which of the workgroup's two units this thread works on
    if (kcontig) {
        row = by * 32 + tid / 8;
        k0 = bx * 64 + (tid % 8) * 8;
        u = (tid % 8) / 4;
    } else {
        row = by * 64 + tid % 64;
        k0 = bx * 32 + (tid / 64) * 8;
        u = (tid % 64) / 32;
    }
    const bool live = k0 < kblocks * kUnitK;     // k-contiguous slabs cover two k-blocks; the last may be half
    uint32_t v[8];
    if (live && kcontig && o.vec4 && row < rows && k0 + 8 <= K) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(X + (size_t)row * ld + k0);
        const u32x4 lo = __builtin_nontemporal_load(src), hi = __builtin_nontemporal_load(src + 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = lo[j];
            v[4 + j] = hi[j];
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = k0 + j;
            const bool ok = live && row < rows && k < K;
            const size_t idx = kcontig ? (size_t)row * ld + k : (size_t)k * ld + row;
            v[j] = ok ? X[idx] : 0u;
        }
    }
    uint32_t r[8];
    u32x4 p0, pa, pb;
    quantize_run<MODE, FTZ>(v, run_is_rare(v, p), p, round_masks(p), r);
    const uint32_t mine = split_planes(o.pl, o.pl.S[row], row, k0, r, p0, pa, pb);      // S covers the padded rows
    __syncthreads();                             // s_planes has been cleared
    if (mine != 0u) atomicOr(&s_planes[u], mine);
    __syncthreads();
    if (!live) return;
    store_planes(o, row, k0, kblocks, p0, pa, pb, s_planes[u],
                 kcontig ? (tid / 8 == 0 && tid % 4 == 0) : (tid / 64 == 0 && tid % 32 == 0));
}

// Both orientations of one tile of a plain matrix X -- 32 rows (32 ty ..) by 64 columns (64 tx ..) -- as scaled
// exponent planes: o0 is X as stored (its rows are X's, k runs along X's columns), o1 is X transposed.  The
// tile is one workgroup's share of either operand in prepare_scaled_block; it is read and rounded once, and the
// rounded patterns cross over to that function's mappings (a row's eight consecutive columns per
// thread, a column's eight consecutive rows) through LDS.
// A workgroup takes kPairTiles tiles side by side (columns 64 tx0 ..): all their loads are issued before the first
// is worked on (measured: two tiles 2 - 4 % faster than one, four slower than two).
constexpr int kPairTiles = 2;

// ROUND: the pass also does what fmt_quantize does with the tensor -- the rounded values go to Y (leading
// dimension ldy) as fp32 and every element of X is counted in the workgroup's statistics table (tbl, w).
constexpr int kPairCopies = 8;                          // replicas of the statistics table (lane l uses l % 8)
constexpr int kRoundSteps = 4;                          // steps of kPairTiles tiles per workgroup of a ROUND launch, at most

template <int MODE, bool FTZ, bool ROUND, bool DEEP, class OP>
__device__ __forceinline__ void prepare_pair_tile(const OP &o0, const OP &o1, const QuantParams &p, int ty, int tx0,
                                                  uint32_t *Y, int64_t ldy, uint32_t *tbl, Counts &w)
{
    __shared__ __align__(16) uint32_t s_r[32][68];      // 68: rows stay 16-byte aligned, 128-bit writes spread over all banks
    __shared__ uint32_t s_planes[4 * kPairTiles];       // per tile: o0's two units (halves of k), then o1's two (halves of its rows)
    const int tid = threadIdx.x;
    if (tid < 4 * kPairTiles) s_planes[tid] = 0u;
    const RoundMasks masks = round_masks(p);
    const int R = o0.rows, C = o1.rows;                 // X is R x C
    // X is read, and Y written, 16 bytes per lane and side by side: four columns of two rows per thread.  With a row's eight
    // consecutive columns per thread, as o0 wants them, every instruction covers half lines (12 tensors of 4 M to 16 M elements, ROUND:
    // 572 -> 545 us with the products).  512 instead of 256 bytes of a row per instruction: 160 -> 167 us for the launch.
    const int rr = ty * 32 + tid / 16, cc = (tid % 16) * 4;
    uint32_t v[kPairTiles][8];
#pragma unroll
    for (int n = 0; n < kPairTiles; ++n) {
        const int xc = (tx0 + n) * 64 + cc;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = rr + 16 * h;
            if (o0.vec4 && row < R && xc + 4 <= C) {
                const u32x4 w4 = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(o0.X + (size_t)row * o0.ld + xc));
#pragma unroll
                for (int j = 0; j < 4; ++j) v[n][4 * h + j] = w4[j];
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[n][4 * h + j] = (row < R && xc + j < C) ? o0.X[(size_t)row * o0.ld + xc + j] : 0u;
            }
        }
    }
    const int xr = ty * 32 + tid / 8;                   // o0's mapping
#pragma unroll
    for (int n = 0; n < kPairTiles; ++n) {
        const int tx = tx0 + n;
        const int xc = tx * 64 + (tid % 8) * 8;
        {
            uint32_t q[8];
            bool rare;
            if (ROUND && ty * 32 + 32 <= R && tx * 64 + 64 <= C) {       // the whole tile lies in X: the same in the workgroup
                uint32_t amax = 0u;
#pragma unroll
                for (int j = 0; j < 8; ++j) account_run<DEEP, kPairCopies>(v[n][j] & 0x7FFFFFFFu, p, tbl, (uint32_t)tid % kPairCopies, w, amax);
                account_run_top(v[n], amax, p, w);
                rare = amax >= p.t_ovf;
            } else {
                if constexpr (ROUND) {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        account<DEEP, kPairCopies>(v[n][j] & 0x7FFFFFFFu, rr + 4 * (j & 4) < R && tx * 64 + cc + (j & 3) < C, p, tbl,
                                                   (uint32_t)tid % kPairCopies, w);
                }
                rare = run_is_rare(v[n], p);
            }
            quantize_run<MODE, FTZ>(v[n], rare, p, masks, q);
            const bool vec = ROUND && ((reinterpret_cast<uintptr_t>(Y) | (uintptr_t)(ldy * 4)) & 15) == 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 q4{q[4 * h], q[4 * h + 1], q[4 * h + 2], q[4 * h + 3]};
                if constexpr (ROUND) {
                    const int row = rr + 16 * h, col = tx * 64 + cc;
                    uint32_t *dst = Y + (size_t)row * ldy + col;
                    if (row < R && vec && col + 4 <= C) {
                        __builtin_nontemporal_store(q4, reinterpret_cast<u32x4 *>(dst));
                    } else if (row < R) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (col + j < C) dst[j] = q4[j];
                    }
                }
                // (the reads of the tile before this one ended before that tile's second barrier)
                *reinterpret_cast<u32x4 *>(&s_r[tid / 16 + 16 * h][cc]) = q4;
            }
        }
        __syncthreads();
        // beyond an operand's k-blocks there is nothing of it to write (the other operand's padded rows lie there)
        const bool do0 = tx < (o0.kblocks + 1) / 2, do1 = ty < o1.kblocks;
        const bool live0 = do0 && xc < o0.kblocks * kUnitK;       // the last slab of o0 may hold one k-block only
        const int row1 = tx * 64 + tid % 64, k1 = ty * 32 + (tid / 64) * 8;
        const int u0 = 4 * n + (tid % 8) / 4, u1 = 4 * n + 2 + (tid % 64) / 32;
        // (where an operand has nothing to write the tile holds zeros only and its rows are padded ones, whose
        // scales exist: the split is harmless there and leaves no records)
        uint32_t r[8], t[8];
        u32x4 p0a, paa, pba, p0b, pab, pbb;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x4 r4 = *reinterpret_cast<const u32x4 *>(&s_r[tid / 8][(tid % 8) * 8 + 4 * h]);
#pragma unroll
            for (int j = 0; j < 4; ++j) r[4 * h + j] = r4[j];
        }
        const uint32_t mine0 = split_planes(o0.pl, o0.pl.S[xr], xr, xc, r, p0a, paa, pba);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = s_r[(tid / 64) * 8 + j][tid % 64];
        const uint32_t mine1 = split_planes(o1.pl, o1.pl.S[row1], row1, k1, t, p0b, pab, pbb);
        if (mine0 != 0u) atomicOr(&s_planes[u0], mine0);
        if (mine1 != 0u) atomicOr(&s_planes[u1], mine1);
        __syncthreads();
        if (live0) store_planes(o0, xr, xc, o0.kblocks, p0a, paa, pba, s_planes[u0], tid / 8 == 0 && tid % 4 == 0);
        if (do1) store_planes(o1, row1, k1, o1.kblocks, p0b, pab, pbb, s_planes[u1], tid / 64 == 0 && tid % 32 == 0);
    }
}

// One launch prepares both operands of a product (or one: b.nblocks == 0).
template <int MODE, bool FTZ, int PS, bool TAPS>
__global__ __launch_bounds__(256) void prepare_kernel(PrepOperand a, PrepOperand b, int K, int kblocks, QuantParams p)
{
    prepare_block<MODE, FTZ, PS, TAPS>(a, b, K, kblocks, p, blockIdx.x);
}

// What a product needs that gathers its patches itself, in one launch: the filter as a prepared operand (workgroups below
// split_first) and the tensor in pixel-major pieces (the others, nx of them along the pixels).  Two launches of 6 and 8 us before.
template <int MODE, bool FTZ, int PS>
__global__ __launch_bounds__(256) void prepare_implicit_kernel(PrepOperand a, int K, int kblocks, unsigned split_first, unsigned nx,
                                                               const uint32_t *__restrict__ x, u32x4 *__restrict__ out, int C, int HW,
                                                               int npix, QuantParams p)
{
    if (blockIdx.x < split_first) {              // workgroup-uniform
        PrepOperand none = a;
        none.nblocks = 0u;
        prepare_block<MODE, FTZ, PS>(a, none, K, kblocks, p, blockIdx.x);
    } else {
        const unsigned id = blockIdx.x - split_first;
        nhwc_split_block<MODE, FTZ, PS>(x, out, C, HW, npix, p, (int)(id % nx), (int)(id / nx));
    }
}

// The two for exponent planes with one scale per tensor: an operand whose elements gather8 finds (k along the lanes), in the layout that
// prepare_scaled_block writes, ...  look() gives what window_pair found, behind a barrier of the workgroup.  Of wide tensors: two bf16 pieces, laid
// out as prepare_block and nhwc_split_block have them.
template <int MODE, bool FTZ, class LOOK>
__device__ __forceinline__ void prepare_window_block(const PrepOperand &o, LOOK &&look, int K, int kblocks, const QuantParams &p, unsigned bid)
{
    __shared__ uint32_t s_planes[2];
    const int tid = threadIdx.x;
    if (tid < 2) s_planes[tid] = 0u;
    const int nslabs = (kblocks + 1) / 2;
    const int row = (int)(bid / (unsigned)nslabs) * 32 + tid / 8, k0 = (int)(bid % (unsigned)nslabs) * 64 + (tid % 8) * 8;
    const int u = (tid % 8) / 4;                 // which of the workgroup's two units
    int idx[8];
    uint32_t v[8], r[8];
    gather8(o, row, k0, K, idx);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = idx[j] >= 0 ? o.X[(uint32_t)idx[j]] : 0u;
    const WindowPair pair = look();                          // its barrier: s_planes has been cleared
    if (pair.wide) {                                         // the same in the whole launch
        u32x4 w[2];
        split8<MODE, FTZ, 2>(v, p, w);
        if (k0 >= kblocks * kUnitK) return;
#pragma unroll
        for (int q = 0; q < 2; ++q) o.W[unit_vec_index(row / kUnitRows, k0 / kUnitK, kblocks, 2, q, k0 % kUnitK / 8, row % kUnitRows)] = w[q];
        return;
    }
    u32x4 p0, pa, pb;
    quantize_run<MODE, FTZ>(v, run_is_rare(v, p), p, round_masks(p), r);
    const uint32_t mine = split_planes<false>(o.pl, pair.S[0], row, k0, r, p0, pa, pb);
    if (mine != 0u) atomicOr(&s_planes[u], mine);
    __syncthreads();
    if (k0 < kblocks * kUnitK) store_planes(o, row, k0, kblocks, p0, pa, pb, s_planes[u], tid / 8 == 0 && tid % 4 == 0);
}

// ... and a tensor in pixel-major order, out[plane][pixel][channel] (nhwc_split_block), with the masks of 64 pixels x 32 channels.
// Planes above and below are written where these are not zero.  (Fewer workgroups that take several blocks, and the sample once: 77
// registers instead of 57, 11.8 us instead of 11.3.)
template <int MODE, bool FTZ>
__device__ __forceinline__ void nhwc_window_block(const WindowTensor &ta, const WindowTensor &t, int adapt, u32x4 *__restrict__ out, const Planes &pl,
                                                  int C, int HW, int npix, const QuantParams &p, int bx, int cb)
{
    constexpr int kPitch = 18;
    __shared__ uint32_t tile[64][kPitch];
    __shared__ unsigned long long s_have[2];
    const int tid = threadIdx.x;
    if (tid < 2) s_have[tid] = 0ull;
    const int pix = tid % 64, cg = tid / 64;
    const int gp = bx * 64 + pix;
    const bool valid = gp < npix;
    const int n = valid ? gp / HW : 0, hw = valid ? gp - n * HW : 0;
    const uint32_t *src = t.x + ((size_t)n * C + cb * 32 + cg * 8) * HW + hw;
    uint32_t u[8], r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) u[i] = valid ? src[(size_t)i * HW] : 0u;
    const WindowPair pair = window_pair(ta, t, adapt);       // its barrier: s_have has been cleared
    u32x4 pc[3];
    uint32_t mine = 0u;
    if (pair.wide) {                                         // the same in the whole launch
        u32x4 w[2];
        split8<MODE, FTZ, 2>(u, p, w);
        pc[0] = w[0], pc[1] = w[1], pc[2] = w[1];
    } else {
        quantize_run<MODE, FTZ>(u, run_is_rare(u, p), p, round_masks(p), r);
        mine = split_planes<false>(pl, pair.S[1], 0, 0, r, pc[0], pc[1], pc[2]);
    }
    if (__ballot(mine != 0u) != 0ull) {
        const unsigned long long above = __ballot((mine & 2u) != 0u), below = __ballot((mine & 4u) != 0u);      // a lane per pixel
        if (pix == 0) {
            atomicOr(&s_have[0], above);
            atomicOr(&s_have[1], below);
        }
    }
    const int opix = tid / 4, part = tid % 4;
    const int ogp = bx * 64 + opix;
    const size_t piece_vec = (size_t)npix * (C / 8);
    uint32_t have = 1u;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (!((have >> q) & 1u)) continue;       // the same in the whole workgroup
        if (q > 0) __syncthreads();              // the plane before has been read
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[pix][cg * 4 + i] = pc[q][i];
        __syncthreads();
        if (q == 0) have = pair.wide ? 3u : 1u | (s_have[0] != 0ull ? 2u : 0u) | (s_have[1] != 0ull ? 4u : 0u);
        if (ogp < npix) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = tile[opix][part * 4 + i];
            out[q * piece_vec + (size_t)ogp * (C / 8) + cb * 4 + part] = w;
        }
    }
    if (tid < 2) reinterpret_cast<unsigned long long *>(pl.mask)[((size_t)bx * (C / 32) + cb) * 2 + tid] = s_have[tid];
    if (bx == 0 && cb == 0 && tid == 0) {
        pl.S[0] = pair.S[1];
        out[3 * piece_vec] = u32x4{0u, 0u, 0u, 0u};
    }
}

template <int MODE, bool FTZ>
__global__ __launch_bounds__(256) void prepare_implicit_window_kernel(PrepOperand a, WindowTensor ta, int K, int kblocks, unsigned split_first,
                                                                      unsigned nx, WindowTensor tb, int adapt, u32x4 *__restrict__ out, Planes pl,
                                                                      int C, int HW, int npix, QuantParams p)
{
    if (blockIdx.x < split_first) {              // workgroup-uniform, as are the returns
        const unsigned per_xcd = split_first / 8u, bid = (blockIdx.x % 8u) * per_xcd + blockIdx.x / 8u;
        if (bid >= a.nblocks) return;
        prepare_window_block<MODE, FTZ>(a, [&]() __attribute__((always_inline)) {
            const WindowPair pair = window_pair(ta, tb, adapt);
            if (bid == 0u && threadIdx.x == 0) {
                a.pl.S[0] = pair.S[0];
                a.pl.S[1] = pair.wide ? 1 : 0;
            }
            return pair;
        }, K, kblocks, p, bid);
    } else {
        const unsigned id = blockIdx.x - split_first;
        nhwc_window_block<MODE, FTZ>(ta, tb, adapt, out, pl, C, HW, npix, p, (int)(id % nx), (int)(id / nx));
    }
}

// The operands of the weight gradient: a as above, b gathered from a tensor of words (round_window_kernel, which left the scales).
template <int MODE, bool FTZ>
__global__ __launch_bounds__(256) void prepare_taps_window_kernel(PrepOperand a, PrepOperand b, int K, int kblocks, QuantParams p)
{
    const unsigned a_ids = (a.nblocks + 7u) / 8u * 8u;
    const bool second = blockIdx.x >= a_ids;
    const unsigned lid = blockIdx.x - (second ? a_ids : 0u), nblocks = second ? b.nblocks : a.nblocks;
    const unsigned bid = (lid % 8u) * ((nblocks + 7u) / 8u) + lid / 8u;
    if (bid >= nblocks) return;                  // workgroup-uniform: before any barrier
    const WindowPair pair{{a.pl.S[0], 0}, a.pl.S[1] != 0};
    if (second) {
        gather_taps<1, true>(b, bid, K, kblocks, pair.wide);
        return;
    }
    prepare_window_block<MODE, FTZ>(a, [&]() __attribute__((always_inline)) {
        __syncthreads();
        return pair;
    }, K, kblocks, p, bid);
}

template <int MODE, bool FTZ>
__global__ __launch_bounds__(256) void prepare_scaled_kernel(PrepOperand a, PrepOperand b, int Ka, int kblocks_a, int Kb,
                                                             int kblocks_b, QuantParams p)
{
    // operands own runs of workgroup ids padded to a multiple of 8, remapped XCD by XCD as in prepare_block
    const unsigned a_ids = (a.nblocks + 7u) / 8u * 8u;
    const bool second = blockIdx.x >= a_ids;
    const PrepOperand &o = second ? b : a;
    const unsigned lid = blockIdx.x - (second ? a_ids : 0u);
    const unsigned per_xcd = (o.nblocks + 7u) / 8u;
    const unsigned bid = (lid % 8u) * per_xcd + lid / 8u;
    if (bid >= o.nblocks) return;                // workgroup-uniform: before any barrier
    prepare_scaled_block<MODE, FTZ>(o, second ? Kb : Ka, second ? kblocks_b : kblocks_a, p, bid);
}

// The exponent planes of both orientations of up to kMaxPrepGroup / 2 plain matrices in one launch.  Operands
// 2i (X as stored: rows of X, k along its columns) and 2i + 1 (X transposed) belong to matrix i; the table
// travels by value in the kernel arguments.  A workgroup takes tiles of 32 rows x 64 columns of X and
// prepares them for both operands (prepare_pair_tile): X is read and rounded once.  Every
// matrix owns a run of workgroup ids padded to a multiple of 8 (first[] = the runs' first ids, ascending).
// Tiles go to the workgroups in id order, and a workgroup's further steps are a whole run of workgroups on, so that what the chip works
// on at a time is one stretch of X, Y and the planes: memory takes that at 6.0 TB/s (964 MB in 160 us), and at 4.8 (198) with the
// ids remapped to give each XCD a stretch of its own and a workgroup consecutive tiles.  No line is used twice here.
constexpr int kMaxPrepGroup = 32;

struct PrepPlain {
    const uint32_t *X;
    u32x4 *W;
    int64_t ld;
    int rows;
    int kcontig;
    int vec4;
    int units;
    int K, kblocks;
    Planes pl;
};

struct PrepGroup {
    unsigned first[kMaxPrepGroup / 2];   // 0xFFFFFFFF beyond the last matrix
    unsigned tiles[kMaxPrepGroup / 2];
    PrepPlain o[kMaxPrepGroup];
};

// index of the run that holds workgroup `id`: the number of runs that start at or before it, minus one
// (first[] ascending, 0xFFFFFFFF beyond the last run)
template <int CAP>
__device__ __forceinline__ int run_of(const unsigned (&first)[CAP], unsigned id)
{
    int at = -1;
#pragma unroll
    for (int i = 0; i < CAP; ++i) at += id >= first[i] ? 1 : 0;
    return at;
}

// what the ROUND variant needs of every matrix: the rounded fp32 copy and the partial statistics records
struct RoundGroup {
    uint32_t *Y[kMaxPrepGroup / 2];
    int64_t ldy[kMaxPrepGroup / 2];
    unsigned long long *hist[kMaxPrepGroup / 2];     // the callers' records
    unsigned long long *records;                     // kSetWords words of partial records per matrix
    int steps;                                   // steps of kPairTiles tiles per workgroup
};

template <int MODE, bool FTZ, bool ROUND, bool DEEP>
__global__ __launch_bounds__(256) void prepare_scaled_group_kernel(PrepGroup grp, RoundGroup rg, QuantParams p)
{
    __shared__ __align__(16) uint32_t tbl[ROUND ? kHistRows * kPairCopies : 4];
    __shared__ uint32_t s_bins[ROUND ? FMT_NBINS : 1], s_cls[ROUND ? 8 : 1];
    const int at = __builtin_amdgcn_readfirstlane(run_of(grp.first, blockIdx.x));
    const PrepPlain &o0 = grp.o[2 * at], &o1 = grp.o[2 * at + 1];
    // ROUND: a workgroup takes up to kRoundSteps consecutive steps of kPairTiles tiles, so that clearing and folding
    // its statistics table is paid once per 16 K elements (as in the stream kernels); fewer when the launch is small
    const unsigned kSteps = ROUND ? (unsigned)rg.steps : 1u;
    const unsigned lid = blockIdx.x - grp.first[at], ntiles = grp.tiles[at];
    const unsigned nwg = (ntiles + kSteps - 1u) / kSteps;
    const unsigned g = lid;
    if (g >= nwg) return;                        // workgroup-uniform: before any barrier
    // rows of X in 32s: o0's units (rows padded to the tile grid) cover o1's k-blocks; columns of X in 64s:
    // pairs of o1's units cover o0's slabs of two k-blocks
    const int ntx = o1.units / (2 * kPairTiles);
    Counts w;
    if constexpr (ROUND) hist_begin<kPairCopies, 256>(tbl, s_bins, s_cls, threadIdx.x);
#pragma unroll 1
    for (unsigned step = 0; step < kSteps; ++step) {
        const unsigned t = g + step * nwg;
        if (t >= ntiles) break;                  // workgroup-uniform
        if (step > 0) __syncthreads();           // the step before has read its words of LDS
        const int ty = (int)(t / (unsigned)ntx), tx = (int)(t % (unsigned)ntx) * kPairTiles;
        prepare_pair_tile<MODE, FTZ, ROUND, DEEP>(o0, o1, p, ty, tx, ROUND ? rg.Y[at] : nullptr, ROUND ? rg.ldy[at] : 0, tbl, w);
    }
    if constexpr (ROUND)
        hist_end<kPairCopies, 256>(tbl, s_bins, s_cls, w, p,
                                   HistSink{rg.records + (size_t)at * kSetWords, rg.hist[at],
                                            (unsigned long long)o0.rows * (unsigned long long)o1.rows, (uint32_t)kShards, 0u, nullptr},
                                   g, nwg, threadIdx.x);
}

__global__ __launch_bounds__(256) void planes_tail_kernel(const u32x4 *__restrict__ Aw, const u32x4 *__restrict__ Bw, Planes pa,
                                                          Planes pb, float *__restrict__ C, int64_t ldc, int M, int N, int kblocks,
                                                          int col_chunks, int tail_cols)
{
    __shared__ TailLds lds;
    planes_tail_body(Aw, Bw, pa, pb, C, ldc, M, N, kblocks, (int)blockIdx.x / col_chunks, (int)blockIdx.x % col_chunks * tail_cols, tail_cols,
                     lds);
}

// The tails of a group of products in one launch: blocks [first, next first) belong to product g.
struct TailGroupItem {
    const u32x4 *Aw, *Bw;
    float *C;
    int64_t ldc;
    int M, N, kblocks, col_chunks;
    unsigned first;
    Planes pa, pb;
};
struct TailGroup {
    int count, tail_cols;
    unsigned first[kMaxGroup];
    TailGroupItem p[kMaxGroup];
};

__global__ __launch_bounds__(256) void planes_tail_group_kernel(TailGroup grp)
{
    const TailGroupItem &it = grp.p[group_member(grp.first, blockIdx.x)];  // the same in the whole workgroup
    __shared__ TailLds lds;
    const int bid = (int)(blockIdx.x - it.first);
    planes_tail_body(it.Aw, it.Bw, it.pa, it.pb, it.C, it.ldc, it.M, it.N, it.kblocks, bid / it.col_chunks, bid % it.col_chunks * grp.tail_cols,
                     grp.tail_cols, lds);
}

// Columns per tail block for a launch whose blocks would number `blocks256` at 256 columns each: the widest
// of 1024, 512, 256 that still leaves four blocks per resident slot (three workgroups per compute unit).
static int tail_cols_for(uint64_t blocks256, int cus)
{
    if (const char *env = getenv("FMT_GEMM_TAIL_COLS")) {        // tuning override
        const int t = atoi(env);
        if (t == 256 || t == 512 || t == 1024) return t;
    }
    const uint64_t want = (uint64_t)cus * 12;
    return blocks256 / 4 >= want ? 1024 : blocks256 / 2 >= want ? 512 : 256;
}

int launch_planes_tail(const u32x4 *Aw, const u32x4 *Bw, const Planes &pa, const Planes &pb, float *C, int64_t ldc, int M, int N,
                       int kblocks, hipStream_t stream)
{
    int cus = 0;
    const int rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    const int64_t rbs = (M + kUnitRows - 1) / kUnitRows;
    const int tc = tail_cols_for((uint64_t)rbs * ((N + 255) / 256), cus);
    const int64_t col_chunks = (N + tc - 1) / tc, blocks = rbs * col_chunks;
    if (blocks >= ((int64_t)1 << 31)) return FMT_ERR_SHAPE;
    hipLaunchKernelGGL(planes_tail_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, Aw, Bw, pa, pb, C, ldc, M, N, kblocks,
                       (int)col_chunks, tc);
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

// C[r][c] = sum over the k parts of part[s][r][c]  (parts are dense M x N slabs), in part order.  Four neighbouring elements
// per thread, the slabs' loads issued U at a time: what bounds the kernel is the latency of its loads (256 x 2304 in eight
// parts: 10.9 us with one element and one load at a time, 5.3 with these).  U is the number of parts up to four, then
// eight; an element's place in C takes one division, in 32 bits where they suffice.
template <int U>
__global__ __launch_bounds__(256) void reduce_kernel(const float *__restrict__ part, int nsplit, float *__restrict__ C,
                                                     int M, int N, int64_t ldc, int img)
{
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const size_t total = (size_t)M * N;
    for (size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4; i < total; i += (size_t)gridDim.x * 1024) {
        const bool four = i + 4 <= total;
        const size_t last = total >= 4 ? total - 4 : 0;
        float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int q0 = 0; q0 < nsplit; q0 += U) {
            float v[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // the last elements are loaded as the last four and moved down (fewer than four in all: one by one)
                const float *src = part + (size_t)min(q0 + u, nsplit - 1) * total + (four ? i : last);
                if (total >= 4) {
                    const f32x4u w = *reinterpret_cast<const f32x4u *>(src);
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[u][j] = w[j];
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[u][j] = j < (int)total ? src[j] : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (q0 + u < nsplit) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) s[j] += v[u][j];
                }
        }
        if (!four) {
            const int by = (int)(i - last);
            if (by & 1) s[0] = s[1], s[1] = s[2], s[2] = s[3];
            if (by & 2) s[0] = s[2], s[1] = s[3];
        }
        size_t row = total >> 32 == 0 ? (uint32_t)i / (uint32_t)N : i / N;
        int col = (int)(i - row * N);
        if (img == 0 && four && col + 4 <= N) {
            *reinterpret_cast<f32x4u *>(C + row * ldc + col) = f32x4u{s[0], s[1], s[2], s[3]};
            continue;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i + j >= total) break;
            if (img > 0)
                C[((size_t)(col / img) * M + row) * img + col % img] = s[j];
            else
                C[row * ldc + col] = s[j];
            if (++col == N) {
                col = 0;
                ++row;
            }
        }
    }
}

int launch_reduce(const float *part, int nsplit, float *C, int M, int N, int64_t ldc, int img, hipStream_t stream)
{
    const size_t groups = ((size_t)M * N + 1023) / 1024;
    auto kern = nsplit <= 2 ? reduce_kernel<2> : nsplit == 3 ? reduce_kernel<3> : nsplit == 4 ? reduce_kernel<4> : reduce_kernel<8>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(groups < 4096 ? groups : 4096)), dim3(256), 0, stream, part, nsplit, C, M, N, ldc, img);
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

__global__ void zero_fill_kernel(float *__restrict__ C, int M, int N, int64_t ldc, int col_blocks)
{
    const int col = (blockIdx.x % col_blocks) * blockDim.x + threadIdx.x;
    const int row = blockIdx.x / col_blocks;
    if (col < N && row < M) C[(size_t)row * ldc + col] = 0.0f;
}

// Picks the workgroup tile and the number of k parts from a small cost model fitted to
// measurements on MI355X: large tiles move fewer LDS and L2 bytes per MFMA, small tiles need
// several resident workgroups per compute unit to reach their rate, the busiest compute unit sets
// the time, and cutting k fills the machine at the price of writing and re-reading partial sums.
// most: the largest tile, in 64 x 64 (a forced plan may be larger).
static Plan make_plan(int M, int N, int kblocks, int cus, int pieces, int most = 16)
{
    // eff1 / effmax: relative MFMA rate of a compute unit with one / with max_occ resident workgroups
    struct Shape { int tm, tn, max_occ; double eff1, effmax; };
    static const Shape multi[5] = {
        {4, 4, 1, 1.15, 1.15}, {4, 2, 1, 1.0, 1.0}, {2, 4, 1, 1.03, 1.03}, {2, 2, 2, 0.80, 0.95}, {1, 1, 4, 0.45, 0.78}};
    // one piece: a quarter of the MFMA work per byte, the small tiles lose less
    static const Shape single[5] = {
        {4, 4, 1, 1.21, 1.21}, {4, 2, 1, 1.0, 1.0}, {2, 4, 1, 1.03, 1.03}, {2, 2, 2, 0.98, 1.11}, {1, 1, 4, 0.53, 0.68}};
    const Shape(&shapes)[5] = pieces == 1 ? single : multi;
    const double wg_cost = pieces == 1 ? 68.0 : 40.0, split_cost = pieces == 1 ? 5.76 : 2.5;
    if (const char *env = getenv("FMT_GEMM_PLAN")) {      // tuning override: "tm,tn,nsplit[,sched]" (other values leave the plan to the model)
        Plan forced{2, 2, 1, 1, cus, true};
        if (sscanf(env, "%d,%d,%d,%d", &forced.tm, &forced.tn, &forced.nsplit, &forced.sched) >= 3) {
            bool known = forced.tm == 2 && forced.tn == 1;        // layers only (layer_plan); other products take 64 x 64 then
            for (const auto &sh : shapes) known = known || (sh.tm == forced.tm && sh.tn == forced.tn);
            if (known && forced.nsplit >= 1 && forced.nsplit <= 64 &&
                lds_bytes(forced.tm, forced.tn, pieces, pipe_ks(pieces), 2) <= 160 * 1024)
                return forced;
        }
    }
    Plan best{2, 2, 1, 1, cus};
    double best_t = 1e300;
    for (const auto &sh : shapes) {
        if (sh.tm * sh.tn > most || lds_bytes(sh.tm, sh.tn, pieces, pipe_ks(pieces), 2) > 160 * 1024) continue;
        const int bm = 64 * sh.tm, bn = 64 * sh.tn;
        const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        for (int ns = 1; ns <= 32; ns = ns < 4 ? ns + 1 : ns * 2) {
            if (ns > 1 && kblocks / ns < 8) break;
            const int kb_per = (kblocks + ns - 1) / ns;
            const long wgs = tiles * ns;
            const long per_cu = (wgs + cus - 1) / cus;                  // workgroups on the busiest compute unit
            const long resident = per_cu < sh.max_occ ? per_cu : sh.max_occ;
            const double eff = sh.max_occ > 1 ? sh.eff1 + (sh.effmax - sh.eff1) * (resident - 1) / (sh.max_occ - 1) : sh.eff1;
            // MFMA time on that compute unit (arbitrary units) + start-up / epilogue cost per workgroup
            double t = per_cu * ((double)bm * bn * kb_per / eff + wg_cost * bm * bn / 128.0);
            if (ns > 1) t += split_cost * (double)M * N * (ns + 1) / cus * 8.0;   // partial sums out and back
            if (t < best_t) { best_t = t; best = Plan{sh.tm, sh.tn, ns, 1, cus}; }
        }
    }
    return best;
}

// One operand of a product as the caller describes it: a plain matrix (kind kSrcMatrix, leading
// dimension ld) or a gathered view of a convolution tensor.
struct OperandSpec {
    const float *X;
    int64_t ld;
    bool kcontig;
    Gather g;
    int64_t pre_elems;   // > 0: round and split the tensor (that many elements) once before gathering from it
};

// How a format's values reach the matrix cores: ps = piece scheme (0: one fp16 piece, 1-3: that many
// bf16 pieces); scaled: ps == 0 with per-row scales and exponent planes (1/6/8 and 1/6/9).
struct Scheme {
    int ps;
    bool scaled;
};

// 0: never scaled planes, 1: whenever the format allows, 2: by size.  Environment override for tests and tuning (3: as 1, but a
// convolution's samples may still choose pieces, see window_adapts).
static int window_mode()
{
    if (const char *env = getenv("FMT_GEMM_WINDOW")) return env[0] == '0' ? 0 : (env[0] == '1' || env[0] == '3' ? 1 : 2);
    return 2;
}

static bool planes_possible(fmt_format_t f) { return f.e == 6 && f.m >= 8 && f.m <= 9; }

static Scheme scheme_of(fmt_format_t f, bool want_planes)
{
    if (want_planes && planes_possible(f)) return Scheme{0, true};
    // one fp16 piece for formats inside binary16, else 1-3 bf16 pieces by significand width
    return Scheme{f.m <= 7 ? 1 : (f.e <= 5 && f.m <= 10 ? 0 : (f.m <= 15 ? 2 : 3)), false};
}

// Memory layout of one prepared operand (`rows` x K after op(), padded to kRowPad rows and 32 k):
//   [pieces]  units x kblocks x P units of 128 vectors; with planes: three planes of units x kblocks units
//   [S]       with planes: one int per padded row
//   [mask]    with planes: one byte per unit
// every part 256-byte aligned.
struct OperandLayout {
    Scheme sch;
    int w;                       // planes: binades per plane
    int rows, kblocks, units;
    size_t plane_vec, s_off, mask_off, cnt_off, rec_off, bytes;
};

static int operand_layout(int64_t rows, int64_t K, Scheme sch, int m, OperandLayout *L)
{
    auto up256 = [](size_t b) { return (b + 255) / 256 * 256; };
    L->sch = sch;
    L->w = 40 - m;
    L->rows = (int)rows;
    L->kblocks = (int)((K + kUnitK - 1) / kUnitK);
    L->units = (int)((rows + kRowPad - 1) / kRowPad * (kRowPad / kUnitRows));
    if ((int64_t)L->kblocks * L->units >= ((int64_t)1 << 30)) return FMT_ERR_SHAPE;
    const int P = pieces_of(sch.ps);
    L->plane_vec = (size_t)L->units * L->kblocks * P * kUnitVec;
    const size_t piece_bytes = up256(L->plane_vec * sizeof(u32x4) * (sch.scaled ? 3 : 1));
    L->s_off = piece_bytes;
    L->mask_off = L->s_off + (sch.scaled ? up256((size_t)L->units * kUnitRows * sizeof(int)) : 0);
    L->cnt_off = L->mask_off + (sch.scaled ? up256((size_t)L->units * L->kblocks) : 0);
    L->rec_off = L->cnt_off + (sch.scaled ? up256((size_t)L->units * sizeof(uint32_t)) : 0);
    L->bytes = L->rec_off + (sch.scaled ? up256((size_t)L->units * kRecCap * 2 * sizeof(uint32_t)) : 0);
    return FMT_OK;
}

static OperandView view_of(void *base, const OperandLayout &L)
{
    char *b = static_cast<char *>(base);
    OperandView v;
    v.W = reinterpret_cast<u32x4 *>(b);
    v.pl = Planes{nullptr, nullptr, 0, L.w, nullptr, nullptr};
    if (L.sch.scaled) {
        v.pl.S = reinterpret_cast<int *>(b + L.s_off);
        v.pl.mask = reinterpret_cast<uint8_t *>(b + L.mask_off);
        v.pl.plane = L.plane_vec;
        v.pl.rec_cnt = reinterpret_cast<uint32_t *>(b + L.cnt_off);
        v.pl.recs = reinterpret_cast<uint32_t *>(b + L.rec_off);
    }
    return v;
}

// ---- exponent planes: the scale of every row -------------------------------------------------

struct StatOperand {
    const uint32_t *X;
    int64_t ld;
    int rows;
    int rows_pad;
    int kcontig;
    int vec4;                // base 16-byte aligned and ld a multiple of 4: a k-contiguous row is read in 16-byte pieces
    int *S;
    uint32_t *rec_cnt;       // record counts of the operand's rows of units: cleared here, filled by the prepare pass
    unsigned nblocks;
};

// Picks each row's scale S = 15 - T, T the top binade of plane 0, from the binades of a sample of its
// elements (every kstep-th slab of k).  Plane 0 with top T holds the normal values of binades
// [T - wid, T] exactly, and the format's denormal values (multiples of 2^(Emin-m)) exactly iff
// T <= 9 - m.  With hi the largest binade seen (+1: rounding may carry) and lo the smallest binade of
// a value that is normal in the format, every T in [hi + 1, lo + wid] keeps all elements seen in plane 0:
//   - a denormal value was seen: T = 9 - m, the highest choice that keeps the denormals (gradient
//     tensors live here);
//   - otherwise up to four binades above hi + 1 (not beyond the middle of [hi + 1, lo + wid]),
//     which leaves room on both sides for the elements the sample did not see; if the row spans
//     more than a plane, T = lo + wid (the small values stay, the large ones go to the plane above).
// Any T in [kWinTmin, kWinTmax] is correct -- what does not fit plane 0 goes to another plane -- the
// choice only decides how often the other planes are needed, which is why a sample suffices: kStatSlabs * 64 = 128 elements of a
// row with four binades of room leave no more outside plane 0 than 256 with three (log2|x| ~ N(mu, 3^2 .. 6^2) around the format's
// middle, rows of 4096: 2e-5 .. 2e-2 either way; normal and uniform rows: none; where denormals are met: the same), and the
// launch, which reads its sample in pieces of 128 and 256 bytes from all over the tensors, is the shorter.
constexpr int kStatSlabs = 2;
__device__ __forceinline__ void window_stats_block(const StatOperand &o, int K, int kstep, int emin, int m, int by)
{
    __shared__ int s_hi[8][32], s_lo[8][32];
    const int tid = threadIdx.x;
    int hi = kNoBinade, lo = 1000;
    auto look = [&](uint32_t u) { window_look(u, emin, m, hi, lo); };
    // 32 rows per workgroup, 8 lanes per row; eight loads are issued before any is looked at
    const int row = by * 32 + (o.kcontig ? tid / 8 : tid % 32);
    const int kl = o.kcontig ? tid % 8 : tid / 32;
    if (row < o.rows) {
        // at most kStatSlabs slabs of 64 k are visited (kstep = ceil(slabs / kStatSlabs)); all their loads are issued first
        uint32_t u[kStatSlabs][8];
#pragma unroll
        for (int i = 0; i < kStatSlabs; ++i) {
            const int k0 = min(kl * 8 + i * 64 * kstep, K - 1);
            if (o.kcontig && o.vec4 && k0 + 8 <= K) {      // k0 is a multiple of 8 here
                const u32x4 *src = reinterpret_cast<const u32x4 *>(o.X + (size_t)row * o.ld + k0);
                const u32x4 a = src[0], b = src[1];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    u[i][j] = a[j];
                    u[i][4 + j] = b[j];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = min(k0 + j, K - 1);      // a repeated element does not change max / min
                    u[i][j] = o.kcontig ? o.X[(size_t)row * o.ld + k] : o.X[(size_t)k * o.ld + row];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kStatSlabs; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) look(u[i][j]);
    }
    if (o.kcontig) {
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {
            hi = max(hi, __shfl_xor(hi, off, 64));
            lo = min(lo, __shfl_xor(lo, off, 64));
        }
        if (kl != 0) return;
    } else {
        s_hi[kl][tid % 32] = hi;
        s_lo[kl][tid % 32] = lo;
        __syncthreads();
        if (kl != 0) return;
#pragma unroll
        for (int q = 1; q < 8; ++q) {
            hi = max(hi, s_hi[q][tid]);
            lo = min(lo, s_lo[q][tid]);
        }
    }
    if (row >= o.rows_pad) return;
    o.S[row] = window_scale(hi, lo, emin, m);
    if (row % kUnitRows == 0) o.rec_cnt[row / kUnitRows] = 0u;
}

__global__ __launch_bounds__(256) void window_stats_kernel(StatOperand a, StatOperand b, int Ka, int kstep_a, int Kb,
                                                           int kstep_b, int emin, int m)
{
    const bool second = blockIdx.x >= a.nblocks;
    window_stats_block(second ? b : a, second ? Kb : Ka, second ? kstep_b : kstep_a, emin, m,
                       (int)(blockIdx.x - (second ? a.nblocks : 0u)));
}

// The same for the operands of a prepare group (see prepare_scaled_group_kernel): run i starts at first[i].
struct StatGroup {
    unsigned first[kMaxPrepGroup];   // 0xFFFFFFFF beyond the last operand
    StatOperand o[kMaxPrepGroup];
    int K[kMaxPrepGroup], kstep[kMaxPrepGroup];
};

// clear (nclear words): the partial records of the group kernel that follows.  A completed group leaves them zero; clearing them
// here, in the same call, makes sure of it whatever an earlier call left (see hist_clear).
__global__ __launch_bounds__(256) void window_stats_group_kernel(StatGroup grp, int emin, int m, unsigned long long *clear, unsigned nclear)
{
    for (unsigned i = blockIdx.x * 256u + threadIdx.x; i < nclear; i += gridDim.x * 256u)
        __hip_atomic_store(&clear[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int at = run_of(grp.first, blockIdx.x);
    window_stats_block(grp.o[at], grp.K[at], grp.kstep[at], emin, m, (int)(blockIdx.x - grp.first[at]));
}

// ---- operand preparation ------------------------------------------------------------------------

// Launches what turns the described operands into prepared ones: the pre-rounding of a tensor that is
// gathered from, the row scales of exponent planes, and the prepare kernel.  sb == nullptr: one operand.
// pre_a / pre_b: room for the pre-rounded tensors (only for specs with pre_elems > 0).
template <int MODE, bool FTZ, int PS>
static int prepare_operands(const OperandSpec &sa, const OperandLayout &la, const OperandView &va, uint32_t *pre_a,
                            const OperandSpec *sb, const OperandLayout *lb, const OperandView *vb, uint32_t *pre_b, int K,
                            fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    const int kblocks = la.kblocks;
    const bool scaled = la.sch.scaled;
    auto operand = [&](const OperandSpec &sp, const OperandLayout &L, const OperandView &v, uint32_t *pre_buf) {
        PrepOperand o;
        o.X = reinterpret_cast<const uint32_t *>(sp.X);
        o.g = sp.g;
        if (sp.pre_elems > 0) {
            const int n = (int)sp.pre_elems;
            const int grid = (n + 1023) / 1024 < 4096 ? (n + 1023) / 1024 : 4096;
            hipLaunchKernelGGL((round_split_kernel<MODE, FTZ, PS>), dim3(grid), dim3(256), 0, stream, o.X, pre_buf, n, p);
            o.X = pre_buf;
            o.g.pre = 1;
            o.g.plane = n + 1;
            const bool simple = o.g.den_y == 1 && o.g.den_x == 1 && o.g.R * o.g.S <= 32;
            o.g.fast = simple && o.g.kind == kSrcPatchRows && !sp.kcontig ? 1
                       : simple && o.g.kind == kSrcPatchK && sp.kcontig && o.g.tap > 0 ? 2 : 0;
        }
        o.W = v.W;
        o.ld = sp.ld;
        o.rows = L.rows;
        o.kcontig = sp.kcontig;
        o.vec4 = (reinterpret_cast<uintptr_t>(sp.X) & 15) == 0 && sp.ld % 4 == 0;
        o.nblocks = o.g.fast == 2 ? (unsigned)((kblocks + 7) / 8) * L.units            // 32 taps x 256 positions each
                    : sp.kcontig ? (unsigned)((kblocks + 1) / 2) * L.units
                                 : (unsigned)kblocks * (L.units / (o.g.fast ? 2 * kFastRows : 2));
        o.pl = v.pl;
        return o;
    };
    const PrepOperand oa = operand(sa, la, va, pre_a);
    PrepOperand ob = oa;
    ob.nblocks = 0u;
    if (sb != nullptr) ob = operand(*sb, *lb, *vb, pre_b);
    FMT_HIP_CHECK(hipGetLastError());
    const unsigned prep_grid = (oa.nblocks + 7u) / 8u * 8u + (ob.nblocks + 7u) / 8u * 8u;
    if (scaled) {
        if constexpr (PS == 0 && MODE == kModeMagic) {
            auto stat = [&](const PrepOperand &o, const OperandLayout &L, bool present) {
                StatOperand t;
                t.X = o.X;
                t.ld = o.ld;
                t.rows = L.rows;
                t.rows_pad = L.units * kUnitRows;
                t.kcontig = o.kcontig;
                t.vec4 = o.vec4;
                t.S = o.pl.S;
                t.rec_cnt = o.pl.rec_cnt;
                t.nblocks = present ? (unsigned)L.units : 0u;
                return t;
            };
            const StatOperand ta = stat(oa, la, true), tb = stat(ob, sb ? *lb : la, sb != nullptr);
            // a sample of the row: the scale only has to be a good guess
            const int slabs = (K + 63) / 64;
            const int bias = (1 << (f.e - 1)) - 1;
            hipLaunchKernelGGL(window_stats_kernel, dim3(ta.nblocks + tb.nblocks), dim3(256), 0, stream, ta, tb, K,
                               (slabs + kStatSlabs - 1) / kStatSlabs, K, (slabs + kStatSlabs - 1) / kStatSlabs, 1 - bias, f.m);
            FMT_HIP_CHECK(hipGetLastError());
            hipLaunchKernelGGL((prepare_scaled_kernel<MODE, FTZ>), dim3(prep_grid), dim3(256), 0, stream, oa, ob, K, kblocks, K,
                               kblocks, p);
        } else {
            return FMT_ERR_FORMAT;               // planes exist for e == 6 formats only (rounding mode kModeMagic)
        }
    } else if (oa.g.fast == 2 || ob.g.fast == 2) {
        hipLaunchKernelGGL((prepare_kernel<MODE, FTZ, PS, true>), dim3(prep_grid), dim3(256), 0, stream, oa, ob, K, kblocks, p);
    } else {
        hipLaunchKernelGGL((prepare_kernel<MODE, FTZ, PS, false>), dim3(prep_grid), dim3(256), 0, stream, oa, ob, K, kblocks, p);
    }
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

static Scheme api_scheme(fmt_format_t f, int64_t K);

// Parts of k of a direct product (fmt_direct.hip), or 0 where the general route is the better one (or forced by a plan).
// FMT_GEMM_PLAN=direct (tests): wherever the kernel can; any other value: nowhere.  Both routes' times on the GPU (us), fitted to 900
// products of 8 x 8 to 2048 x 1200 with k of 8 to 3000 in all layouts, replayed from graphs (both fits within 6 to 10 %):
//   direct   2.7, and per block of 32 k that a wave takes one after the other, with n waves on a SIMD of the busiest compute unit,
//            0.62 + 0.38 n (one piece 0.22 + 0.16 n; 0.18 more with the flush); 4.4 per further round of workgroups (a SIMD holds two
//            waves); 1.3 per 10^6 results and 0.65 per 10^6 operand elements; up to 11 blocks (long chains come out slower)
//   general  two launches: 5.8, 0.23 (one piece 0.07) per block of k, 2.05 per 10^6 operand elements, 1.06 (0.69) per 10^6
//            results; three where the plan splits k: 6.7, 0.37 (0.25) per block of a part, 3.3 (1.9) and 0.9 (1.9)
//            per part and 10^6 results; a layer's output roundings are then a launch of their own, 4
// A launch less also saves the host 2.5 - 3 us (from Python 7.2, 9.7 and 12.2 us with one, two and three), so a direct product may
// take 1.2 us more than three launches: with that, the 900 take 5.90 ms from graphs (6.19 before operands
// whose rows lie along k came through LDS; 5.84 with the better route each time).  Measured (us in a graph, general / direct): 256 x 256 x
// 511 in 1/6/9 10.9 / 6.5; 256 x 1024 x 1024 14.4 / 9.5 - 10.0; 300 x 300 x 333 in 1/5/10 8 / 7.2; not taken: 559 x 489 x 1289 in
// 1/6/9 18.1 / 23.9, 973 x 608 x 1264 in 1/8/7 14.9 / 32.1.
// Of a layer with nsplit == 1 the general route ends in its product's kernel, statistics and codes included, which the direct one has to
// leave to a pass of 4 - 10 us: more than it saves (general / direct and pass, from Python: 192 x 101 x 192 in 1/5/10 with statistics
// 12.0 / 18.2, 752 x 552 x 192 with codes and statistics 12.7 / 18.0, 276 x 1210 x 194 in 1/8/7 with codes 10.7 / 12.0).  So such layers take
// the general route (in_product) -- where its sums are the direct one's.  1/6/8 and 1/6/9 have parts of their own, and where the general
// route does not cut k a layer's outputs depend neither on whether statistics are asked for nor on which of fmt_gemm and fmt_linear makes the sums: in one part
// (k <= 96) the sums are the same, 20 layers 18.0 -> 11.8 with statistics, 12.0 -> 10.4 with codes, 19.2 -> 12.7 with both; in several the product
// decides, and a pass follows (general / direct and pass, 165 x 156 x 252: 12.4 / 16.8 with statistics, 10.0 / 7.6 without).  Where there are two waves
// for a SIMD, and a wave takes more than two blocks, a product whose rows lie along k, as a layer's do, gains so little that the general
// route takes it for the layers' sake (40 products and layers of 110 x 1400 to 1400 x 1400, k 129 to 480, from Python, general / direct: products 11.4 / 10.9,
// in graphs 11.4 / 11.3, plain layers 12.4 / 12.1, with codes 13.1 / 14.8, with statistics 15.6 / 19.5, with both 16.3 / 20.5).
// Where these formats need a second round of workgroups and the general route cuts k, the direct one comes out slower than the times above say: 40
// shapes of 32 x 32 to 4000 x 4000, k 256 to 3000, in graphs, general / direct: products with rows along k 20.1 / 21.8, without 19.5 / 20.9, plain
// layers, whose rounding is a launch of its own in general, 26.5 / 25.0.  So the products leave it there.  The layers keep it, those with codes (25.5 / 27.0) and
// statistics (34.5 / 36.1) too: their sums are the plain ones'.
static int direct_parts(int M, int N, int K, const OperandSpec &sa, const OperandSpec &sb, const Plan &plan, fmt_format_t f, Scheme sch,
                        int mode, const LinearOut *lin, int cus)
{
    const char *env = getenv("FMT_GEMM_PLAN");
    if (env != nullptr && strcmp(env, "direct") != 0) return 0;
    // formats whose rounding has the short form of direct_convert
    if (!(mode == kModeMagic && sch.ps <= 2) && !(mode == kModeInteger && sch.ps == 1)) return 0;
    // offsets inside an operand in 32 bits
    auto fits = [](const OperandSpec &o, int rows) { return o.kcontig ? (int64_t)rows * o.ld < ((int64_t)1 << 32) : o.ld < ((int64_t)1 << 28); };
    if (!fits(sa, M) || !fits(sb, N)) return 0;
    const int kblocks = (K + kUnitK - 1) / kUnitK;
    const int64_t tiles = (((int64_t)M + 31) / 32) * (((int64_t)N + 31) / 32);
    int parts = plan.nsplit;
    const bool own_parts = planes_possible(f) && api_scheme(f, K).scaled;
    if (own_parts) {
        // the prepared calls of these formats take the planes, so no other call promises these sums and the parts are
        // free: enough for two waves per SIMD (2048), two blocks each at least
        parts = 1;
        while (parts < kDirectParts && tiles * parts < 2048 && kblocks / (parts * 2) >= 2) parts *= 2;
    }
    if (parts > kDirectParts) return 0;
    if (env != nullptr) return parts;
    const bool layer = lin != nullptr && lin->hist == nullptr && lin->codes == nullptr;     // rounded by the direct kernel
    const bool in_product = lin != nullptr && plan.nsplit == 1 && (lin->hist == nullptr || lin->p.exp_lo >= -126);
    if (in_product && !layer && (!own_parts || parts == 1)) return 0;
    const bool one = pieces_of(sch.ps) == 1;
    const int64_t per_wg = direct_blocks_per_workgroup(parts), wgs = (tiles + per_wg - 1) / per_wg;
    const double n = (double)((wgs + cus - 1) / cus) * (double)(parts * per_wg) / 4.0;
    const double rounds = std::max(0.0, std::ceil(n / 2.0) - 1.0);
    const double blocks = (double)((kblocks + parts - 1) / parts);
    if (blocks > 11.0) return 0;
    if (own_parts && plan.nsplit > 1 && n > 2.0 && lin == nullptr) return 0;
    if (own_parts && plan.nsplit == 1 && parts > 1 && sa.kcontig && sb.kcontig && blocks > 2.0 && tiles * parts >= 4 * (int64_t)cus) return 0;
    const double operands = ((double)M + N) * K * 1e-6, results = (double)M * N * 1e-6;
    const double each = (one ? 0.22 + 0.16 * n : 0.62 + 0.38 * n) + (f.denorm == 0 ? 0.18 : 0.0);
    const double direct = 2.7 + blocks * each + 4.4 * rounds + 1.3 * results + 0.65 * operands;
    const double kb_per = (double)((kblocks + plan.nsplit - 1) / plan.nsplit);
    const double general = plan.nsplit == 1
                               ? 5.8 + (one ? 0.07 : 0.23) * kb_per + 2.05 * operands + (one ? 0.69 : 1.06) * results
                               : 6.7 + (one ? 0.25 : 0.365) * kb_per + (one ? 1.9 : 3.3) * operands +
                                     (one ? 1.9 : 0.9) * plan.nsplit * results + 1.2 + (layer ? 4.0 : 0.0);
    return direct < general ? parts : 0;
}

// Room for the split-k partial sums of a plan.
static size_t part_bytes_of(const Plan &plan, int M, int N)
{
    return plan.nsplit > 1 ? ((size_t)plan.nsplit * M * N * sizeof(float) + 255) / 256 * 256 : 0;
}

static int product_dispatch(int ps, const OperandView &va, const OperandView &vb, int M, int N, int kblocks,
                            const OutSpec &out, const Plan &plan, float *part, hipStream_t stream)
{
    switch (ps) {
        case 0: return product_of_views<0>(va, vb, M, N, kblocks, out, plan, part, stream);
        case 1: return product_of_views<1>(va, vb, M, N, kblocks, out, plan, part, stream);
        case 2: return product_of_views<2>(va, vb, M, N, kblocks, out, plan, part, stream);
        default: return product_of_views<3>(va, vb, M, N, kblocks, out, plan, part, stream);
    }
}

// Prepare + product (+ reduction) of described operands in library scratch.
template <int MODE, bool FTZ, int PS>
static int run(int M, int N, int K, const OperandSpec &sa, const OperandSpec &sb, const OutSpec &out, fmt_format_t f,
               const QuantParams &p, hipStream_t stream, bool scaled)
{
    const Scheme sch{PS, scaled};
    OperandLayout la, lb;
    int rc = operand_layout(M, K, sch, f.m, &la);
    if (rc != FMT_OK) return rc;
    rc = operand_layout(N, K, sch, f.m, &lb);
    if (rc != FMT_OK) return rc;
    int cus = 0;
    rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    const Plan plan = make_plan(M, N, la.kblocks, cus, pieces_of(PS));
    auto up256 = [](size_t b) { return (b + 255) / 256 * 256; };
    const int words = (pieces_of(PS) + 1) / 2;
    const size_t pre_a = sa.pre_elems ? up256((size_t)(sa.pre_elems + 1) * words * sizeof(uint32_t)) : 0;
    const size_t pre_b = sb.pre_elems ? up256((size_t)(sb.pre_elems + 1) * words * sizeof(uint32_t)) : 0;
    const size_t part = part_bytes_of(plan, M, N);
    Scratch s;
    rc = get_scratch(stream, 0, la.bytes + lb.bytes + part + pre_a + pre_b, &s);
    if (rc != FMT_OK) return rc;
    // (the scratch of the general route is kept even where it is not used: what a call needs, and whether it can be
    // recorded into a graph, does not depend on the route)
    if (!scaled && sa.g.kind == kSrcMatrix && sb.g.kind == kSrcMatrix && out.img == 0) {
        const bool plain = out.lin != nullptr && out.lin->hist == nullptr && out.lin->codes == nullptr;   // a layer's fp32 outputs without statistics
        const int parts = direct_parts(M, N, K, sa, sb, plan, f, sch, p.mode, out.lin, cus);
        if (parts > 0) {
            const int rcd = launch_direct_product(M, N, K, MatrixOperand{sa.X, sa.ld, sa.kcontig}, MatrixOperand{sb.X, sb.ld, sb.kcontig},
                                                  out.C, out.ldc, parts, PS, FTZ, p, plain ? out.lin : nullptr, stream);
            if (rcd == FMT_OK && plain) *out.rounded = true;
            return rcd;
        }
    }
    char *ws = static_cast<char *>(s.gemm_ws);
    const OperandView va = view_of(ws, la), vb = view_of(ws + la.bytes, lb);
    float *partp = reinterpret_cast<float *>(ws + la.bytes + lb.bytes);
    uint32_t *pa = reinterpret_cast<uint32_t *>(ws + la.bytes + lb.bytes + part);
    uint32_t *pb = reinterpret_cast<uint32_t *>(ws + la.bytes + lb.bytes + part + pre_a);
    rc = prepare_operands<MODE, FTZ, PS>(sa, la, va, pa, &sb, &lb, &vb, pb, K, f, p, stream);
    if (rc != FMT_OK) return rc;
    return product_of_views<PS>(va, vb, M, N, la.kblocks, out, plan, partp, stream);
}

template <int MODE, bool FTZ>
static int run_p(Scheme sch, int M, int N, int K, const OperandSpec &sa, const OperandSpec &sb, const OutSpec &out,
                 fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    switch (sch.ps) {
        case 0: return run<MODE, FTZ, 0>(M, N, K, sa, sb, out, f, p, stream, sch.scaled);
        case 1: return run<MODE, FTZ, 1>(M, N, K, sa, sb, out, f, p, stream, false);
        case 2: return run<MODE, FTZ, 2>(M, N, K, sa, sb, out, f, p, stream, false);
        default: return run<MODE, FTZ, 3>(M, N, K, sa, sb, out, f, p, stream, false);
    }
}

// Product of two described operands (K > 0): picks the piece scheme and the rounding variant.
static int run_product(int M, int N, int K, const OperandSpec &sa, const OperandSpec &sb, const OutSpec &out,
                       fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    const bool ftz = f.denorm == 0;
    // 1/6/9 and 1/6/8: exponent planes (a quarter of the MFMA work of two bf16 pieces) for plain matrix
    // operands, when the product is large enough to pay for the launch that picks the row scales
    const int wmode = window_mode();
    const bool planes = sa.g.kind == kSrcMatrix && sb.g.kind == kSrcMatrix && out.img == 0 &&
                        K < (1 << 27) && (wmode == 1 || (wmode == 2 && 2.0 * M * N * K >= 1e9 && K >= 128));
    const Scheme sch = scheme_of(f, planes);
#define FMT_RUN(MD)                                                                     \
    (ftz ? run_p<MD, true>(sch, M, N, K, sa, sb, out, f, p, stream)                      \
         : run_p<MD, false>(sch, M, N, K, sa, sb, out, f, p, stream))
    if (p.mode == kModeMagic) return FMT_RUN(kModeMagic);
    if (p.mode == kModeInteger) return FMT_RUN(kModeInteger);
    return FMT_RUN(kModeMixed);
#undef FMT_RUN
}

// ---- prepared operands in caller-owned memory ---------------------------------------------------

// (the tail's element records hold k in 27 bits: longer sums take the bf16 pieces)
static Scheme api_scheme(fmt_format_t f, int64_t K) { return scheme_of(f, window_mode() != 0 && K < ((int64_t)1 << 27)); }

int prepared_operand_bytes(int64_t rows, int64_t K, fmt_format_t f, size_t *bytes, int *scheme)
{
    OperandLayout L;
    const Scheme sch = api_scheme(f, K);
    int rc = operand_layout(rows, K, sch, f.m, &L);
    if (rc != FMT_OK) return rc;
    *bytes = L.bytes;
    *scheme = sch.ps + (sch.scaled ? 16 : 0);
    return FMT_OK;
}

template <int MODE, bool FTZ>
static int prepare_one_p(Scheme sch, const OperandSpec &sp, const OperandLayout &L, const OperandView &v, int K,
                         fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    switch (sch.ps) {
        case 0: return prepare_operands<MODE, FTZ, 0>(sp, L, v, nullptr, nullptr, nullptr, nullptr, nullptr, K, f, p, stream);
        case 1: return prepare_operands<MODE, FTZ, 1>(sp, L, v, nullptr, nullptr, nullptr, nullptr, nullptr, K, f, p, stream);
        case 2: return prepare_operands<MODE, FTZ, 2>(sp, L, v, nullptr, nullptr, nullptr, nullptr, nullptr, K, f, p, stream);
        default: return prepare_operands<MODE, FTZ, 3>(sp, L, v, nullptr, nullptr, nullptr, nullptr, nullptr, K, f, p, stream);
    }
}

// X is `rows` x K after op(): trans == 0: X[r*ld + k], trans != 0: X[k*ld + r].  rows, K > 0.
int launch_prepare_operand(const float *X, int64_t ld, int trans, int64_t rows, int64_t K, fmt_format_t f,
                           const QuantParams &p, void *buf, hipStream_t stream)
{
    const Scheme sch = api_scheme(f, K);
    OperandLayout L;
    int rc = operand_layout(rows, K, sch, f.m, &L);
    if (rc != FMT_OK) return rc;
    const OperandView v = view_of(buf, L);
    const OperandSpec sp{X, ld, trans == 0, Gather{}, 0};
    const bool ftz = f.denorm == 0;
#define FMT_PREP(MD)                                                                \
    (ftz ? prepare_one_p<MD, true>(sch, sp, L, v, (int)K, f, p, stream)              \
         : prepare_one_p<MD, false>(sch, sp, L, v, (int)K, f, p, stream))
    if (p.mode == kModeMagic) return FMT_PREP(kModeMagic);
    if (p.mode == kModeInteger) return FMT_PREP(kModeInteger);
    return FMT_PREP(kModeMixed);
#undef FMT_PREP
}

// Both orientations of several matrices (buf0 = X as stored, buf1 = X transposed) with shared launches:
// matrices whose two operands take exponent planes are gathered, up to kMaxPrepGroup / 2 at a time, into one
// statistics launch and one prepare launch; the others are prepared operand by operand.  The operands equal
// those of two launch_prepare_operand calls (the same block functions on the same blocks; only the order of
// the records within a list may differ, which the product's tail sorts away).
// round != nullptr: the same launch also writes every matrix rounded to fp32 (round[i].Y) and counts its elements
// into round[i].hist, as fmt_quantize does (window from p.exp_lo); planes formats only (FMT_ERR_FORMAT otherwise).
static_assert(sizeof(PrepGroup) + sizeof(RoundGroup) + sizeof(QuantParams) <= 4096 && sizeof(StatGroup) + 24 <= 4096,
              "group tables travel in the kernel arguments");

int launch_prepare_pair_batch(int64_t count, const PrepPairItem *items, fmt_format_t f, const QuantParams &p, hipStream_t stream,
                              const RoundItem *round)
{
    StatGroup sg;
    PrepGroup pg;
    RoundGroup rg{};
    if (round != nullptr) {
        for (int64_t i = 0; i < count; ++i)
            if (!(api_scheme(f, items[i].cols).scaled && api_scheme(f, items[i].rows).scaled && p.mode == kModeMagic))
                return FMT_ERR_FORMAT;
        Scratch sc;
        const int rc = get_scratch(stream, kHistScratchBytes + (size_t)(kMaxPrepGroup / 2) * kSetWords * sizeof(unsigned long long), 0, &sc);
        if (rc != FMT_OK) return rc;
        rg.records = static_cast<unsigned long long *>(sc.hist_partials) + kHistScratchBytes / sizeof(unsigned long long);
        // steps per workgroup: as many as leave every compute unit four workgroups (measured on 12 tensors of 4 M to 16 M
        // elements: one step 267 us, four 242 us, eight 258 us; one tensor of 4 M elements: four 36 us)
        int cus = 0;
        const int rc2 = device_cu_count(&cus);
        if (rc2 != FMT_OK) return rc2;
        uint64_t all_tiles = 0;
        for (int64_t i = 0; i < count; ++i)
            all_tiles += (uint64_t)((items[i].rows + 31) / 32) * (uint64_t)((items[i].cols + 64 * kPairTiles - 1) / (64 * kPairTiles));
        rg.steps = kRoundSteps;
        while (rg.steps > 1 && all_tiles / (uint64_t)rg.steps < (uint64_t)cus * 4) rg.steps /= 2;
    }
    int n = 0;
    unsigned stat_ids = 0, prep_ids = 0;
    const int bias = (1 << (f.e - 1)) - 1;
    auto flush = [&]() -> int {
        if (n == 0) return FMT_OK;
        for (int i = n; i < kMaxPrepGroup; ++i) {
            sg.first[i] = 0xFFFFFFFFu;
            sg.o[i] = StatOperand{};
            sg.K[i] = sg.kstep[i] = 0;
            pg.o[i] = PrepPlain{};
        }
        for (int i = n / 2; i < kMaxPrepGroup / 2; ++i) {
            pg.first[i] = 0xFFFFFFFFu;
            pg.tiles[i] = 0u;
        }
        hipLaunchKernelGGL(window_stats_group_kernel, dim3(stat_ids), dim3(256), 0, stream, sg, 1 - bias, f.m, rg.records,
                           round != nullptr ? (unsigned)(n / 2 * kSetWords) : 0u);
        FMT_HIP_CHECK(hipGetLastError());
#define FMT_PAIR_LAUNCH(FTZV, ROUNDV, DEEPV)                                                                           \
    hipLaunchKernelGGL((prepare_scaled_group_kernel<kModeMagic, FTZV, ROUNDV, DEEPV>), dim3(prep_ids), dim3(256), 0, stream, pg, \
                       rg, p)
        const bool ftz = f.denorm == 0, deep = p.exp_lo < -126;
        if (round == nullptr) {
            if (ftz) FMT_PAIR_LAUNCH(true, false, false); else FMT_PAIR_LAUNCH(false, false, false);
        } else if (deep) {
            if (ftz) FMT_PAIR_LAUNCH(true, true, true); else FMT_PAIR_LAUNCH(false, true, true);
        } else {
            if (ftz) FMT_PAIR_LAUNCH(true, true, false); else FMT_PAIR_LAUNCH(false, true, false);
        }
#undef FMT_PAIR_LAUNCH
        FMT_HIP_CHECK(hipGetLastError());
        n = 0;
        stat_ids = prep_ids = 0;
        return FMT_OK;
    };
    auto add = [&](const PrepPairItem &it, bool kcontig, const OperandLayout &L, const OperandView &v, int K) {
        PrepPlain &o = pg.o[n];
        o.X = reinterpret_cast<const uint32_t *>(it.X);
        o.W = v.W;
        o.ld = it.ld;
        o.rows = L.rows;
        o.kcontig = kcontig;
        o.vec4 = (reinterpret_cast<uintptr_t>(it.X) & 15) == 0 && it.ld % 4 == 0;
        o.units = L.units;
        o.K = K;
        o.kblocks = L.kblocks;
        o.pl = v.pl;
        StatOperand &t = sg.o[n];
        t.X = o.X;
        t.ld = o.ld;
        t.rows = L.rows;
        t.rows_pad = L.units * kUnitRows;
        t.kcontig = kcontig;
        t.vec4 = o.vec4;
        t.S = v.pl.S;
        t.rec_cnt = v.pl.rec_cnt;
        t.nblocks = (unsigned)L.units;
        sg.K[n] = K;
        sg.kstep[n] = ((K + 63) / 64 + kStatSlabs - 1) / kStatSlabs;
        sg.first[n] = stat_ids;
        stat_ids += t.nblocks;
        ++n;
    };
    for (int64_t i = 0; i < count; ++i) {
        const PrepPairItem &it = items[i];
        const Scheme s0 = api_scheme(f, it.cols), s1 = api_scheme(f, it.rows);
        if (!(s0.scaled && s1.scaled && p.mode == kModeMagic)) {
            int rc = launch_prepare_operand(it.X, it.ld, 0, it.rows, it.cols, f, p, it.buf0, stream);
            if (rc == FMT_OK) rc = launch_prepare_operand(it.X, it.ld, 1, it.cols, it.rows, f, p, it.buf1, stream);
            if (rc != FMT_OK) return rc;
            continue;
        }
        OperandLayout L0, L1;
        int rc = operand_layout(it.rows, it.cols, s0, f.m, &L0);
        if (rc != FMT_OK) return rc;
        rc = operand_layout(it.cols, it.rows, s1, f.m, &L1);
        if (rc != FMT_OK) return rc;
        if (n + 2 > kMaxPrepGroup || prep_ids > 0x40000000u) {
            rc = flush();
            if (rc != FMT_OK) return rc;
        }
        // workgroups: kPairTiles tiles of 32 rows x 64 columns of X each; L0's units by pairs of L1's units cover X (and
        // either operand's k)
        const unsigned tiles = (unsigned)L0.units * (unsigned)(L1.units / (2 * kPairTiles));
        pg.first[n / 2] = prep_ids;
        pg.tiles[n / 2] = tiles;
        if (round != nullptr) {
            const int slot = n / 2;
            rg.Y[slot] = reinterpret_cast<uint32_t *>(round[i].Y);
            rg.ldy[slot] = round[i].ldy;
            rg.hist[slot] = reinterpret_cast<unsigned long long *>(round[i].hist);
        }
        const unsigned steps = round != nullptr ? (unsigned)rg.steps : 1u;
        prep_ids += ((tiles + steps - 1u) / steps + 7u) / 8u * 8u;
        add(it, true, L0, view_of(it.buf0, L0), (int)it.cols);
        add(it, false, L1, view_of(it.buf1, L1), (int)it.rows);
    }
    return flush();
}

// Both orientations of one matrix X (rows x cols, X[r*ld + c]) as prepared operands: buf0 = X as stored
// (rows, k = cols), buf1 = X transposed (cols, k = rows).  Exponent planes: one statistics launch and one
// prepare launch that reads X once serve both (launch_prepare_pair_batch); other schemes: two prepare calls.
int launch_prepare_pair(const float *X, int64_t ld, int64_t rows, int64_t cols, fmt_format_t f, const QuantParams &p, void *buf0,
                        void *buf1, hipStream_t stream)
{
    const Scheme s0 = api_scheme(f, cols), s1 = api_scheme(f, rows);
    if (s0.scaled && s1.scaled && p.mode == kModeMagic) {
        const PrepPairItem it{X, ld, rows, cols, buf0, buf1};
        return launch_prepare_pair_batch(1, &it, f, p, stream, nullptr);
    }
    const int rc = launch_prepare_operand(X, ld, 0, rows, cols, f, p, buf0, stream);
    return rc != FMT_OK ? rc : launch_prepare_operand(X, ld, 1, cols, rows, f, p, buf1, stream);
}

// C = A B^T on two prepared operands (A: M rows, B: N rows, both with the same K and scheme).
int launch_gemm_prepared(const void *A, const void *B, int64_t M64, int64_t N64, int64_t K64, int scheme, fmt_format_t f,
                         float *C, int64_t ldc, hipStream_t stream, const LinearOut *lin, bool *rounded)
{
    const int M = (int)M64, N = (int)N64;
    const Scheme sch{scheme & 15, (scheme & 16) != 0};
    OperandLayout la, lb;
    int rc = operand_layout(M64, K64, sch, f.m, &la);
    if (rc != FMT_OK) return rc;
    rc = operand_layout(N64, K64, sch, f.m, &lb);
    if (rc != FMT_OK) return rc;
    int cus = 0;
    rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    const Plan plan = make_plan(M, N, la.kblocks, cus, pieces_of(sch.ps));
    float *part = nullptr;
    if (plan.nsplit > 1) {
        Scratch s;
        rc = get_scratch(stream, 0, part_bytes_of(plan, M, N), &s);
        if (rc != FMT_OK) return rc;
        part = static_cast<float *>(s.gemm_ws);
    }
    const OperandView va = view_of(const_cast<void *>(A), la), vb = view_of(const_cast<void *>(B), lb);
    return product_dispatch(sch.ps, va, vb, M, N, la.kblocks, OutSpec{C, ldc, 0, lin, rounded}, plan, part, stream);
}

// Workgroup tile of a shared launch: 64 t x 64 t with t = 2 or 4.  The 256 x 256 tile runs one workgroup per
// compute unit, the 128 x 128 tile two; per unit of k both keep the matrix cores about equally busy when every
// slot has work, so what decides is how the tiles fill the slots.  A tile of kb blocks of 32 k takes about
// 9.5 + 0.89 kb us (large) or 9.8 + 0.47 kb us (small, two to a compute unit) on one fp16 piece -- fitted to
// per-workgroup timestamps on MI355X -- and P x P times the k term on P bf16 pieces.  Workgroups start in
// id order, longest tiles first, so the launch takes about as long as the larger of: all tile time spread
// over all slots; for each product, the rounds that the tiles up to and including its own need, times its
// tile time.  The shape with the smaller estimate is taken.
struct GroupEntry {
    int item;            // index into the batch
    int nparts;          // k parts (1: the product writes its result itself)
    int kb_per_part;     // k blocks per part
    size_t part_off;     // bytes from the start of the scratch to this product's slabs
};

// time estimate (us) of a shared launch of entries [g0, g0 + n) with workgroup tiles of 64 t x 64 t
static double group_estimate(const BatchItem *items, const std::vector<GroupEntry> &e, size_t g0, int n, int cus, int pieces, int t)
{
    const double fixed = t == 4 ? 9.5 : 9.8, per_kb = (t == 4 ? 0.89 : 0.47) * pieces * pieces;
    const double slots = (double)cus * (t == 4 ? 1 : 2);
    double work = 0.0, tiles = 0.0, rounds_bound = 0.0;
    for (int j = 0; j < n; ++j) {                            // longest parts first
        const BatchItem &it = items[e[g0 + j].item];
        const double tile_time = fixed + per_kb * e[g0 + j].kb_per_part;
        const double nt = (double)((it.M + 64 * t - 1) / (64 * t)) * (double)((it.N + 64 * t - 1) / (64 * t)) * e[g0 + j].nparts;
        tiles += nt;
        work += nt * tile_time;
        rounds_bound = std::max(rounds_bound, std::ceil(tiles / slots) * tile_time);
    }
    return std::max(work / slots, rounds_bound);
}

static int group_tile(const BatchItem *items, const std::vector<GroupEntry> &e, size_t g0, int n, int cus, int pieces)
{
    if (const char *env = getenv("FMT_GEMM_GROUP_TILE")) {      // tuning override: "2" or "4"
        const int t = atoi(env);
        if (t == 2 || (t == 4 && lds_bytes(4, 4, pieces, pipe_ks(pieces), 2) <= 160 * 1024)) return t;
    }
    if (lds_bytes(4, 4, pieces, pipe_ks(pieces), 2) > 160 * 1024) return 2;
    return group_estimate(items, e, g0, n, cus, pieces, 4) < group_estimate(items, e, g0, n, cus, pieces, 2) ? 4 : 2;
}

// Several products on prepared operands (all of one format and scheme).  A product joins a shared launch when
// it needs no split over k: its own plan has none, or one of its tiles is no longer than the work the whole
// batch leaves to each compute unit (then the other products fill the machine while its few long tiles run).
// A product that does need its k in parts (few tiles, long k) joins with its parts -- each part a run of tiles
// of its own that writes a slab of partial sums, summed by reduce_kernel after the launch -- when a part's
// tile takes no longer than the launch is estimated to take without it.  Shared launches hold up to kMaxGroup
// products, longest parts first (their tiles take longest and workgroups start in id order); what is left
// runs one by one as launch_gemm_prepared runs it.
int launch_gemm_prepared_batch(int count, const BatchItem *items, int scheme, fmt_format_t f, hipStream_t stream)
{
    const Scheme sch{scheme & 15, (scheme & 16) != 0};
    const int pieces = pieces_of(sch.ps);
    int cus = 0;
    int rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    std::vector<GroupEntry> grouped;
    std::vector<int> alone, parted;
    std::vector<Plan> plans((size_t)count);
    double load = 0.0;                                   // 256 x 256 x 32 blocks of multiplications per compute unit
    for (int i = 0; i < count; ++i)
        load += (double)((items[i].M + 255) / 256) * (double)((items[i].N + 255) / 256) * (double)((items[i].K + kUnitK - 1) / kUnitK);
    load /= cus;
    for (int i = 0; i < count; ++i) {
        const int kblocks = (int)((items[i].K + kUnitK - 1) / kUnitK);
        plans[(size_t)i] = make_plan((int)items[i].M, (int)items[i].N, kblocks, cus, pieces);
        if (plans[(size_t)i].nsplit == 1 || kblocks <= load) grouped.push_back(GroupEntry{i, 1, kblocks, 0});
        else parted.push_back(i);
    }
    size_t part_bytes = 0;
    if (!grouped.empty() && !parted.empty()) {
        const int n0 = (int)std::min<size_t>(kMaxGroup, grouped.size());
        const int t0 = group_tile(items, grouped, 0, n0, cus, pieces);
        const double base = group_estimate(items, grouped, 0, n0, cus, pieces, t0);
        const double fixed = t0 == 4 ? 9.5 : 9.8, per_kb = (t0 == 4 ? 0.89 : 0.47) * pieces * pieces;
        for (int i : parted) {
            const int kblocks = (int)((items[i].K + kUnitK - 1) / kUnitK);
            const int ns = plans[(size_t)i].nsplit, kb_per = (kblocks + ns - 1) / ns;
            if (fixed + per_kb * kb_per <= base) {
                grouped.push_back(GroupEntry{i, ns, kb_per, part_bytes});
                part_bytes += ((size_t)ns * items[i].M * items[i].N * sizeof(float) + 255) / 256 * 256;
            } else {
                alone.push_back(i);
            }
        }
    } else {
        alone = parted;
    }
    if (grouped.size() == 1 && grouped[0].nparts == 1) {
        alone.push_back(grouped[0].item);
        grouped.clear();
    }
    // the scratch for every slab of partial sums of the call, before anything is launched (growing it waits for the device)
    size_t need = part_bytes;
    for (int i : alone) need = std::max(need, part_bytes_of(plans[(size_t)i], (int)items[i].M, (int)items[i].N));
    char *scratch = nullptr;
    if (need > 0) {
        Scratch sc;
        rc = get_scratch(stream, 0, need, &sc);
        if (rc != FMT_OK) return rc;
        scratch = static_cast<char *>(sc.gemm_ws);
    }
    std::stable_sort(grouped.begin(), grouped.end(),
                     [&](const GroupEntry &a, const GroupEntry &b) { return a.kb_per_part > b.kb_per_part; });

    for (size_t g0 = 0; g0 < grouped.size(); g0 += kMaxGroup) {
        const int n = (int)std::min<size_t>(kMaxGroup, grouped.size() - g0);
        const int gt = group_tile(items, grouped, g0, n, cus, pieces);
        Group grp{};
        TailGroup tg{};
        grp.count = tg.count = n;
        for (int j = 0; j < kMaxGroup; ++j) grp.first[j] = tg.first[j] = 0xFFFFFFFFu;
        uint64_t ids = 0, blocks = 0, blocks256 = 0;
        for (int j = 0; j < n; ++j) {
            const BatchItem &it = items[grouped[g0 + j].item];
            blocks256 += (uint64_t)((it.M + kUnitRows - 1) / kUnitRows) * (uint64_t)((it.N + 255) / 256);
        }
        tg.tail_cols = tail_cols_for(blocks256, cus);
        for (int j = 0; j < n; ++j) {
            const GroupEntry &ge = grouped[g0 + j];
            const BatchItem &it = items[ge.item];
            OperandLayout la, lb;
            rc = operand_layout(it.M, it.K, sch, f.m, &la);
            if (rc != FMT_OK) return rc;
            rc = operand_layout(it.N, it.K, sch, f.m, &lb);
            if (rc != FMT_OK) return rc;
            const OperandView va = view_of(const_cast<void *>(it.A), la), vb = view_of(const_cast<void *>(it.B), lb);
            const int M = (int)it.M, N = (int)it.N;
            GroupItem &p = grp.p[j];
            p.Aw = va.W; p.Bw = vb.W;
            p.C = ge.nparts > 1 ? reinterpret_cast<float *>(scratch + ge.part_off) : it.C;
            p.ldc = ge.nparts > 1 ? (int64_t)N : it.ldc;
            p.M = M; p.N = N; p.kblocks = la.kblocks; p.kb_per_part = ge.kb_per_part;
            p.tiles_m = (M + 64 * gt - 1) / (64 * gt); p.tiles_n = (N + 64 * gt - 1) / (64 * gt);
            p.first = grp.first[j] = (unsigned)ids;
            p.pa = va.pl; p.pb = vb.pl;
            ids += ((uint64_t)p.tiles_m * p.tiles_n + 7) / 8 * 8 * (uint64_t)ge.nparts;
            TailGroupItem &t = tg.p[j];
            t.Aw = va.W; t.Bw = vb.W; t.C = it.C; t.ldc = it.ldc;
            t.M = M; t.N = N; t.kblocks = la.kblocks; t.col_chunks = (N + tg.tail_cols - 1) / tg.tail_cols;
            t.first = tg.first[j] = (unsigned)blocks;
            t.pa = va.pl; t.pb = vb.pl;
            blocks += (uint64_t)((M + kUnitRows - 1) / kUnitRows) * t.col_chunks;
            if (ids >= ((uint64_t)1 << 31) || blocks >= ((uint64_t)1 << 31)) return FMT_ERR_SHAPE;
        }
        switch (sch.ps) {
            case 0: rc = sch.scaled ? launch_group<0, true>(grp, (unsigned)ids, gt, stream) : launch_group<0, false>(grp, (unsigned)ids, gt, stream); break;
            case 1: rc = launch_group<1, false>(grp, (unsigned)ids, gt, stream); break;
            case 2: rc = launch_group<2, false>(grp, (unsigned)ids, gt, stream); break;
            default: rc = launch_group<3, false>(grp, (unsigned)ids, gt, stream); break;
        }
        if (rc != FMT_OK) return rc;
        for (int j = 0; j < n; ++j) {                        // the sums of the parts, in part order
            const GroupEntry &ge = grouped[g0 + j];
            if (ge.nparts == 1) continue;
            const BatchItem &it = items[ge.item];
            const int rcr = launch_reduce(reinterpret_cast<const float *>(scratch + ge.part_off), ge.nparts, it.C, (int)it.M, (int)it.N,
                                          it.ldc, 0, stream);
            if (rcr != FMT_OK) return rcr;
        }
        if (sch.scaled) {
            hipLaunchKernelGGL(planes_tail_group_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, tg);
            FMT_HIP_CHECK(hipGetLastError());
        }
    }
    for (int i : alone) {
        rc = launch_gemm_prepared(items[i].A, items[i].B, items[i].M, items[i].N, items[i].K, scheme, f, items[i].C, items[i].ldc,
                                  stream);
        if (rc != FMT_OK) return rc;
    }
    return FMT_OK;
}

static int zero_fill(float *C, int64_t rows, int64_t cols, int64_t ldc, hipStream_t stream)
{
    if (rows == 0 || cols == 0) return FMT_OK;
    const int64_t col_blocks = (cols + 255) / 256;
    if (col_blocks * rows >= ((int64_t)1 << 31)) return FMT_ERR_SHAPE;
    hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)(col_blocks * rows)), dim3(256), 0, stream, C, (int)rows, (int)cols,
                       ldc, (int)col_blocks);
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

int launch_gemm(int transA, int transB, int64_t M64, int64_t N64, int64_t K64, const float *A, int64_t lda,
                const float *B, int64_t ldb, float *C, int64_t ldc, fmt_format_t f, const QuantParams &p,
                hipStream_t stream, const LinearOut *lin, bool *rounded)
{
    const int M = (int)M64, N = (int)N64, K = (int)K64;
    if (K == 0) return zero_fill(C, M, N, ldc, stream);
    // op(A) is M x K: k-contiguous unless transposed.  op(B) is K x N, consumed as N rows of K:
    // k-contiguous when B is stored transposed (N x K).
    const OperandSpec sa{A, lda, !transA, Gather{}, 0};
    const OperandSpec sb{B, ldb, transB != 0, Gather{}, 0};
    return run_product(M, N, K, sa, sb, OutSpec{C, ldc, 0, lin, rounded}, f, p, stream);
}

// Forward and dgrad with the patches gathered inside the product kernel: the tensor behind the patches is
// rounded once into pixel-major 16-bit pieces (2P bytes per tensor element), the filter into an ordinary
// prepared operand whose k runs (tap, channel), and no patch-sized operand exists anywhere.
template <int MODE, bool FTZ, int PS>
static int run_implicit(int M, int N, int K, const OperandSpec &sa, const float *tensor, int64_t tensor_elems, int HW,
                        Implicit im, const OutSpec &out, fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    constexpr int P = pieces_of(PS);
    const Scheme sch{PS, false};
    OperandLayout la;
    int rc = operand_layout(M, K, sch, f.m, &la);
    if (rc != FMT_OK) return rc;
    int cus = 0;
    rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    const Plan plan = make_plan(M, N, la.kblocks, cus, P);
    auto up256 = [](size_t b) { return (b + 255) / 256 * 256; };
    const int C = im.c8 * 8;
    const int npix = (int)(tensor_elems / C);
    const size_t piece_vec = (size_t)npix * im.c8;
    const size_t nhwc = up256((P * piece_vec + 1) * sizeof(u32x4));
    const size_t part = part_bytes_of(plan, M, N);
    Scratch s;
    rc = get_scratch(stream, 0, la.bytes + nhwc + part, &s);
    if (rc != FMT_OK) return rc;
    char *ws = static_cast<char *>(s.gemm_ws);
    const OperandView va = view_of(ws, la);
    u32x4 *T = reinterpret_cast<u32x4 *>(ws + la.bytes);
    float *partp = reinterpret_cast<float *>(ws + la.bytes + nhwc);
    PrepOperand o;
    o.X = reinterpret_cast<const uint32_t *>(sa.X);
    o.W = va.W;
    o.ld = sa.ld;
    o.rows = la.rows;
    o.kcontig = sa.kcontig;
    o.vec4 = 0;
    o.nblocks = (unsigned)((la.kblocks + 1) / 2) * la.units;
    o.g = sa.g;
    o.pl = va.pl;
    const unsigned split_first = (o.nblocks + 7u) / 8u * 8u, nx = (unsigned)((npix + 63) / 64);
    hipLaunchKernelGGL((prepare_implicit_kernel<MODE, FTZ, PS>), dim3(split_first + nx * (unsigned)(C / 32)), dim3(256), 0, stream, o, K,
                       la.kblocks, split_first, nx, reinterpret_cast<const uint32_t *>(tensor), T, C, HW, npix, p);
    FMT_HIP_CHECK(hipGetLastError());
    im.T = T;
    im.piece_vec = (int)piece_vec;
    im.zero = (int)(P * piece_vec);
    return product_gathered<PS>(va, im, M, N, la.kblocks, out, plan, partp, stream);
}

constexpr int kWindowTile = 4;           // the products of planes: 128 x 128 at most (product_window)

// Convolutions in 1/6/8 and 1/6/9 on exponent planes with one scale per tensor: one fp16 MFMA product per multiply instead of the four of
// two bf16 pieces (forward, dgrad and wgrad, 256 -> 256 channels of 14 x 14, 3 x 3 taps, batch 64, us: 80 -> 45, 78 -> 60, 102 -> 76).
// Below `least` products the scales' samples and the tail cost more than they save.  us, bf16 pieces / planes:
//   forward   0.25 - 0.5 x 10^8 products 9.5 / 10.3, 11.2 / 14.5; 2 x 10^8 22.5 / 20, 12.2 / 11.8, 18.4 / 16.5; 5 x 10^8 21.5 / 16.3
//   dgrad     gathers gradients, of which a few lie outside plane 0 (log2|x| ~ N(-20, 5^2), 1e-5): 2 x 10^8 16.7 / 20.4, 17.2 / 19.9;
//             5 x 10^8 18.4 / 20.2, 15.8 / 18.2, 20.7 / 21; 9.6 x 10^8 22.2 / 24.3, 26 / 24.3; 1.1 x 10^9 38 / 35, 22.6 / 21.7; 2.2 x 10^9 37 / 33
//   wgrad     whose operands are prepared as patches: 1.2 x 10^8 34 / 36, 3.5 x 10^8 23.8 / 23.7, 9.6 x 10^8 54 / 49, 1.5 x 10^9 44 / 40
constexpr double kLeastForward = 1.5e8, kLeastDgrad = 1e9, kLeastWgrad = 7e8;
static bool conv_planes(fmt_format_t f, const QuantParams &p, double mults, double least)
{
    const int wmode = window_mode();
    return planes_possible(f) && p.mode == kModeMagic && (wmode == 1 || (wmode == 2 && mults >= least));
}

// Whether the tensors' samples may send a call to the pieces (window_pair): not where planes are asked for (FMT_GEMM_WINDOW=1).
static int window_adapts()
{
    const char *env = getenv("FMT_GEMM_WINDOW");
    return env != nullptr && env[0] == '1' ? 0 : 1;
}

static WindowTensor window_tensor(const float *x, int64_t n, fmt_format_t f)
{
    return WindowTensor{reinterpret_cast<const uint32_t *>(x), (uint32_t)n, 2 - (1 << (f.e - 1)), f.m};
}

// run_implicit for these.  The tensor's planes above and below are held whole and written where they are not empty; where there is no
// scratch for them, 1 comes back and nothing has been launched: two bf16 pieces take a third less.
static int run_implicit_window(int M, int N, int K, const OperandSpec &sa, int64_t filter_elems, const float *tensor, int64_t tensor_elems, int HW,
                               Implicit im, const OutSpec &out, fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    OperandLayout la;
    int rc = operand_layout(M, K, Scheme{0, true}, f.m, &la);
    if (rc != FMT_OK) return rc;
    int cus = 0;
    rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    const Plan plan = make_plan(M, N, la.kblocks, cus, 1, kWindowTile);
    auto up256 = [](size_t b) { return (b + 255) / 256 * 256; };
    const int C = im.c8 * 8;
    const int npix = (int)(tensor_elems / C);
    const unsigned nx = (unsigned)((npix + 63) / 64);
    const size_t piece_vec = (size_t)npix * im.c8;
    const size_t nhwc = up256((3 * piece_vec + 1) * sizeof(u32x4)), masks = up256((size_t)nx * (C / 32) * 2 * sizeof(uint64_t));
    const size_t part = part_bytes_of(plan, M, N);
    Scratch s;
    const size_t need = la.bytes + nhwc + masks + 256 + part;
    if (!scratch_has_room(stream, need) || get_scratch(stream, 0, need, &s) != FMT_OK) return 1;
    char *ws = static_cast<char *>(s.gemm_ws);
    const OperandView va = view_of(ws, la);
    OperandView vb{reinterpret_cast<u32x4 *>(ws + la.bytes), Planes{nullptr, nullptr, piece_vec, la.w, nullptr, nullptr}};
    vb.pl.mask = reinterpret_cast<uint8_t *>(ws + la.bytes + nhwc);
    vb.pl.S = reinterpret_cast<int *>(ws + la.bytes + nhwc + masks);
    float *partp = reinterpret_cast<float *>(ws + la.bytes + nhwc + masks + 256);
    PrepOperand o{};
    o.X = reinterpret_cast<const uint32_t *>(sa.X);
    o.W = va.W;
    o.rows = la.rows;
    o.kcontig = 1;
    o.nblocks = (unsigned)((la.kblocks + 1) / 2) * la.units;
    o.g = sa.g;
    o.pl = va.pl;
    const unsigned split_first = (o.nblocks + 7u) / 8u * 8u;
    const WindowTensor ta = window_tensor(sa.X, filter_elems, f), tb = window_tensor(tensor, tensor_elems, f);
    auto kern = f.denorm == 0 ? prepare_implicit_window_kernel<kModeMagic, true> : prepare_implicit_window_kernel<kModeMagic, false>;
    hipLaunchKernelGGL(kern, dim3(split_first + nx * (unsigned)(C / 32)), dim3(256), 0, stream, o, ta, K, la.kblocks, split_first, nx, tb,
                       window_adapts(), vb.W, vb.pl, C, HW, npix, p);
    FMT_HIP_CHECK(hipGetLastError());
    im.T = vb.W;
    im.piece_vec = (int)piece_vec;
    im.zero = (int)(3 * piece_vec);
    return product_window<true>(va, vb, im, M, N, la.kblocks, out, plan, partp, stream);
}

// The weight gradient on these planes: dY as the matrix [K][n*P*Q], the patches of X through gather_taps (at most 32 taps).  1: no scratch.
static int run_wgrad_window(int M, int N, int K, const OperandSpec &sa, int64_t grad_elems, const OperandSpec &sb, const OutSpec &out,
                            fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    OperandLayout la, lb;
    int rc = operand_layout(M, K, Scheme{0, true}, f.m, &la);
    if (rc != FMT_OK) return rc;
    rc = operand_layout(N, K, Scheme{0, true}, f.m, &lb);
    if (rc != FMT_OK) return rc;
    int cus = 0;
    rc = device_cu_count(&cus);
    if (rc != FMT_OK) return rc;
    const Plan plan = make_plan(M, N, la.kblocks, cus, 1, kWindowTile);
    const size_t part = part_bytes_of(plan, M, N);
    const int n = (int)sb.pre_elems;
    Scratch s;
    const size_t need = la.bytes + lb.bytes + part + ((size_t)n + 1) * sizeof(uint32_t);
    if (!scratch_has_room(stream, need) || get_scratch(stream, 0, need, &s) != FMT_OK) return 1;
    char *ws = static_cast<char *>(s.gemm_ws);
    const OperandView va = view_of(ws, la), vb = view_of(ws + la.bytes, lb);
    float *partp = reinterpret_cast<float *>(ws + la.bytes + lb.bytes);
    uint32_t *words = reinterpret_cast<uint32_t *>(ws + la.bytes + lb.bytes + part);
    const bool ftz = f.denorm == 0;
    constexpr int kPer = 256 * kRoundEach;
    const int grid = n / kPer < 8 * cus ? (n + kPer - 1) / kPer : 8 * cus;
    hipLaunchKernelGGL((ftz ? round_window_kernel<kModeMagic, true> : round_window_kernel<kModeMagic, false>), dim3(grid), dim3(256), 0, stream,
                       window_tensor(sb.X, n, f), window_tensor(sa.X, grad_elems, f), window_adapts(), words, lb.w, vb.pl.S, va.pl.S, p);
    FMT_HIP_CHECK(hipGetLastError());
    PrepOperand a{}, b{};
    a.X = reinterpret_cast<const uint32_t *>(sa.X);
    a.W = va.W;
    a.rows = la.rows;
    a.kcontig = 1;
    a.nblocks = (unsigned)((la.kblocks + 1) / 2) * la.units;
    a.g = sa.g;
    a.pl = va.pl;
    b.X = words;
    b.W = vb.W;
    b.rows = lb.rows;
    b.kcontig = 1;
    b.nblocks = (unsigned)((lb.kblocks + 7) / 8) * lb.units;
    b.g = sb.g;
    b.g.pre = 1;
    b.g.plane = n + 1;
    b.g.fast = 2;
    b.pl = vb.pl;
    hipLaunchKernelGGL((ftz ? prepare_taps_window_kernel<kModeMagic, true> : prepare_taps_window_kernel<kModeMagic, false>),
                       dim3((a.nblocks + 7u) / 8u * 8u + (b.nblocks + 7u) / 8u * 8u), dim3(256), 0, stream, a, b, K, la.kblocks, p);
    FMT_HIP_CHECK(hipGetLastError());
    return product_window<false>(va, vb, Implicit{}, M, N, la.kblocks, out, plan, partp, stream);
}

// In-kernel gather for forward (which == 0) and dgrad (which == 1): returns FMT_OK after launching, or 1 when
// the geometry is not covered (channels of the gathered tensor not a multiple of 32, more than 32 taps, dgrad
// with a stride, index ranges), in which case the caller takes the route through a gathered operand.
static int conv_implicit(int which, const fmt_conv2d_t &g, int64_t P, int64_t Q, const float *tensor, const float *filt,
                         float *out, fmt_format_t f, const QuantParams &p, hipStream_t stream)
{
    if (const char *env = getenv("FMT_CONV_IMPLICIT"))
        if (env[0] == '0') return 1;
    const int tc = which == 0 ? g.c : g.k;                       // channels of the gathered tensor
    const int64_t th = which == 0 ? g.h : P, tw = which == 0 ? g.w : Q;
    const int64_t elems = (int64_t)g.n * tc * th * tw;
    if (tc % 32 != 0 || g.r * g.s > 32 || elems >= ((int64_t)1 << 31)) return 1;
    if (which == 1 && (g.stride_h != 1 || g.stride_w != 1)) return 1;
    const Scheme sch = scheme_of(f, false);
    if ((elems / 8) * pieces_of(sch.ps) + (int64_t)(g.r * tw + g.s) * (tc / 8) >= ((int64_t)1 << 31)) return 1;
    const int rs = g.r * g.s;
    const int64_t M = which == 0 ? g.k : g.c, K = (int64_t)tc * rs;
    const int64_t gy = which == 0 ? P : g.h, gx = which == 0 ? Q : g.w;
    const int64_t N = (int64_t)g.n * gy * gx;
    Implicit im{};
    im.c8 = tc / 8;
    im.th = (int)th; im.tw = (int)tw; im.gy = (int)gy; im.gx = (int)gx;
    im.mul_y = which == 0 ? g.stride_h : 1; im.mul_x = which == 0 ? g.stride_w : 1;
    im.off_y = which == 0 ? -g.pad_h : g.pad_h; im.off_x = which == 0 ? -g.pad_w : g.pad_w;
    im.tap_sign = which == 0 ? 1 : -1;
    im.R = g.r; im.S = g.s;
    im.rows = (int)N;
    im.r0 = make_fastdiv((int)gx); im.r1 = make_fastdiv((int)gy);
    im.ks = make_fastdiv(g.s);
    Gather ft{};
    ft.kind = kSrcFilterTap;
    ft.k0 = make_fastdiv(tc);
    // filter [K][C][R][S]: forward row = filter, k = (tap, c); dgrad row = c, k = (tap, filter)
    ft.th = which == 0 ? g.c * rs : rs;
    ft.tw = which == 0 ? rs : g.c * rs;
    const OperandSpec sa{filt, 0, true, ft, 0};
    const OutSpec os{out, 0, (int)(gy * gx)};
    const bool planes = conv_planes(f, p, (double)g.n * gy * gx * g.k * g.c * rs, which == 0 ? kLeastForward : kLeastDgrad) && elems > 0 && (elems / 8) * 3 + (int64_t)(g.r * tw + g.s) * (tc / 8) < ((int64_t)1 << 31);
    if (planes) {
        const int rc = run_implicit_window((int)M, (int)N, (int)K, sa, (int64_t)g.k * g.c * rs, tensor, elems, (int)(th * tw), im, os, f, p, stream);
        if (rc <= 0) return rc;
    }
    const bool ftz = f.denorm == 0;
#define FMT_IMPL2(MD, FZ)                                                                                                     \
    (sch.ps == 0   ? run_implicit<MD, FZ, 0>((int)M, (int)N, (int)K, sa, tensor, elems, (int)(th * tw), im, os, f, p, stream) \
     : sch.ps == 1 ? run_implicit<MD, FZ, 1>((int)M, (int)N, (int)K, sa, tensor, elems, (int)(th * tw), im, os, f, p, stream) \
     : sch.ps == 2 ? run_implicit<MD, FZ, 2>((int)M, (int)N, (int)K, sa, tensor, elems, (int)(th * tw), im, os, f, p, stream) \
                   : run_implicit<MD, FZ, 3>((int)M, (int)N, (int)K, sa, tensor, elems, (int)(th * tw), im, os, f, p, stream))
#define FMT_IMPL(MD) (ftz ? FMT_IMPL2(MD, true) : FMT_IMPL2(MD, false))
    if (p.mode == kModeMagic) return FMT_IMPL(kModeMagic);
    if (p.mode == kModeInteger) return FMT_IMPL(kModeInteger);
    return FMT_IMPL(kModeMixed);
#undef FMT_IMPL
#undef FMT_IMPL2
}

// Convolutions (Sec. IV-A) as products on patches that are never materialised in fp32.
//   forward  Y[n][k][p][q]:  M = K filters (rows of the filter matrix), N = n*P*Q output positions
//            (patches of X), k = C*R*S, result stored NCHW
//   dgrad    dX[n][c][h][w]: M = C (filter seen from the input channel), N = n*H*W input positions
//            (patches of dY through the taps that reach them), k = K*R*S, result stored NCHW
//   wgrad    dW[k][c][r][s]: M = K (dY as [K][n*P*Q]), N = C*R*S (patches of X, transposed),
//            k = n*P*Q, result is the plain [K][C*R*S] matrix
// Forward and (stride 1) dgrad with a channel count that is a multiple of 32 and at most 32 taps gather
// the patches inside the product kernel from the once-rounded tensor (conv_implicit: scratch is 2P bytes
// per TENSOR element); the other cases, and wgrad, go through a prepare pass that gathers from the once
// rounded tensor into a patch-sized 16-bit prepared operand.  1/6/8 and 1/6/9 take exponent planes where conv_planes says so (6 bytes
// instead of 4 per element of scratch).
int launch_conv2d(int which, const fmt_conv2d_t &g, const float *a, const float *b, float *out, fmt_format_t f,
                  const QuantParams &p, hipStream_t stream)
{
    const int64_t P = (g.h + 2 * g.pad_h - g.r) / g.stride_h + 1, Q = (g.w + 2 * g.pad_w - g.s) / g.stride_w + 1;
    Gather patch{};
    patch.R = g.r;
    patch.S = g.s;
    Gather none{};
    if (which == 0) {
        const int64_t M = g.k, N = (int64_t)g.n * P * Q, K = (int64_t)g.c * g.r * g.s;
        if (M == 0 || N == 0) return FMT_OK;
        patch.kind = kSrcPatchRows;
        patch.tc = g.c; patch.th = g.h; patch.tw = g.w;
        patch.gy = (int)P; patch.gx = (int)Q;
        patch.mul_y = g.stride_h; patch.mul_x = g.stride_w; patch.off_y = -g.pad_h; patch.off_x = -g.pad_w;
        patch.tap = 1; patch.den_y = 1; patch.den_x = 1;
        patch.r0 = make_fastdiv(patch.gx); patch.r1 = make_fastdiv(patch.gy);
        patch.k0 = make_fastdiv(g.s); patch.k1 = make_fastdiv(g.r);
        if (K == 0) return zero_fill(out, (int64_t)g.n * M, P * Q, P * Q, stream);
        {
            const int rci = conv_implicit(0, g, P, Q, a, b, out, f, p, stream);
            if (rci <= 0) return rci;
        }
        const OperandSpec sa{b, K, true, none, 0};                 // filter [K][C*R*S]
        const OperandSpec sb{a, 0, false, patch, (int64_t)g.n * g.c * g.h * g.w};   // patches of X, lanes along positions
        return run_product((int)M, (int)N, (int)K, sa, sb, OutSpec{out, 0, (int)(P * Q)}, f, p, stream);
    }
    if (which == 1) {
        const int64_t M = g.c, N = (int64_t)g.n * g.h * g.w, K = (int64_t)g.k * g.r * g.s;
        if (M == 0 || N == 0) return FMT_OK;
        patch.kind = kSrcPatchRows;
        patch.tc = g.k; patch.th = (int)P; patch.tw = (int)Q;
        patch.gy = g.h; patch.gx = g.w;
        patch.mul_y = 1; patch.mul_x = 1; patch.off_y = g.pad_h; patch.off_x = g.pad_w;
        patch.tap = -1; patch.den_y = g.stride_h; patch.den_x = g.stride_w;
        patch.r0 = make_fastdiv(patch.gx); patch.r1 = make_fastdiv(patch.gy);
        patch.k0 = make_fastdiv(g.s); patch.k1 = make_fastdiv(g.r);
        if (K == 0) return zero_fill(out, (int64_t)g.n * M, (int64_t)g.h * g.w, (int64_t)g.h * g.w, stream);
        {
            const int rci = conv_implicit(1, g, P, Q, a, b, out, f, p, stream);
            if (rci <= 0) return rci;
        }
        Gather ft{};
        ft.kind = kSrcFilterT;
        ft.tc = g.c; ft.R = g.r; ft.S = g.s;
        ft.k0 = make_fastdiv(g.r * g.s);
        const OperandSpec sa{b, 0, true, ft, 0};                   // filter as [C][K*R*S]
        const OperandSpec sb{a, 0, false, patch, (int64_t)g.n * g.k * P * Q};       // patches of dY
        return run_product((int)M, (int)N, (int)K, sa, sb, OutSpec{out, 0, g.h * g.w}, f, p, stream);
    }
    const int64_t M = g.k, N = (int64_t)g.c * g.r * g.s, K = (int64_t)g.n * P * Q;
    if (M == 0 || N == 0) return FMT_OK;
    if (K == 0) return zero_fill(out, M, N, N, stream);
    Gather ch{};
    ch.kind = kSrcChannelRows;
    ch.tc = g.k; ch.th = (int)P; ch.tw = (int)Q;
    ch.k0 = make_fastdiv((int)(P * Q));
    patch.kind = kSrcPatchK;
    patch.tc = g.c; patch.th = g.h; patch.tw = g.w;
    patch.gy = (int)P; patch.gx = (int)Q;
    patch.mul_y = g.stride_h; patch.mul_x = g.stride_w; patch.off_y = -g.pad_h; patch.off_x = -g.pad_w;
    patch.tap = 1; patch.den_y = 1; patch.den_x = 1;
    patch.r0 = make_fastdiv(g.s); patch.r1 = make_fastdiv(g.r);
    patch.k0 = make_fastdiv(patch.gx); patch.k1 = make_fastdiv(patch.gy);
    const OperandSpec sa{a, 0, true, ch, 0};                       // dY as [K][n*P*Q]
    const OperandSpec sb{b, 0, true, patch, (int64_t)g.n * g.c * g.h * g.w};      // patches of X, k along positions
    if (conv_planes(f, p, (double)M * N * K, kLeastWgrad) && g.r * g.s <= 32 && sb.pre_elems > 0) {
        const int rc = run_wgrad_window((int)M, (int)N, (int)K, sa, M * K, sb, OutSpec{out, N, 0}, f, p, stream);
        if (rc <= 0) return rc;
    }
    return run_product((int)M, (int)N, (int)K, sa, sb, OutSpec{out, N, 0}, f, p, stream);
}

}  // namespace fmt
