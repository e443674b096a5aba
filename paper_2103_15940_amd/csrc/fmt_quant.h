// Device-side rounding to a 1/e/m format on the fp32 bit pattern (Sec. IV-A), shared by the
// stream kernels and the GEMM operand loaders.
#pragma once

#include "fmt_internal.h"

namespace fmt {

// How the rounding is carried out (uniform per launch, chosen on the host from (e, m)):
enum : int {
    kModeMagic = 0,    // e < 8, m <= 22: (|x| + C) - C with C = 2^(max(E, Emin) + 23 - m)
    kModeInteger = 1,  // e == 8: RNE on the integer pattern (fp32's denormal grid is the format's own)
    kModeMixed = 2     // e < 8, m == 23: nothing to round at or above minN, fixed grid below
};

// Q_{e,m,d|n} on one fp32 bit pattern.
template <int MODE, bool FTZ>
__device__ __forceinline__ uint32_t quantize_bits(uint32_t u, const QuantParams &p)
{
    const uint32_t a = u & 0x7FFFFFFFu;
    uint32_t r;
    if (MODE == kModeMagic) {
        // C has ulp 2^(max(E,Emin)-m) and |x| < C, so the hardware's RNE addition lands on the
        // format's grid and the subtraction is exact.  For |x| >= t_ovf the pattern of C may be
        // meaningless; those lanes are overwritten below.
        const uint32_t ce = max(a & 0x7F800000u, p.minn_bits) + p.shift23;
        const float c = __uint_as_float(ce);
        r = __float_as_uint((__uint_as_float(a) + c) - c);
    } else if (MODE == kModeInteger) {
        const uint32_t lsb = __builtin_amdgcn_ubfe(a, p.shift, p.lsb_width);
        r = (a + p.rbias + lsb) & p.nmask;
    } else {
        const float rbf = (__uint_as_float(a) + p.cmagic) - p.cmagic;
        r = (a < p.minn_bits) ? __float_as_uint(rbf) : a;
    }
    if (FTZ) r = (a < p.t_den) ? 0u : r;
    r = (a >= p.t_ovf) ? 0x7F800000u : r;
    r |= (u & 0x80000000u);
    return (a > 0x7F800000u) ? 0x7FC00000u : r;
}

// What programs round is finite and far from overflow.  A run of elements in which every |x| is below t_ovf (a look of one
// instruction per two elements) takes the short form: 5 vector instructions per element (7 with the flush; e == 8: 3 and 6)
// where quantize_bits takes 13 to 15.

// Constants in registers: v_and_or_b32 takes no literal, and one scalar operand only.
struct RoundMasks {
    uint32_t exponent, half, sign, floor;        // 0x7F800000, 0x00400000, 0x80000000 and the pattern of 1.5 * minN
};

__device__ __forceinline__ RoundMasks round_masks(const QuantParams &p)
{
    RoundMasks k{0x7F800000u, 0x00400000u, 0x80000000u, p.minn_bits | 0x00400000u};
    asm("" : "+s"(k.exponent), "+v"(k.half));
    asm("" : "+s"(k.sign));
    return k;
}

// Whether an |x| of a run is at or above t_ovf, infinite or NaN (v_maximum3_f32 hands a NaN on; not as inline assembly: a run may
// come straight from the matrix cores, whose results the compiler knows when to read).
template <int N>
__device__ __forceinline__ bool run_is_rare(const uint32_t (&u)[N], const QuantParams &p)
{
    static_assert(N % 2 == 0, "pairs");
    float top = 0.0f;
#pragma unroll
    for (int j = 0; j < N; j += 2)
        top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(__uint_as_float(u[j])), fabsf(__uint_as_float(u[j + 1]))), top);
    return !(top < __uint_as_float(p.t_ovf));
}

// Q of one element with |x| < t_ovf.  e < 8: (C + x) - C with C = 1.5 * 2^(max(E, Emin) + 23 - m), whose last place is the format's step
// for either sign of x; C is formed inside the two fused multiply-adds.  e == 8: to nearest even on the integer pattern.  SIGN: the sign of a zero is kept.
template <int MODE, bool FTZ, bool SIGN = true>
__device__ __forceinline__ uint32_t quantize_short(uint32_t u, const QuantParams &p, const RoundMasks &k)
{
    static_assert(MODE != kModeMixed, "no short form");
    if constexpr (MODE == kModeMagic) {
        const float c = __uint_as_float(max((u & k.exponent) | k.half, k.floor)), scale = __uint_as_float((127u + p.shift) << 23);
        float q = __fmaf_rn(c, -scale, __fmaf_rn(c, scale, __uint_as_float(u)));
        if (FTZ) q = fabsf(q) < __uint_as_float(p.minn_bits) ? 0.0f : q;
        return SIGN ? (u & k.sign) | __float_as_uint(q) : __float_as_uint(q);
    } else {
        uint32_t r = (u + p.rbias + __builtin_amdgcn_ubfe(u, p.shift, p.lsb_width)) & p.nmask;
        // On its way to the matrix cores as floats, denormal ones among them: the magnitude costs that comparison nothing (64 x 256 x 784 in
        // 1/8/7/n in one launch 11.9 -> 10.6 us).  Not where statistics need the magnitude's pattern anyway (a layer 48.6 -> 50.1).
        if (FTZ && SIGN) r = (u & 0x7FFFFFFFu) < p.t_den ? u & 0x80000000u : r;
        if (FTZ && !SIGN) r = fabsf(__uint_as_float(u)) < __uint_as_float(p.t_den) ? 0u : r;
        return r;
    }
}

// Q of a run; rare: what run_is_rare says of it.
template <int MODE, bool FTZ, int N>
__device__ __forceinline__ void quantize_run(const uint32_t (&u)[N], bool rare, const QuantParams &p, const RoundMasks &k, uint32_t (&r)[N])
{
    if constexpr (MODE != kModeMixed) {
        if (__ballot(rare) == 0ull) {            // the same in the whole wave
#pragma unroll
            for (int j = 0; j < N; ++j) r[j] = quantize_short<MODE, FTZ>(u[j], p, k);
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) r[j] = quantize_bits<MODE, FTZ>(u[j], p);
}

// (1+e+m)-bit code (Sec. III) of r, the pattern of a value of the format (quantize_bits' result);
// needs 1 + e + m <= 16, so MODE is kModeMagic (e < 8) or kModeInteger (e == 8).  At or above minN
// the code is the fp32 pattern rebased to the format's bias and shifted; below minN the stored
// mantissa is |r| / minD, read off the pattern of |r| + minN (exact: |r| is a multiple of minD);
// with e == 8 fp32's own denormal patterns are the format's.
template <int MODE>
__device__ __forceinline__ uint32_t encode_bits(uint32_t r, const QuantParams &p)
{
    const uint32_t a = r & 0x7FFFFFFFu;
    uint32_t ae = a;
    if (MODE != kModeInteger) {
        const float t = __uint_as_float(a) + __uint_as_float(p.minn_bits);
        ae = a < p.minn_bits ? __float_as_uint(t) - 0x00800000u : a;
    }
    uint32_t c = (ae - (p.minn_bits - 0x00800000u)) >> p.shift;
    const uint32_t quiet = 1u << (22u - p.shift);                          // top mantissa bit, 2^(m-1)
    c = a >= 0x7F800000u ? (a > 0x7F800000u ? p.top_code | quiet : p.top_code) : c;
    return c | ((r >> 31) << p.sign_pos);
}

// fp32 pattern of the value of a (1+e+m)-bit code; bits above the sign are ignored, NaN codes
// give the quiet NaN 0x7FC00000.  INTEGER: e == 8.
template <bool INTEGER>
__device__ __forceinline__ uint32_t decode_bits(uint32_t code, const QuantParams &p)
{
    const uint32_t body = code & ((1u << p.sign_pos) - 1u);
    const uint32_t sign = ((code >> p.sign_pos) & 1u) << 31;
    uint32_t a = (body << p.shift) + (p.minn_bits - 0x00800000u);
    if (!INTEGER) {
        // exponent field 0: mantissa * minD = (minN with that mantissa) - minN, exactly
        const float t = __uint_as_float(p.minn_bits | (body << p.shift)) - __uint_as_float(p.minn_bits);
        a = body < (1u << (23u - p.shift)) ? __float_as_uint(t) : a;
    }
    if (body >= p.top_code) return body == p.top_code ? (0x7F800000u | sign) : 0x7FC00000u;
    return a | sign;
}

// The same rounding with the variant chosen at run time (uniform per launch), for kernels that
// round a handful of values and are not worth six instantiations.
__device__ __forceinline__ uint32_t quantize_bits_rt(uint32_t u, const QuantParams &p, bool ftz)
{
    if (p.mode == kModeMagic) return ftz ? quantize_bits<kModeMagic, true>(u, p) : quantize_bits<kModeMagic, false>(u, p);
    if (p.mode == kModeInteger) return ftz ? quantize_bits<kModeInteger, true>(u, p) : quantize_bits<kModeInteger, false>(u, p);
    return ftz ? quantize_bits<kModeMixed, true>(u, p) : quantize_bits<kModeMixed, false>(u, p);
}

// Outputs of a fully connected layer from their accumulators, in place (Sec. IV-A): R(R(acc) + R(b)), two roundings around ONE
// single-precision addition; without a bias the second rounding changes nothing.  get(i) / set(i, y): the i-th of N accumulators;
// bias(i): its column's unrounded bias (the caller loads them early: they come from memory).  The variant of the rounding is
// chosen once for all of them.
template <int N, class GET, class SET, class BIAS>
__device__ __forceinline__ void linear_round(const LinearRound &lin, GET &&get, SET &&set, BIAS &&bias)
{
    const bool has_bias = lin.bias != nullptr;
    auto run = [&](auto round) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            uint32_t r = round(__float_as_uint(get(i)));
            if (has_bias) r = round(__float_as_uint(__fadd_rn(__uint_as_float(r), __uint_as_float(round(bias(i))))));
            set(i, __uint_as_float(r));
        }
    };
    const QuantParams &p = lin.p;
    if (p.mode == kModeInteger) {
        if (lin.ftz) run([&](uint32_t u) { return quantize_bits<kModeInteger, true>(u, p); });
        else run([&](uint32_t u) { return quantize_bits<kModeInteger, false>(u, p); });
    } else if (p.mode == kModeMagic) {
        if (lin.ftz) run([&](uint32_t u) { return quantize_bits<kModeMagic, true>(u, p); });
        else run([&](uint32_t u) { return quantize_bits<kModeMagic, false>(u, p); });
    } else {
        if (lin.ftz) run([&](uint32_t u) { return quantize_bits<kModeMixed, true>(u, p); });
        else run([&](uint32_t u) { return quantize_bits<kModeMixed, false>(u, p); });
    }
}

// Unrounded bias of a column (0 without a bias or beyond the columns).
__device__ __forceinline__ uint32_t linear_bias(const LinearRound &lin, int col, int N)
{
    return lin.bias != nullptr && col < N ? __float_as_uint(lin.bias[col]) : 0u;
}

}  // namespace fmt
