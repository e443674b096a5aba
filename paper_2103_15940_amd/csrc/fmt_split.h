// How a rounded value reaches the matrix cores, shared by the kernels that prepare operands and the one that rounds
// them on the way in.
#pragma once

#include <type_traits>

#include "fmt_internal.h"
#include "fmt_quant.h"

namespace fmt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Piece scheme PS: 1, 2, 3 = that many bf16 pieces; 0 = one fp16 piece (formats inside binary16).
constexpr int pieces_of(int ps) { return ps == 0 ? 1 : ps; }
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kUnitRows = 32;                 // rows per unit (one MFMA fragment)
constexpr int kUnitK = 32;                    // k per unit (two MFMA steps of 16)
constexpr int kUnitVec = kUnitRows * kUnitK * 2 / 16;   // 16-byte vectors per unit per piece = 128
constexpr int kFastRows = 4;                  // groups of 64 rows per workgroup in the fast patch gather (kRowPad = 64 * kFastRows)
constexpr int kRowPad = 256;                  // prepared operands are padded to a multiple of this many rows

// Rounds one fp32 pattern to the format and splits the result into the 16-bit patterns of its
// pieces: P bf16 pieces, or the single fp16 pattern when the format's values are all binary16
// values (e <= 5, m <= 10).
template <int MODE, bool FTZ, int PS>
__device__ __forceinline__ void round_and_split(uint32_t u, const QuantParams &p, uint32_t (&piece)[pieces_of(PS)])
{
    constexpr int P = pieces_of(PS);
    const uint32_t r = quantize_bits<MODE, FTZ>(u, p);
    if (PS == 0) {
        // exact fp32 -> fp16 of a value known to be representable: normal numbers by moving the
        // fields, denormals as the integer count of 2^-24 steps (an exact fp32 product)
        const uint32_t a = r & 0x7FFFFFFFu;
        uint32_t h = a >= 0x38800000u ? (a - 0x38000000u) >> 13 : (uint32_t)(__uint_as_float(a) * 16777216.0f);
        h = a >= 0x7F800000u ? (a > 0x7F800000u ? 0x7E00u : 0x7C00u) : h;
        piece[0] = h | ((r >> 16) & 0x8000u);
        return;
    }
    const uint32_t hi = r & 0xFFFF0000u;
    piece[0] = hi >> 16;
    if (P >= 2) {
        // infinities and NaN stay in the first piece alone
        const bool finite = (r & 0x7F800000u) != 0x7F800000u;
        const float rem = finite ? __uint_as_float(r) - __uint_as_float(hi) : 0.0f;   // exact
        const uint32_t rb = __float_as_uint(rem);
        piece[P >= 2 ? 1 : 0] = rb >> 16;
        if (P >= 3) {
            const float rem2 = rem - __uint_as_float(rb & 0xFFFF0000u);                // exact
            piece[P >= 3 ? 2 : 0] = __float_as_uint(rem2) >> 16;
        }
    }
}

// binary16 and bfloat16 themselves: the conversion of the vector units, two elements per instruction, is the rounding with denormals
// kept -- equal to round_and_split over all 2^32 patterns, infinities included (NaN stay NaN) -- so nothing is rare.
constexpr bool hardware_scheme(int mode, int ps) { return (mode == kModeMagic && ps == 0) || (mode == kModeInteger && ps == 1); }
template <int MODE, int PS>
__device__ __forceinline__ bool hardware_format(const QuantParams &p)
{
    if constexpr (!hardware_scheme(MODE, PS)) return false;
    return PS == 0 ? p.shift == 13u && p.minn_bits == 0x38800000u : p.shift == 16u;
}

template <bool FTZ, int PS>
__device__ __forceinline__ void hardware_convert(const uint32_t (&v)[8], const QuantParams &p, u32x4 (&out)[1])
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef typename std::conditional<PS == 0, _Float16, __bf16>::type half_t;
    typedef half_t half2_t __attribute__((ext_vector_type(2)));
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        x[j] = __uint_as_float(v[j]);
        if (FTZ) x[j] = fabsf(x[j]) < __uint_as_float(p.t_den) ? 0.0f : x[j];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) out[0][i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x[2 * i], x[2 * i + 1]}), half2_t));
}

// Eight consecutive k of one row (fp32 patterns) as MFMA operand vectors, one per piece: Q and the split of
// round_and_split.  What a product of network tensors meets is finite and far from overflow, so the
// common path takes the short form of the rounding (the sign of a zero is lost, which no sum can show: it starts from +0) and looks once per
// eight elements whether the wave holds anything else.  5 to 8 vector instructions per element where the general path takes about 20.
constexpr bool direct_form(int mode, int ps) { return (mode == kModeMagic && ps <= 2) || (mode == kModeInteger && ps == 1); }

template <int MODE, bool FTZ, int PS>
__device__ __forceinline__ void short_convert(const uint32_t (&v)[8], const QuantParams &p, const RoundMasks &k, u32x4 (&out)[pieces_of(PS)])
{
    constexpr int P = pieces_of(PS);
    static_assert(direct_form(MODE, PS), "formats with a short form");
    uint32_t r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = quantize_short<MODE, FTZ, false>(v[j], p, k);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (PS == 0) {         // values of the format are binary16 values: the conversion is exact
            out[0][i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(r[2 * i]), __uint_as_float(r[2 * i + 1])));
        } else {
            out[0][i] = __builtin_amdgcn_perm(r[2 * i + 1], r[2 * i], 0x07060302u);
            if constexpr (P >= 2) {
                const float l0 = __uint_as_float(r[2 * i]) - __uint_as_float(r[2 * i] & 0xFFFF0000u);              // exact
                const float l1 = __uint_as_float(r[2 * i + 1]) - __uint_as_float(r[2 * i + 1] & 0xFFFF0000u);
                out[P >= 2 ? 1 : 0][i] = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);
            }
        }
    }
}

template <int MODE, bool FTZ, int PS>
__device__ __forceinline__ void direct_convert(const uint32_t (&v)[8], const QuantParams &p, const RoundMasks &k,
                                               u32x4 (&out)[pieces_of(PS)])
{
    constexpr int P = pieces_of(PS);
    if constexpr (hardware_scheme(MODE, PS)) {
        if (hardware_format<MODE, PS>(p)) {
            hardware_convert<FTZ, PS>(v, p, out);
            return;
        }
    }
    if (__ballot(run_is_rare(v, p)) == 0ull) {            // the same in the whole wave
        short_convert<MODE, FTZ, PS>(v, p, k, out);
        return;
    }
    uint32_t pc[8][P];
#pragma unroll
    for (int j = 0; j < 8; ++j) round_and_split<MODE, FTZ, PS>(v[j], p, pc[j]);
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[q][i] = pc[2 * i][q] | (pc[2 * i + 1][q] << 16);
}

// The same for any format: two elements per word, one set of words per piece.
template <int MODE, bool FTZ, int PS>
__device__ __forceinline__ void split8(const uint32_t (&v)[8], const QuantParams &p, u32x4 (&out)[pieces_of(PS)])
{
    constexpr int P = pieces_of(PS);
    if constexpr (direct_form(MODE, PS)) {
        direct_convert<MODE, FTZ, PS>(v, p, round_masks(p), out);
    } else {
        uint32_t pc[8][P];
#pragma unroll
        for (int j = 0; j < 8; ++j) round_and_split<MODE, FTZ, PS>(v[j], p, pc[j]);
#pragma unroll
        for (int q = 0; q < P; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) out[q][i] = pc[2 * i][q] | (pc[2 * i + 1][q] << 16);
    }
}

}  // namespace fmt
