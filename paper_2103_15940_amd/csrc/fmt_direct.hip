// Small products of two fp32 matrices in one launch: the operands are rounded on the way into the matrix cores
// (fmt_gemm.hip chooses between this and its own route of prepared operands).
#include <type_traits>

#include "fmt_internal.h"
#include "fmt_quant.h"
#include "fmt_split.h"

namespace fmt {

// An fp32 matrix operand of a direct product: element (row, k) at X[row*row_step + k*k_step], one of the two 1.  VEC:
// k_step == 1; k is then loaded in 16-byte vectors, which global memory accesses take at any 4-byte alignment.
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
struct DirectOperand {
    const uint32_t *X;
    uint32_t row_step, k_step;       // every offset of an element fits 32 bits (the host checks)
    int rows;
};

// C = Q(A) Q(B)^T of two fp32 matrices in one launch, for products so small that the three launches of the general route
// (prepare, product, sum of the k parts: 5 - 6 us each on the GPU and 3 us each on the host) are what they cost.
// A wave owns a block of 32 x 32 results and one of `parts` ranges of k; it loads its operands straight into
// the layout of the MFMA fragments (lane l: row l % 32, eight consecutive k), rounds and splits them in
// registers and multiplies: no LDS, no barrier, the next 32 k in flight meanwhile.  The parts of a block
// meet in LDS and are summed in order.  Every element is rounded once per block of its row or column instead of
// once, which is what bounds it (vector instructions) and why larger products keep the general route
// (direct_parts).  The sums are those of the general route bit for bit when `parts` is its plan's: same pieces, same
// steps of 16 k, same order.
template <int MODE, bool FTZ, int PS, bool AVEC, bool BVEC>
__global__ __launch_bounds__(512) void direct_product_kernel(DirectOperand a, DirectOperand b, float *__restrict__ C, int64_t ldc,
                                                              int M, int N, int K, int kblocks, int tiles_m, int ntiles, int parts,
                                                              int kb_per, int tiles_per_wg, QuantParams p, LinearRound lin, int linear)
{
    constexpr int P = pieces_of(PS);
    extern __shared__ float s_part[];            // parts > 1: [wave][16][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = wave % parts, tile = blockIdx.x * tiles_per_wg + wave / parts;
    const bool live = tile < ntiles;
    const int row0 = (tile % tiles_m) * 32, col0 = (tile / tiles_m) * 32;
    const int kb0 = part * kb_per, kb1 = live ? min(kblocks, kb0 + kb_per) : 0;

    uint32_t bias[16];                           // a layer's bias, loaded ahead of the products (columns as below)
    if (linear) {
#pragma unroll
        for (int v = 0; v < 16; ++v) bias[v] = linear_bias(lin, col0 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3), N);
    }

    const RoundMasks masks = round_masks(p);

    // Rows beyond the operand read its last row: their results are not stored.  A load's address is one that is the same in
    // the whole wave plus a lane's offset.
    const int half = lane >> 5;
    const uint32_t off_a = (uint32_t)min(row0 + (lane & 31), a.rows - 1) * a.row_step + (uint32_t)half * 8u * a.k_step;
    const uint32_t off_b = (uint32_t)min(col0 + (lane & 31), b.rows - 1) * b.row_step + (uint32_t)half * 8u * b.k_step;
    // no branch in here: the compiler keeps the loads of several blocks in flight
    auto load_one = [&](auto vec, const DirectOperand &o, uint32_t off, int kb, uint32_t (&raw)[2][8]) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const uint32_t *src = o.X + (size_t)(uint32_t)(kb * kUnitK + kk * 16) * o.k_step;
            if constexpr (decltype(vec)::value) {
                const u32x4u lo = *reinterpret_cast<const u32x4u *>(src + off), hi = *reinterpret_cast<const u32x4u *>(src + off + 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    raw[kk][j] = lo[j];
                    raw[kk][4 + j] = hi[j];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j, src += o.k_step) raw[kk][j] = src[off];
            }
        }
    };
    auto load = [&](int kb, uint32_t (&raw)[2][2][8]) __attribute__((always_inline)) {
        load_one(std::integral_constant<bool, AVEC>{}, a, off_a, kb, raw[0]);
        load_one(std::integral_constant<bool, BVEC>{}, b, off_b, kb, raw[1]);
    };
    // The block that K ends in, zero beyond K.  A lane's eight k that K cuts are loaded as the last eight of the row and
    // moved down; single elements (and rows shorter than eight) beyond K read the last k: no load waits behind a test of its own.
    auto load_last = [&](auto vec, const DirectOperand &o, uint32_t off, int kb, uint32_t (&raw)[2][8]) __attribute__((always_inline)) {
        const uint32_t *row = o.X + (off - (uint32_t)half * 8u * o.k_step);
        if (decltype(vec)::value && K >= 8) {
            int skip[2];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int k0 = kb * kUnitK + kk * 16 + half * 8, at = min(k0, K - 8);
                const u32x4 lo = *reinterpret_cast<const u32x4u *>(row + at), hi = *reinterpret_cast<const u32x4u *>(row + at + 4);
                skip[kk] = k0 - at;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    raw[kk][j] = lo[j];
                    raw[kk][4 + j] = hi[j];
                }
            }
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int by = 1; by <= 8; by *= 2) {
                    const bool move = by < 8 ? (skip[kk] & by) != 0 : skip[kk] >= 8;
#pragma unroll
                    for (int j = 0; j < 8; ++j) raw[kk][j] = !move ? raw[kk][j] : j + by < 8 ? raw[kk][j + by < 8 ? j + by : 7] : 0u;
                }
        } else {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = kb * kUnitK + kk * 16 + half * 8 + j;
                    const uint32_t v = row[(size_t)(uint32_t)min(k, K - 1) * o.k_step];
                    raw[kk][j] = k < K ? v : 0u;
                }
        }
    };
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    auto multiply = [&](const uint32_t (&raw)[2][2][8]) __attribute__((always_inline)) {
        u32x4 f[2][2][P];                                            // [operand][16 k][piece]
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) direct_convert<MODE, FTZ, PS>(raw[o][kk], p, masks, f[o][kk]);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int qa = 0; qa < P; ++qa)
#pragma unroll
                for (int qb = 0; qb < P; ++qb)                       // B's fragment first: the block comes out transposed (see store_tile)
                    acc = PS == 0 ? __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, f[1][kk][qb]),
                                                                          __builtin_bit_cast(f16x8, f[0][kk][qa]), acc, 0, 0, 0)
                                  : __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f[1][kk][qb]),
                                                                            __builtin_bit_cast(bf16x8, f[0][kk][qa]), acc, 0, 0, 0);
    };
    // kDepth blocks of 32 k are in flight: a block takes 0.4 us of rounding and multiplying, a load up to three times that
    constexpr int kDepth = 4;
    const int whole = min(kb1, K / kUnitK);                          // blocks [kb0, whole) lie inside K; at most one more follows
    uint32_t raw[kDepth][2][2][8];
#pragma unroll
    for (int u = 0; u < kDepth; ++u)
        if (kb0 + u < whole) load(kb0 + u, raw[u]);
    for (int kb = kb0; kb < whole; kb += kDepth) {
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            if (kb + u >= whole) break;                              // the same in the whole wave
            multiply(raw[u]);
            if (kb + u + kDepth < whole) load(kb + u + kDepth, raw[u]);
        }
    }
    if (kb0 <= whole && whole < kb1) {                                // the block that K ends in, if it is this part's
        load_last(std::integral_constant<bool, AVEC>{}, a, off_a, whole, raw[0][0]);
        load_last(std::integral_constant<bool, BVEC>{}, b, off_b, whole, raw[0][1]);
        multiply(raw[0]);
    }

    // register 4g + c of lane l: row l % 32, column 8g + 4 (l / 32) + c of the block
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const int row = row0 + (lane & 31);
    auto put = [&](int g, float x0, float x1, float x2, float x3) __attribute__((always_inline)) {
        const int col = col0 + g * 8 + half * 4;
        if (row >= M || col >= N) return;
        if (linear) {                                                // a layer's output roundings
            float y[4] = {x0, x1, x2, x3};
            linear_round<4>(lin, [&](int i) { return y[i]; }, [&](int i, float v) { y[i] = v; }, [&](int i) { return bias[4 * g + i]; });
            x0 = y[0], x1 = y[1], x2 = y[2], x3 = y[3];
        }
        float *dst = C + (size_t)row * ldc + col;
        if (col + 3 < N) {
            *reinterpret_cast<f32x4u *>(dst) = f32x4u{x0, x1, x2, x3};
        } else {
            dst[0] = x0;
            if (col + 1 < N) dst[1] = x1;
            if (col + 2 < N) dst[2] = x2;
        }
    };
    if (parts == 1) {
        if (!live) return;
#pragma unroll
        for (int g = 0; g < 4; ++g) put(g, acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
        return;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) s_part[(wave * 16 + v) * 64 + lane] = acc[v];
    __syncthreads();
    if (!live) return;
    const int w0 = wave - part;                                      // the block's first wave
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (g % parts != part) continue;                             // the same in the whole wave
        float sum[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            sum[c] = 0.0f;
            for (int q = 0; q < parts; ++q) sum[c] += s_part[((w0 + q) * 16 + 4 * g + c) * 64 + lane];
        }
        put(g, sum[0], sum[1], sum[2], sum[3]);
    }
}

template <int MODE, bool FTZ, int PS>
static int launch(int M, int N, int K, const MatrixOperand &A, const MatrixOperand &B, float *C, int64_t ldc, int parts,
                  const QuantParams &p, const LinearRound *lin, hipStream_t stream)
{
    auto operand = [](const MatrixOperand &m, int rows) {
        return DirectOperand{reinterpret_cast<const uint32_t *>(m.X), m.kcontig ? (uint32_t)m.ld : 1u, m.kcontig ? 1u : (uint32_t)m.ld, rows};
    };
    const int kblocks = (K + kUnitK - 1) / kUnitK;
    const int tiles_m = (M + 31) / 32, tiles = tiles_m * ((N + 31) / 32);
    const int per_wg = direct_blocks_per_workgroup(parts);
    const int waves = parts * per_wg;
    const size_t lds = parts > 1 ? (size_t)waves * 16 * 64 * sizeof(float) : 0;
    auto kern = A.kcontig ? (B.kcontig ? direct_product_kernel<MODE, FTZ, PS, true, true> : direct_product_kernel<MODE, FTZ, PS, true, false>)
                          : (B.kcontig ? direct_product_kernel<MODE, FTZ, PS, false, true> : direct_product_kernel<MODE, FTZ, PS, false, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)((tiles + per_wg - 1) / per_wg)), dim3(64 * waves), lds, stream, operand(A, M), operand(B, N), C,
                       ldc, M, N, K, kblocks, tiles_m, tiles, parts, (kblocks + parts - 1) / parts, per_wg, p,
                       lin != nullptr ? *lin : LinearRound{}, lin != nullptr ? 1 : 0);
    FMT_HIP_CHECK(hipGetLastError());
    return FMT_OK;
}

// C (M x N) = Q(A) Q(B)^T; K >= 1, 1 <= parts <= kDirectParts, fewer than 2^31 blocks of 32 x 32 (the caller's size limit).
int launch_direct_product(int M, int N, int K, const MatrixOperand &A, const MatrixOperand &B, float *C, int64_t ldc, int parts, int ps,
                          bool ftz, const QuantParams &p, const LinearRound *lin, hipStream_t stream)
{
    if (parts < 1 || parts > kDirectParts) return FMT_ERR_SHAPE;
#define FMT_RUN(MD, PSV)                                                                      \
    (ftz ? launch<MD, true, PSV>(M, N, K, A, B, C, ldc, parts, p, lin, stream)                      \
         : launch<MD, false, PSV>(M, N, K, A, B, C, ldc, parts, p, lin, stream))
    if (p.mode == kModeMagic && ps == 0) return FMT_RUN(kModeMagic, 0);
    if (p.mode == kModeMagic && ps == 1) return FMT_RUN(kModeMagic, 1);
    if (p.mode == kModeMagic && ps == 2) return FMT_RUN(kModeMagic, 2);
    if (p.mode == kModeInteger && ps == 1) return FMT_RUN(kModeInteger, 1);
    return FMT_ERR_FORMAT;                       // direct_parts leaves the others to the general route
#undef FMT_RUN
}

}  // namespace fmt
