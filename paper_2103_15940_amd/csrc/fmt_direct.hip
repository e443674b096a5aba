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

// LDS of a wave, in bytes: per staged operand and piece 4 chunks of 8 k x 32 rows of 16 bytes; the 32 bytes between chunks put the 16 lanes that
// write at a time (two rows, 32 k) on different banks.  The sums of a part take the place of the operands.
constexpr int kDirectChunk = 32 * 16 + 32, kDirectPiece = 4 * kDirectChunk;
constexpr int direct_lds_at(int operand, int piece, int P, int k4, int row)     // k4: k / 4
{
    return (operand * P + piece) * kDirectPiece + k4 / 2 * kDirectChunk + row * 16 + k4 % 2 * 8;
}
constexpr int direct_lds_bytes(int P, bool avec, bool bvec)
{
    const int staged = ((avec ? 1 : 0) + (bvec ? 1 : 0)) * P * kDirectPiece;
    return staged > 16 * 64 * 4 ? staged : 16 * 64 * 4;
}

// C = Q(A) Q(B)^T of two fp32 matrices in one launch, for products so small that the three launches of the general route
// (prepare, product, sum of the k parts: 5 - 6 us each on the GPU and 3 us each on the host) are what they cost.
// A wave owns a block of 32 x 32 results and one of `parts` ranges of k; it loads its operands, rounds and splits them in
// registers and multiplies: no barrier, four blocks of 32 k in flight meanwhile.  The parts of a block
// meet in LDS and are summed in order.  Every element is rounded once per block of its row or column instead of
// once, which is what bounds it (vector instructions: 0.6 us per block of 32 k and wave in 1/6/9, of it 0.1 the matrix cores) and why larger
// products keep the general route (direct_parts).  256 x 1024 x 1024 in 1/6/9 takes 9.5 - 10.0 us in a graph (rows along k
// loaded straight into the fragments' layout, and every XCD all of the larger operand: 11.1 - 12.7), 256 x 10 x 1024 8.5 (9.8),
// 128 x 512 x 512 in 1/8/7 8.0 (11.9; with the conversion in the vector units alone 8.9 -> 8.0).  The sums are those of the general route bit for bit when `parts` is its plan's: same pieces, same
// steps of 16 k, same order.
template <int MODE, bool FTZ, int PS, bool AVEC, bool BVEC>
__global__ __launch_bounds__(512) void direct_product_kernel(DirectOperand a, DirectOperand b, float *__restrict__ C, int64_t ldc,
                                                              int M, int N, int K, int kblocks, int tiles_m, int ntiles, int parts,
                                                              int kb_per, int tiles_per_wg, QuantParams p, LinearRound lin, int linear)
{
    constexpr int P = pieces_of(PS);
    extern __shared__ u32x4 s_mem[];             // a stretch per wave: its operands' pieces, then (parts > 1) its sums [16][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int kOwn = direct_lds_bytes(P, AVEC, BVEC);
    char *const own = reinterpret_cast<char *>(s_mem) + wave * kOwn;
    // Workgroups go to the XCDs in turn: every XCD gets a run of tiles, so that its L2 holds few of the larger operand's rows
    const int per_xcd = gridDim.x / 8, wg = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
    const int part = wave % parts, tile = wg * tiles_per_wg + wave / parts;
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
    // the whole wave plus a lane's offset.  Sixteen elements of an operand's 32 rows x 32 k to a lane:
    //   rows along k (VEC)   8 lanes take the 128 bytes of a row, four k each: rows 8 i + l / 8, i = 0 .. 3, k 4 (l % 8) + j at raw[4 i + j].  They
    //                        reach the fragments' layout through LDS, as pieces, in a stretch of the wave's own.  Loaded straight into
    //                        the fragments' layout, 32 rows to an instruction, a load touches 64 pieces of lines.
    //   rows side by side    the fragments' layout: row l % 32, k 16 kk + 8 (l / 32) + j at raw[8 kk + j]; 32 lanes take 128 bytes
    const int half = lane >> 5, part_row = lane >> 3, part_k = (lane & 7) * 4;
    uint32_t off_a[AVEC ? 4 : 1], off_b[BVEC ? 4 : 1];
    auto offsets = [&](auto vec, const DirectOperand &o, int first, auto &off) __attribute__((always_inline)) {
        if constexpr (decltype(vec)::value) {
#pragma unroll
            for (int i = 0; i < 4; ++i) off[i] = (uint32_t)min(first + 8 * i + part_row, o.rows - 1) * o.row_step;
        } else {
            off[0] = (uint32_t)min(first + (lane & 31), o.rows - 1) * o.row_step + (uint32_t)half * 8u * o.k_step;
        }
    };
    constexpr std::integral_constant<bool, AVEC> avec{};
    constexpr std::integral_constant<bool, BVEC> bvec{};
    offsets(avec, a, row0, off_a);
    offsets(bvec, b, col0, off_b);
    // no branch in here: the compiler keeps the loads of several blocks in flight
    auto load_one = [&](auto vec, const DirectOperand &o, const auto &off, int kb, uint32_t (&raw)[16]) __attribute__((always_inline)) {
        if constexpr (decltype(vec)::value) {
            const uint32_t *src = o.X + (uint32_t)(kb * kUnitK);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x4u w = *reinterpret_cast<const u32x4u *>(src + (off[i] + (uint32_t)part_k));
#pragma unroll
                for (int j = 0; j < 4; ++j) raw[4 * i + j] = w[j];
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const uint32_t *src = o.X + (size_t)(uint32_t)(kb * kUnitK + kk * 16) * o.k_step;
#pragma unroll
                for (int j = 0; j < 8; ++j, src += o.k_step) raw[8 * kk + j] = src[off[0]];
            }
        }
    };
    auto load = [&](int kb, uint32_t (&raw)[2][16]) __attribute__((always_inline)) {
        load_one(avec, a, off_a, kb, raw[0]);
        load_one(bvec, b, off_b, kb, raw[1]);
    };
    // The block that K ends in, zero beyond K.  A lane's four k that K cuts are loaded as the last four of the row and
    // moved down; single elements (and rows shorter than four) beyond K read the last k: no load waits behind a test of its own.
    auto load_last = [&](auto vec, const DirectOperand &o, const auto &off, int kb, uint32_t (&raw)[16]) __attribute__((always_inline)) {
        if constexpr (decltype(vec)::value) {
            const uint32_t at = (uint32_t)min(kb * kUnitK + part_k, K - 4);      // K >= 4 (launch)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x4u w = *reinterpret_cast<const u32x4u *>(o.X + (off[i] + at));
#pragma unroll
                for (int j = 0; j < 4; ++j) raw[4 * i + j] = w[j];
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = kb * kUnitK + kk * 16 + half * 8 + j;
                    raw[8 * kk + j] = o.X[off[0] - (uint32_t)half * 8u * o.k_step + (size_t)(uint32_t)min(k, K - 1) * o.k_step];
                }
        }
    };
    auto cut_last = [&](auto vec, int kb, uint32_t (&raw)[16]) __attribute__((always_inline)) {
        if constexpr (decltype(vec)::value) {
            const int k0 = kb * kUnitK + part_k, skip = k0 - min(k0, K - 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = (skip & 1) != 0 ? raw[4 * i + (j < 3 ? j + 1 : 3)] : raw[4 * i + j];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t moved = (skip & 2) != 0 ? v[j < 2 ? j + 2 : 3] : v[j];
                    raw[4 * i + j] = k0 + j < K ? moved : 0u;
                }
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < 8; ++j) raw[8 * kk + j] = kb * kUnitK + kk * 16 + half * 8 + j < K ? raw[8 * kk + j] : 0u;
        }
    };
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    // A lane's sixteen elements as pieces.  Elements near overflow or beyond go through the general conversion in a loop over
    // LDS: it stands in the code once per block of the ring, and code that runs but a few times per wave has to be short.
    auto convert = [&](const uint32_t (&raw)[16], u32x4 (&pc)[2][P]) __attribute__((always_inline)) {
        auto eights = [&](auto &&one) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                uint32_t v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = raw[8 * i + j];
                one(v, pc[i]);
            }
        };
        if constexpr (hardware_scheme(MODE, PS)) {
            if (hardware_format<MODE, PS>(p)) {
                eights([&](const uint32_t (&v)[8], u32x4 (&out)[P]) __attribute__((always_inline)) { hardware_convert<FTZ, PS>(v, p, out); });
                return;
            }
        }
        if (__ballot(run_is_rare(raw, p)) == 0ull) {
            eights([&](const uint32_t (&v)[8], u32x4 (&out)[P]) __attribute__((always_inline)) { short_convert<MODE, FTZ, PS>(v, p, masks, out); });
            return;
        }
        uint32_t *words = reinterpret_cast<uint32_t *>(own) + lane;
#pragma unroll
        for (int j = 0; j < 16; ++j) words[j * 64] = raw[j];
#pragma unroll 1
        for (int j = 0; j < 16; ++j) {
            uint32_t piece[P];
            round_and_split<MODE, FTZ, PS>(words[j * 64], p, piece);
            words[j * 64] = piece[0] | (P >= 2 ? piece[P >= 2 ? 1 : 0] << 16 : 0u);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t lo = words[(8 * i + 2 * j) * 64], hi = words[(8 * i + 2 * j + 1) * 64];
                pc[i][0][j] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                if constexpr (P >= 2) pc[i][P >= 2 ? 1 : 0][j] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
            }
    };
    auto multiply = [&](const uint32_t (&raw)[2][16]) __attribute__((always_inline)) {
        u32x4 f[2][2][P];                                            // [operand][16 k][piece]
        convert(raw[0], f[0]);
        convert(raw[1], f[1]);
        if constexpr (AVEC || BVEC) {
            // LDS takes a wave's accesses in order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            auto staged = [&](auto &&move) __attribute__((always_inline)) {
#pragma unroll
                for (int o = 0; o < 2; ++o)
                    if (o == 0 ? AVEC : BVEC) move(o, o == 1 && AVEC ? 1 : 0);
            };
            staged([&](int o, int place) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int q = 0; q < P; ++q)
                        *reinterpret_cast<u32x2 *>(own + direct_lds_at(place, q, P, lane & 7, 8 * i + part_row)) =
                            u32x2{f[o][i / 2][q][i % 2 * 2], f[o][i / 2][q][i % 2 * 2 + 1]};
            });
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            staged([&](int o, int place) __attribute__((always_inline)) {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int q = 0; q < P; ++q)
                        f[o][kk][q] = *reinterpret_cast<const u32x4 *>(own + direct_lds_at(place, q, P, 2 * (2 * kk + half), lane & 31));
            });
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
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
    const bool cut = kb0 <= whole && whole < kb1;                    // the block that K ends in is this part's
    uint32_t raw[kDepth][2][16], raw_cut[2][16];
    if (cut) {
        load_last(avec, a, off_a, whole, raw_cut[0]);
        load_last(bvec, b, off_b, whole, raw_cut[1]);
    }
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
    if (cut) {
        cut_last(avec, whole, raw_cut[0]);
        cut_last(bvec, whole, raw_cut[1]);
        multiply(raw_cut);
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
    for (int v = 0; v < 16; ++v) reinterpret_cast<float *>(own)[v * 64 + lane] = acc[v];
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
            for (int q = 0; q < parts; ++q)
                sum[c] += reinterpret_cast<const float *>(reinterpret_cast<const char *>(s_mem) + (w0 + q) * kOwn)[(4 * g + c) * 64 + lane];
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
    const bool avec = A.kcontig && K >= 4, bvec = B.kcontig && K >= 4;       // 16-byte vectors of a row
    const int per_wg = direct_blocks_per_workgroup(parts);
    const int waves = parts * per_wg;
    const size_t lds = (size_t)waves * direct_lds_bytes(pieces_of(PS), avec, bvec);
    const unsigned wgs = (unsigned)((tiles + per_wg - 1) / per_wg);
    auto kern = avec ? (bvec ? direct_product_kernel<MODE, FTZ, PS, true, true> : direct_product_kernel<MODE, FTZ, PS, true, false>)
                     : (bvec ? direct_product_kernel<MODE, FTZ, PS, false, true> : direct_product_kernel<MODE, FTZ, PS, false, false>);
    hipLaunchKernelGGL(kern, dim3((wgs + 7u) / 8u * 8u), dim3(64 * waves), lds, stream, operand(A, M), operand(B, N), C,
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
