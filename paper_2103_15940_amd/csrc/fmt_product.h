// The product kernels' interface: what fmt_gemm.hip hands to the translation units that hold them (fmt_product_<scheme>.hip, one
// per piece scheme, so that they compile side by side).
#pragma once

#include "fmt_internal.h"
#include "fmt_split.h"

#ifndef FMT_GEMM_KS
#define FMT_GEMM_KS 2      // 16-k steps per LDS stage
#endif
#ifndef FMT_GEMM_KS_MULTI
#define FMT_GEMM_KS_MULTI 1  // ... with two or three pieces per operand (twice / three times the bytes per k)
#endif
#ifndef FMT_GEMM_NST
#define FMT_GEMM_NST 4     // LDS stage buffers (at most; see pipe_nst)
#endif

namespace fmt {

// Exponent planes of one prepared operand (formats with e == 6 and m <= 9; see the top of this file).
//   S      scale exponent per (padded) row: plane 0 holds value * 2^S, the plane above value * 2^(S-w),
//          the plane below value * 2^(S+w), each as a binary16 value
//   mask   one byte per unit (32 rows x 32 k): bit 0 set always, bit 1 / bit 2 set when the unit has
//          an element in the plane above / below; only then has that plane's unit been written
//   plane  16-byte vectors from one plane's pieces to the next (planes 1 and 2 follow plane 0)
//   recs   per row of units (32 rows x all k), the elements outside plane 0 as records (k << 5 | row in the unit,
//          true value as fp32 bits), in no particular order, and rec_cnt how many there are; a row of units
//          with more than kRecCap of them keeps only the count (its elements are then found through the masks)
struct Planes {
    int *S;
    uint8_t *mask;
    size_t plane;
    int w;               // 40 - m: binades one plane holds
    uint32_t *rec_cnt;
    uint32_t *recs;      // pairs of words, kRecCap pairs per row of units
};
constexpr int kRecCap = 64;
// Convolutions (product_window) use planes with one scale for the whole tensor: S[0] alone, no records.  A tensor whose patches the
// product kernel gathers has, per 64 pixels x 32 channels, two words of 64 bits in the mask's place, a bit per pixel: what has elements in the plane
// above, and below.  S[1] of operand A is 1 where both operands are two bf16 pieces instead (window_pair).

// Division of a 31-bit dividend by a divisor fixed at launch, as a multiply-high and a shift
// (m = floor(2^(31+l) / d) + 1 with l = ceil(log2 d) gives floor(a / d) for every 0 <= a < 2^31).
struct FastDiv {
    uint32_t m;
    int sh;      // l - 1; d == 1 is handled apart
    int d;
};

inline FastDiv make_fastdiv(int d)
{
    FastDiv f{0u, 0, d < 1 ? 1 : d};
    if (f.d > 1) {
        int l = 0;
        while (((int64_t)1 << l) < f.d) ++l;
        f.m = (uint32_t)((((uint64_t)1 << (31 + l)) / (uint64_t)f.d) + 1);
        f.sh = l - 1;
    }
    return f;
}

__device__ __forceinline__ void divmod(const FastDiv &f, int a, int &q, int &r)
{
    q = f.d == 1 ? a : (int)(__umulhi((uint32_t)a, f.m) >> f.sh);
    r = a - q * f.d;
}

// Division by twice the divisor (make_fastdiv(2 d): the same m, l one more).
__device__ __forceinline__ FastDiv fastdiv_twice(const FastDiv &f)
{
    return f.d == 1 ? FastDiv{0x80000001u, 0, 2} : FastDiv{f.m, f.sh + 1, 2 * f.d};
}

// Operand B of a convolution product gathered by the product kernel itself: row = position (n, y, x)
// on a grid gy x gx, k = (tap, channel) with the channel running fastest, read from the rounded tensor
// in pixel-major order T[piece][n][iy][ix][channel] (16-bit pieces, 8 channels per 16-byte vector; tc is a
// multiple of 32, so a stage of 16 or 32 k lies inside one tap).  iy = y*mul_y + off_y + tap_sign*r, likewise
// ix; a tap outside the tensor reads the zero vector at index `zero`.  Every index counts 16-byte vectors
// from T and fits 31 bits.
struct Implicit {
    const u32x4 *T;
    int piece_vec;      // vectors per piece
    int zero;           // index of a vector of zeros
    int c8;             // channels / 8
    int th, tw, gy, gx;
    int mul_y, mul_x, off_y, off_x, tap_sign;
    int R, S;
    int rows;
    FastDiv r0, r1;     // row -> (n, y, x): by gx, then by gy
    FastDiv kc;         // stage number -> (tap, channel block): by channels / (k per stage)
    FastDiv ks;         // tap -> (r, s): by S
};

// A group of independent products in one launch (fmt_gemm_prepared_batch): workgroup ids [first, next first)
// belong to product g, each product's run of ids is a multiple of 8 long (so that id % 8, the XCD, means the
// same inside every run), and every product runs the same kernel variant -- no k split, plain row-major output.
// One launch instead of one per product: launch, pipeline fill and drain -- about a third of the time of a
// product with K = 1024 -- are paid once, and the tiles of the next product fill the compute units that the
// last tiles of the previous one leave idle.
constexpr int kMaxGroup = 16;
struct GroupItem {
    const u32x4 *Aw, *Bw;
    float *C;               // the result, or (k in parts) the first of the parts' dense M x N slabs (then ldc = N)
    int64_t ldc;
    int M, N, kblocks, tiles_m, tiles_n;
    int kb_per_part;        // k blocks per part (= kblocks: one part); the product's run of ids holds one run of tiles per part
    unsigned first;
    Planes pa, pb;
};
struct Group {
    int count;
    unsigned first[kMaxGroup];     // p[i].first again, side by side (one scalar load), 0xFFFFFFFF beyond count
    GroupItem p[kMaxGroup];
};

// Which product a workgroup id belongs to: the number of runs that start at or before it, minus one.
__device__ __forceinline__ int group_member(const unsigned (&first)[kMaxGroup], unsigned id)
{
    int g = -1;
#pragma unroll
    for (int i = 0; i < kMaxGroup; ++i) g += id >= first[i] ? 1 : 0;
    return g;
}

struct Plan {
    int tm, tn;      // wave tile in MFMA tiles; workgroup tile = 64*tm x 64*tn
    int nsplit;      // k parts
    int sched;       // 1: pin the issue order inside a trip (sched_group_barrier), 0: leave it to the compiler
    int cus = 256;   // compute units it was made for
    bool forced = false;     // by FMT_GEMM_PLAN
};

constexpr size_t lds_bytes(int tm, int tn, int pieces, int ks, int nst)
{
    return (size_t)nst * (2 * tm + 2 * tn) * pieces * 64 * ks * sizeof(u32x4);
}

// Pipeline shape per piece scheme and tile shape: k16 steps per stage, and as many stage buffers (at
// most FMT_GEMM_NST, at least two) as fit the tile's share of the 160 KiB of LDS -- all of it for the
// large tiles, half for 128 x 128 (two resident workgroups), a third for 128 x 64, a quarter for 64 x 64.
constexpr int pipe_ks(int pieces) { return pieces == 1 ? FMT_GEMM_KS : FMT_GEMM_KS_MULTI; }
constexpr int pipe_nst(int tm, int tn, int pieces, int ks)
{
    if ((tm * pieces * ks) % 2 || (tn * pieces * ks) % 2) return 2;   // stage not a whole number of loads per wave
    const size_t budget = (size_t)160 * 1024 / (tm * tn > 4 ? 1 : tm * tn == 4 ? 2 : tm * tn == 2 ? 3 : 4);
    int n = FMT_GEMM_NST;
    while (n > 2 && lds_bytes(tm, tn, pieces, ks, n) > budget) --n;
    return n;
}
template <int PS, int TM, int TN> struct Pipe {
    static constexpr int ks = pipe_ks(pieces_of(PS)), nst = pipe_nst(TM, TN, pieces_of(PS), ks);
};


// A prepared operand in memory at `base`.
struct OperandView {
    u32x4 *W;
    Planes pl;
};

// Where the M x N result goes: plain row-major with leading dimension ldc, or (img > 0) NCHW with
// columns = (image, position) and `img` positions per image.
// lin != nullptr: the results are the accumulators of a fully connected layer, and a route that can round them on the way
// out does so and says so in *rounded.
struct OutSpec {
    float *C;
    int64_t ldc;
    int img;
    const LinearOut *lin = nullptr;
    bool *rounded = nullptr;
};


// fmt_gemm.hip
int launch_reduce(const float *part, int nsplit, float *C, int M, int N, int64_t ldc, int img, hipStream_t stream);
int launch_planes_tail(const u32x4 *Aw, const u32x4 *Bw, const Planes &pa, const Planes &pb, float *C, int64_t ldc, int M, int N,
                       int kblocks, hipStream_t stream);

// fmt_product_<PS>.hip (fmt_product_kernels.h)
template <int PS>
int product_of_views(const OperandView &va, const OperandView &vb, int M, int N, int kblocks, const OutSpec &out, const Plan &plan,
                     float *part, hipStream_t stream);
template <int PS>
int product_gathered(const OperandView &va, const Implicit &im, int M, int N, int kblocks, const OutSpec &out, const Plan &plan,
                     float *part, hipStream_t stream);
// fmt_product_window.hip
template <bool GATHER>
int product_window(const OperandView &va, const OperandView &vb, const Implicit &im, int M, int N, int kblocks, const OutSpec &out,
                   const Plan &plan, float *part, hipStream_t stream);
template <int PS, bool SCALED>
int launch_group(const Group &grp, unsigned grid, int t, hipStream_t stream);

}  // namespace fmt
