// The products of the elements outside plane 0 (see fmt_gemm.hip): device code shared by the kernels that follow a product and the one
// that rounds a layer's outputs in the product itself.
#pragma once

#include <type_traits>

#include "fmt_product.h"
#include "fmt_split.h"

namespace fmt {

// Half h (0..7) of a 16-byte vector of eight 16-bit patterns, as a float (binary16 -> fp32 is exact).
__device__ __forceinline__ float half_of(const u32x4 &v, int h)
{
    const uint32_t w = (h >> 1) == 0 ? v[0] : (h >> 1) == 1 ? v[1] : (h >> 1) == 2 ? v[2] : v[3];
    return static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)((h & 1) ? w >> 16 : w & 0xFFFFu)));
}

// Element (row r of the unit, k-chunk c, position h) of the unit whose plane-0 vectors start at W + unit_vec,
// in the scale of plane 0, whichever plane holds it: plane 0 as stored, the plane above times 2^w, the
// plane below times 2^-w (exact: a binary16 value times a power of two, far inside fp32's range).
__device__ __forceinline__ float unit_value(const u32x4 *__restrict__ W, size_t unit_vec, const Planes &pl, uint32_t planes,
                                            int c, int r, int h)
{
    const size_t at = unit_vec + (size_t)(c * kUnitRows + r);
    float x = half_of(W[at], h);
    if (planes & 6u) {                            // rare
        if (planes & 2u) x += ldexpf(half_of(W[pl.plane + at], h), pl.w);
        if (planes & 4u) x += ldexpf(half_of(W[2 * pl.plane + at], h), -pl.w);
    }
    return x;
}

// The products of the elements that live outside plane 0, added to C after the product kernel has stored
// plane 0 x plane 0.  Such elements are rare (a few per million for tensors of neural networks) and each
// contributes to one row or one column of C, so they are added one product at a time with fp32 fused
// multiply-adds on the TRUE values (the binary16 pattern with its plane's and its row's scale undone: a
// value of the format, exactly an fp32) -- exact product, one rounding per accumulation, FMACS.
// One workgroup owns a block of 32 rows (one unit of A) x tail_cols columns (8, 16 or 32 units of B) of C.
// Finding the elements of a row of units (masks, the other planes' vectors, the records) is a chain of dependent
// loads and barriers that costs more than using them, and every block of the same rows repeats it: wide blocks
// when the launch has blocks enough to fill the machine anyway, narrow ones otherwise (tail_cols_for).
//   1. every element a of A's other planes in its rows meets the FULL value of B (all planes) at that k
//      in each of its columns, elements in the order (k block, plane, position in the unit);
//   2. then every element b of B's other planes in its columns meets the plane-0 value of A in each of its
//      rows (an element of A outside plane 0 has met b in step 1), in the same kind of order.
// Every element of C has one owner and a fixed order of additions: the result is reproducible bit for bit.
// A block whose units hold nothing but plane 0 -- the usual case -- leaves after reading its masks.
constexpr int kTailRecs = kUnitRows * kUnitK;    // element records held at a time: one plane of one unit always fits

struct TailLds {
    uint32_t rec[kTailRecs];         // row-or-column in the unit (5 bits) | k << 5
    float val[kTailRecs];            // the element's true value
    uint32_t list[256];              // k blocks (of one scan of 256) whose unit has other planes | planes << 16
    int cnt[4];
};

// Records of the rows of units [unit0, unit0 + U) of an operand (count[]: how many each has) that fit their lists (kRecCap each), one row after the other in
// lds.rec and lds.val, each row's in the order (k, row): the prepare pass appends them in whatever order its workgroups run, and
// the additions must not depend on that.  256 threads, a wave per row of units; the record arrays are free before, and filled behind the
// last barrier.
template <int U>
__device__ __forceinline__ void tail_lists(const Planes &pl, size_t unit0, const uint32_t (&count)[U], TailLds &lds)
{
    static_assert(U <= 4 && kRecCap == 64, "a wave per list");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int n = 0, first = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int have = count[u] <= (uint32_t)kRecCap ? (int)count[u] : 0;
        first += u < wave ? have : 0;
        n = u == wave ? have : n;
    }
    uint32_t key = 0u, val = 0u;
    if (lane < n) {
        const uint32_t *rec = pl.recs + ((unit0 + wave) * kRecCap + lane) * 2;
        key = rec[0];
        val = rec[1];
        lds.list[wave * 64 + lane] = key;
    }
    __syncthreads();
    if (lane < n) {
        int rank = 0;
        for (int i = 0; i < n; ++i) rank += lds.list[wave * 64 + i] < key ? 1 : 0;
        lds.rec[first + rank] = key;
        lds.val[first + rank] = __uint_as_float(val);
    }
    __syncthreads();
}

// Where the walk through a row of units is.
struct TailWalk {
    int base = 0, total = -1;    // the blocks of k [base, base + 256): how many of them have other planes (-1: not looked at yet)
    int at = 0, part = 0;        // the group of four of these that comes next; of its parts (see tail_group) the next one
};

// The next records of row of units urow of operand W / pl (row scales S32) whose list does not hold them: walks the units that have
// other planes, k ascending, four units at a time.  The two other planes of a unit are 256 vectors, one per thread (threads 0..127
// the plane above, vector tid: k-chunk tid / 32, row tid % 32; threads 128..255 the plane below), all four units' loads are issued
// together, their non-zero elements become records (row in the unit, k, TRUE value: the pattern with the plane's and the
// row's scale undone) in lds.rec and lds.val, in a fixed order (thread, unit, position).  Returns how many (0: no more).  256
// threads; a barrier lies between the use of the records and the next call.
__device__ __forceinline__ int tail_group(const u32x4 *__restrict__ W, const Planes &pl, size_t urow, int kblocks, TailLds &lds, TailWalk &w)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Ordered compaction over the workgroup: thread t contributes `have` items; returns the index of its
    // first one and, in total, the number of items.  Two barriers.
    auto place = [&](int have, int &total) __attribute__((always_inline)) {
        int incl = have;                                   // inclusive prefix inside the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        __syncthreads();                                   // lds.cnt is free again
        if (lane == 63) lds.cnt[wave] = incl;
        __syncthreads();
        int before = 0;
        total = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            before += q < wave ? lds.cnt[q] : 0;
            total += lds.cnt[q];
        }
        total = __builtin_amdgcn_readfirstlane(total);
        return before + incl - have;
    };
    const int q = tid < kUnitVec ? 1 : 2, vec = tid & (kUnitVec - 1);
    const int r = vec & 31, c = vec >> 5;
    const int undo = -(pl.S[urow * kUnitRows + r] + (q == 1 ? -pl.w : pl.w));   // the plane above carries 2^(S - w), the one below 2^(S + w)
    for (;;) {
        if (w.total < 0) {
            if (w.base >= kblocks) return 0;
            const int kb = w.base + tid;
            const uint32_t m = kb < kblocks ? (uint32_t)pl.mask[urow * kblocks + kb] & 6u : 0u;
            const int at = place(m != 0u ? 1 : 0, w.total);
            if (m != 0u) lds.list[at] = (uint32_t)tid | (m << 16);
            __syncthreads();
            w.at = 0;
        }
        if (w.at >= w.total) {
            w.base += 256;
            w.total = -1;
            continue;
        }
        u32x4 v[4];
        int kbn[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t e = w.at + u < w.total ? lds.list[w.at + u] : 0u;
            kbn[u] = w.base + (int)(e & 0xFFFFu);
            v[u] = u32x4{0u, 0u, 0u, 0u};
            if ((e >> (16 + q)) & 1u) v[u] = W[(size_t)q * pl.plane + (urow * kblocks + kbn[u]) * kUnitVec + vec];
        }
        // part 0: the whole group; where that does not fit (rare: many elements outside plane 0), parts 1 to 8: one plane of one unit each
        const int only_u = w.part == 0 ? -1 : (w.part - 1) >> 1;
        const bool mine = w.part == 0 || 1 + ((w.part - 1) & 1) == q;
        int cnt = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (mine && (only_u < 0 || only_u == u)) {
#pragma unroll
                for (int t = 0; t < 8; ++t) cnt += (((t & 1) ? v[u][t >> 1] >> 16 : v[u][t >> 1]) & 0x7FFFu) != 0u ? 1 : 0;
            }
        int n;
        int to = place(cnt, n);
        if (n > kTailRecs) {                                 // the same in the workgroup
            w.part = 1;
            continue;
        }
        w.part = w.part == 0 || w.part == 8 ? 0 : w.part + 1;
        if (w.part == 0) w.at += 4;
        if (n == 0) continue;
        if (cnt) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (only_u < 0 || only_u == u) {
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const uint32_t hp = ((t & 1) ? v[u][t >> 1] >> 16 : v[u][t >> 1]) & 0xFFFFu;
                        if (hp & 0x7FFFu) {
                            lds.rec[to] = (uint32_t)r | ((uint32_t)(kbn[u] * kUnitK + c * 8 + t) << 5);
                            lds.val[to] = ldexpf(static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)hp)), undo);
                            ++to;
                        }
                    }
                }
        }
        __syncthreads();
        return n;
    }
}

// Hands the `count` (not zero) elements outside plane 0 of row of units urow to apply(n), n records at a time.
template <class APPLY>
__device__ __forceinline__ void tail_records(const u32x4 *__restrict__ W, const Planes &pl, size_t urow, int kblocks, uint32_t count,
                                             TailLds &lds, APPLY &&apply)
{
    if (count <= (uint32_t)kRecCap) {
        const uint32_t counts[1] = {count};
        tail_lists<1>(pl, urow, counts, lds);
        apply((int)count);
        __syncthreads();                                     // the records are free again
        return;
    }
    TailWalk w;
    for (;;) {
        const int n = tail_group(W, pl, urow, kblocks, lds, w);
        if (n == 0) return;
        apply(n);
        __syncthreads();
    }
}

// The block of C of row unit rb and the columns [col0, col0 + cols); 256 threads, col0 and cols multiples of 32.
__device__ __forceinline__ void planes_tail_body(const u32x4 *__restrict__ Aw, const u32x4 *__restrict__ Bw, const Planes &pa,
                                                 const Planes &pb, float *__restrict__ C, int64_t ldc, int M, int N, int kblocks,
                                                 int rb, int col0, int cols, TailLds &lds)
{
    uint32_t(&s_rec)[kTailRecs] = lds.rec;
    float(&s_val)[kTailRecs] = lds.val;
    const int tid = threadIdx.x;
    const int ub0 = col0 / kUnitRows;                // first unit of B of this block
    const int nub = min(cols / kUnitRows, (N + kRowPad - 1) / kRowPad * (kRowPad / kUnitRows) - ub0);   // B is padded to whole groups of 8 units

    // how many elements outside plane 0 A's row of units and B's rows of units hold (counted by the prepare pass)
    const uint32_t cnt_a = pa.rec_cnt[rb];
    const bool do_a = cnt_a != 0u;
    const bool do_b = __syncthreads_or(tid < nub && pb.rec_cnt[ub0 + tid] != 0u ? 1 : 0) != 0;
    if (!do_a && !do_b) return;

    if (do_a) {
        // 1. this block's columns of thread tid, one after the other: C[row][col] += a * b(k, col) for the
        //    records (row, k, a) in order
        auto apply_a = [&](int n) {
#pragma unroll 1
          for (int j = 0; j * 256 < cols; ++j) {
            const int col = col0 + j * 256 + tid;
            if (col >= min(N, col0 + cols)) return;
            const int ub = col / kUnitRows, cr = col % kUnitRows;
            const int sb = pb.S[col];
            // four records at a time: their loads (B's vector and mask, C) are issued together, then the
            // additions follow in record order; a row met earlier in the batch hands its sum on in registers
            for (int i0 = 0; i0 < n; i0 += 4) {
                int row[4], k[4];
                float a[4], c[4];
                u32x4 xv[4];
                uint32_t mk[4];
                size_t uv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool live = i0 + u < n;
                    const uint32_t rec = live ? s_rec[i0 + u] : 0u;
                    row[u] = rb * kUnitRows + (int)(rec & 31u);
                    k[u] = (int)(rec >> 5);
                    a[u] = live ? s_val[i0 + u] : 0.0f;
                    if (!live || row[u] >= M) row[u] = -1;
                    const size_t uidx = (size_t)ub * kblocks + k[u] / kUnitK;
                    uv[u] = uidx * kUnitVec;
                    mk[u] = 0u;
                    xv[u] = u32x4{0u, 0u, 0u, 0u};
                    c[u] = 0.0f;
                    if (row[u] >= 0) {
                        mk[u] = pb.mask[uidx];
                        xv[u] = Bw[uv[u] + (size_t)(((k[u] % kUnitK) / 8) * kUnitRows + cr)];
                        c[u] = C[(size_t)row[u] * ldc + col];
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (row[u] < 0) continue;
#pragma unroll
                    for (int v = 0; v < u; ++v)
                        if (row[v] == row[u]) c[u] = c[v];           // the latest sum of that row (v ascending)
                    float x = half_of(xv[u], k[u] % 8);
                    if (mk[u] & 6u) x = unit_value(Bw, uv[u], pb, mk[u], (k[u] % kUnitK) / 8, cr, k[u] % 8);
                    c[u] = __fmaf_rn(a[u], ldexpf(x, -sb), c[u]);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    bool last = row[u] >= 0;
#pragma unroll
                    for (int v = u + 1; v < 4; ++v) last = last && row[v] != row[u];
                    if (last) C[(size_t)row[u] * ldc + col] = c[u];
                }
            }
          }
        };
        tail_records(Aw, pa, (size_t)rb, kblocks, cnt_a, lds, apply_a);
    }
    if (do_b) {
        // 2. the rows of this block, one per lane of the first half-wave: C[row][col0] += a0(row, k) * b
        const int row = rb * kUnitRows + (tid & 31);
        const int sa = pa.S[rb * kUnitRows + (tid & 31)];
        for (int u = 0; u < nub; ++u) {
            const int ub = ub0 + u;
            if (ub * kUnitRows >= N) break;                  // workgroup-uniform
            const uint32_t cnt_b = pb.rec_cnt[ub];
            if (cnt_b == 0u) continue;                       // workgroup-uniform
            auto apply_b = [&](int n) {
                if (tid >= 32 || row >= M) return;
                for (int i = 0; i < n; ++i) {
                    const uint32_t rec = s_rec[i];
                    const int col = ub * kUnitRows + (int)(rec & 31u), k = (int)(rec >> 5);
                    if (col >= N) continue;
                    const size_t at = ((size_t)rb * kblocks + k / kUnitK) * kUnitVec + (size_t)(((k % kUnitK) / 8) * kUnitRows + (tid & 31));
                    const float a = ldexpf(half_of(Aw[at], k % 8), -sa);      // plane 0 only
                    float *dst = C + (size_t)row * ldc + col;
                    *dst = __fmaf_rn(a, s_val[i], *dst);
                }
            };
            tail_records(Bw, pb, (size_t)ub, kblocks, cnt_b, lds, apply_b);
        }
    }
}

// The same products for a workgroup's tile whose sums (scales undone) wait in LDS: the same additions to every element in the same
// order.  A thread owns the tile's elements of one column (A's records) or one row (B's) and of every second or fourth row or
// column, and takes eight records at a time, the loads of what they meet side by side.
// A function that is called, with the sums in LDS meanwhile: inlined beside the accumulators it takes the registers of the common case
// (128 x 128 with statistics: 800 spills; 4096 x 3072 x 1024 in 1/6/9 74 us instead of 49), and handed the accumulators it
// passes them through memory.  That layer with 0.05 / 1 % of X outside plane 0: 101 / 810 us; 210 / 1320 where they were added to
// sums in C, which were then rounded one by one; 82 / 490 with product, tail kernel and pass, which find the records of a row of
// units once per 256 columns and more, not once per 128.  Other tiles, 2048 x 2048 x 512: 36 / 190, 56 / 320, 41 / 130.
template <class T> using lds_ptr = __attribute__((address_space(3))) T *;

// A 64 TM x 64 TN tile of sums in LDS, R rows in each of up to four arrays; columns in groups of four, which move with the row so that
// a column's elements lie in 16 different groups of banks.
template <int TM, int TN, int R> struct TailTile {
    lds_ptr<float> s[4];
    __device__ __forceinline__ lds_ptr<float> at(int row, int col) const
    {
        const int i = row / R;
        const lds_ptr<float> base = i == 0 ? s[0] : i == 1 ? s[1] : i == 2 ? s[2] : s[3];
        return base + (row - i * R) * (64 * TN) + (col ^ ((row & 15) << 2));
    }
};

template <int TM, int TN, int R>
__device__ __attribute__((noinline)) void tail_tile(const u32x4 *__restrict__ Aw, const u32x4 *__restrict__ Bw, Planes pa, Planes pb, int kblocks,
                                                    int tm, int tn, TailTile<TM, TN, R> tile, lds_ptr<TailLds> ldsp)
{
    constexpr int UA = 2 * TM, UB = 2 * TN, kA = 64 * TM, kB = 64 * TN, kU = 8;
    TailLds &lds = *(TailLds *)ldsp;
    const int tid = threadIdx.x;
    uint32_t count_a[UA], count_b[UB];               // (read again: as arguments they cost the common case 1 us of 40)
#pragma unroll
    for (int u = 0; u < UA; ++u) count_a[u] = pa.rec_cnt[tm * UA + u];
#pragma unroll
    for (int u = 0; u < UB; ++u) count_b[u] = pb.rec_cnt[tn * UB + u];

    // apply(n, unit_of): n records in lds, unit_of(i) the row of units of the i-th; first those of all rows of units whose lists hold
    // them, then the others', one row after the other
    auto records = [&](const u32x4 *__restrict__ W, const Planes &pl, int unit0, const auto &count, auto &&apply) __attribute__((always_inline)) {
        constexpr int U = sizeof(count) / sizeof(count[0]);
        int first[U + 1];                            // of the listed records, the first of each row of units
        uint32_t many = 0u;                          // rows of units with more than their lists hold, a bit each
        first[0] = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool listed = count[u] <= (uint32_t)kRecCap;
            first[u + 1] = __builtin_amdgcn_readfirstlane(first[u] + (listed ? (int)count[u] : 0));
            many |= listed ? 0u : 1u << u;
        }
        many = (uint32_t)__builtin_amdgcn_readfirstlane((int)many);
#pragma unroll 1
        for (int turn = -1; turn < U; ++turn) {
            if (turn < 0 ? first[U] == 0 : ((many >> turn) & 1u) == 0u) continue;
            TailWalk w;
            for (;;) {
                int n = first[U];
                if (turn < 0) tail_lists(pl, (size_t)unit0, count, lds);
                else n = tail_group(W, pl, (size_t)(unit0 + turn), kblocks, lds, w);
                if (n == 0) break;
                apply(n, [&](int i) __attribute__((always_inline)) {
                    int unit = 0;
#pragma unroll
                    for (int u = 1; u < U; ++u) unit += i >= first[u] ? 1 : 0;
                    return turn < 0 ? unit : turn;
                });
                __syncthreads();                     // the records are free again
                if (turn < 0) break;
            }
        }
    };
    // pattern of the binary16 value of plane 0 at (row of the operand's rows from unit0, k)
    auto plane0 = [&](const u32x4 *__restrict__ W, size_t uidx, int row, int k) __attribute__((always_inline)) {
        return reinterpret_cast<const uint16_t *>(W + uidx * kUnitVec + (size_t)(k % kUnitK / 8 * kUnitRows + row % kUnitRows))[k % 8];
    };

    records(Aw, pa, tm * UA, count_a, [&](int n, auto &&unit_of) __attribute__((always_inline)) {
        constexpr int kParts = 256 / kB;
        const int col = tid % kB, part = tid / kB, sb = pb.S[tn * kB + col];
        const size_t unit = (size_t)(tn * UB + col / kUnitRows) * kblocks;
#pragma unroll 1
        for (int i0 = 0; i0 < n; i0 += kU) {
            uint32_t rec[kU], x[kU], mk[kU];
#pragma unroll
            for (int q = 0; q < kU; ++q) {
                rec[q] = lds.rec[min(i0 + q, n - 1)];
                x[q] = mk[q] = 0u;
                if ((int)(rec[q] % kParts) == part) {
                    const int k = (int)(rec[q] >> 5);
                    x[q] = plane0(Bw, unit + k / kUnitK, col, k);
                    mk[q] = pb.mask[unit + k / kUnitK];
                }
            }
#pragma unroll
            for (int q = 0; q < kU; ++q) {
                if (i0 + q >= n || (int)(rec[q] % kParts) != part) continue;
                const int k = (int)(rec[q] >> 5);
                float y = static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)x[q]));
                if (mk[q] & 6u) y = unit_value(Bw, (unit + k / kUnitK) * kUnitVec, pb, mk[q], k % kUnitK / 8, col % kUnitRows, k % 8);
                const lds_ptr<float> sum = tile.at(unit_of(i0 + q) * kUnitRows + (int)(rec[q] & 31u), col);
                *sum = __fmaf_rn(lds.val[i0 + q], ldexpf(y, -sb), *sum);
            }
        }
    });
    // an element of A outside plane 0 has met B's above: plane 0 only
    records(Bw, pb, tn * UB, count_b, [&](int n, auto &&unit_of) __attribute__((always_inline)) {
        constexpr int kParts = 256 / kA;
        const int row = tid % kA, part = tid / kA, sa = pa.S[tm * kA + row];
        const size_t unit = (size_t)(tm * UA + row / kUnitRows) * kblocks;
#pragma unroll 1
        for (int i0 = 0; i0 < n; i0 += kU) {
            uint32_t rec[kU], x[kU];
#pragma unroll
            for (int q = 0; q < kU; ++q) {
                rec[q] = lds.rec[min(i0 + q, n - 1)];
                const int k = (int)(rec[q] >> 5);
                x[q] = 0u;
                if ((int)(rec[q] % kParts) == part) x[q] = plane0(Aw, unit + k / kUnitK, row, k);
            }
#pragma unroll
            for (int q = 0; q < kU; ++q) {
                if (i0 + q >= n || (int)(rec[q] % kParts) != part) continue;
                const float y = ldexpf(static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)x[q])), -sa);
                const lds_ptr<float> sum = tile.at(row, unit_of(i0 + q) * kUnitRows + (int)(rec[q] & 31u));
                *sum = __fmaf_rn(y, lds.val[i0 + q], *sum);
            }
        }
    });
}

}  // namespace fmt
