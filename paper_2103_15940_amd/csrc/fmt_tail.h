// The products of the elements outside plane 0 (see fmt_gemm.hip): device code shared by the kernels that follow a product and the one
// that rounds a layer's outputs in the product itself.
#pragma once

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

// The block of C of row unit rb and the columns [col0, col0 + cols); 256 threads, col0 and cols multiples of 32.
__device__ __forceinline__ void planes_tail_body(const u32x4 *__restrict__ Aw, const u32x4 *__restrict__ Bw, const Planes &pa,
                                                 const Planes &pb, float *__restrict__ C, int64_t ldc, int M, int N, int kblocks,
                                                 int rb, int col0, int cols, TailLds &lds)
{
    uint32_t(&s_rec)[kTailRecs] = lds.rec;
    float(&s_val)[kTailRecs] = lds.val;
    uint32_t(&s_list)[256] = lds.list;
    int(&s_cnt)[4] = lds.cnt;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ub0 = col0 / kUnitRows;                // first unit of B of this block
    const int nub = min(cols / kUnitRows, (N + kRowPad - 1) / kRowPad * (kRowPad / kUnitRows) - ub0);   // B is padded to whole groups of 8 units

    // how many elements outside plane 0 A's row of units and B's rows of units hold (counted by the prepare pass)
    const uint32_t cnt_a = pa.rec_cnt[rb];
    const bool do_a = cnt_a != 0u;
    const bool do_b = __syncthreads_or(tid < nub && pb.rec_cnt[ub0 + tid] != 0u ? 1 : 0) != 0;
    if (!do_a && !do_b) return;

    // The records of a row of units whose count fits its list: read, and put into the order (k, row) -- the
    // prepare pass appends them in whatever order its workgroups run, and the additions below must not depend
    // on that.  One barrier before (the record arrays are free), one after.
    auto take_list = [&](const Planes &pl, size_t urow, int n) __attribute__((always_inline)) {
        uint32_t key = 0u, val = 0u;
        if (tid < n) {
            key = pl.recs[(urow * kRecCap + tid) * 2];
            val = pl.recs[(urow * kRecCap + tid) * 2 + 1];
            s_list[tid] = key;
        }
        __syncthreads();
        if (tid < n) {
            int rank = 0;
            for (int i = 0; i < n; ++i) rank += s_list[i] < key ? 1 : 0;
            s_rec[rank] = key;
            s_val[rank] = __uint_as_float(val);
        }
        __syncthreads();
    };

    // Ordered compaction over the workgroup: thread t contributes `have` items; returns the index of its
    // first one and, in total, the number of items.  Two barriers.
    auto place = [&](int have, int &total) __attribute__((always_inline)) {
        int incl = have;                                   // inclusive prefix inside the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        __syncthreads();                                   // s_cnt is free again
        if (lane == 63) s_cnt[wave] = incl;
        __syncthreads();
        int before = 0;
        total = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            before += q < wave ? s_cnt[q] : 0;
            total += s_cnt[q];
        }
        return before + incl - have;
    };

    // Walks the units of one row of units (mask row urow of operand W / pl, row scales S32) that have
    // other planes, k ascending, four units at a time: the two other planes of a unit are 256 vectors, one
    // per thread (threads 0..127 the plane above, vector tid: k-chunk tid / 32, row tid % 32; threads
    // 128..255 the plane below), all four units' loads are issued together, their non-zero elements become
    // records (row in the unit, k, TRUE value: the pattern with the plane's and the row's scale undone) in a
    // fixed order (thread, unit, position), and `apply(n)` uses up the n records of the group.
    auto walk = [&](const u32x4 *__restrict__ W, const Planes &pl, size_t urow, const int *S32, uint32_t first, bool have_first,
                    auto &&apply) {
        const int q = tid < kUnitVec ? 1 : 2, vec = tid & (kUnitVec - 1);
        const int r = vec & 31, c = vec >> 5;
        const int undo = -(S32[r] + (q == 1 ? -pl.w : pl.w));   // the plane above carries 2^(S - w), the one below 2^(S + w)
        for (int base = 0; base < kblocks; base += 256) {
            const int kb = base + tid;
            const uint32_t m = base == 0 && have_first ? first : (kb < kblocks ? (uint32_t)pl.mask[urow * kblocks + kb] & 6u : 0u);
            int total;
            const int at = place(m != 0u ? 1 : 0, total);
            if (m != 0u) s_list[at] = (uint32_t)tid | (m << 16);
            __syncthreads();
            for (int n0 = 0; n0 < total; n0 += 4) {
                u32x4 v[4];
                int kbn[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t e = n0 + u < total ? s_list[n0 + u] : 0u;
                    kbn[u] = base + (int)(e & 0xFFFFu);
                    v[u] = u32x4{0u, 0u, 0u, 0u};
                    if ((e >> (16 + q)) & 1u) v[u] = W[(size_t)q * pl.plane + (urow * kblocks + kbn[u]) * kUnitVec + vec];
                }
                // records of unit u (all four: u < 0) and plane qq (both: qq == 0) of this group, then their use
                auto emit = [&](int only_u, int only_q) {
                    const bool mine = only_q == 0 || only_q == q;
                    int cnt = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (mine && (only_u < 0 || only_u == u)) {
#pragma unroll
                            for (int t = 0; t < 8; ++t) cnt += (((t & 1) ? v[u][t >> 1] >> 16 : v[u][t >> 1]) & 0x7FFFu) != 0u ? 1 : 0;
                        }
                    int nrec;
                    int at2 = place(cnt, nrec);
                    if (nrec > kTailRecs) return nrec;       // workgroup-uniform: the caller splits the group
                    if (cnt) {
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (only_u < 0 || only_u == u) {
#pragma unroll
                                for (int t = 0; t < 8; ++t) {
                                    const uint32_t hp = ((t & 1) ? v[u][t >> 1] >> 16 : v[u][t >> 1]) & 0xFFFFu;
                                    if (hp & 0x7FFFu) {
                                        s_rec[at2] = (uint32_t)r | ((uint32_t)(kbn[u] * kUnitK + c * 8 + t) << 5);
                                        s_val[at2] = ldexpf(static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)hp)), undo);
                                        ++at2;
                                    }
                                }
                            }
                    }
                    __syncthreads();
                    apply(nrec);
                    __syncthreads();                         // the records are free again
                    return nrec;
                };
                if (emit(-1, 0) > kTailRecs) {               // rare: many elements outside plane 0 -- one plane of one unit at a time
                    for (int u = 0; u < 4; ++u)
                        for (int qq = 1; qq <= 2; ++qq) (void)emit(u, qq);
                }
            }
        }
    };

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
        if (cnt_a <= (uint32_t)kRecCap) {
            take_list(pa, (size_t)rb, (int)cnt_a);
            apply_a((int)cnt_a);
            __syncthreads();                                 // the records are free again
        } else {
            walk(Aw, pa, (size_t)rb, pa.S + rb * kUnitRows, 0u, false, apply_a);
        }
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
            if (cnt_b <= (uint32_t)kRecCap) {
                take_list(pb, (size_t)ub, (int)cnt_b);
                apply_b((int)cnt_b);
                __syncthreads();
            } else {
                walk(Bw, pb, (size_t)ub, pb.S + ub * kUnitRows, 0u, false, apply_b);
            }
        }
    }
}

}  // namespace fmt
