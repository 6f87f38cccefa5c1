// gemm_index.hpp -- which elements the GEMM kernels (gemm.hip) read and which
// kernel a product takes: operand addresses, the walk over K, and the plan.
// Plain arithmetic without device code, so a host program can walk every
// address of a plan (tests/host/gemm_index_check.cpp).
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "elsaa.h"

namespace elsaa {
namespace gemm {

constexpr int BM = 128, BN = 128, BK = 64;   // gemm_kernel's tile; both kernels' K-tile
constexpr int kBig = 256;                    // rows and columns of gemm_big_kernel's tile
constexpr int kThreads = 256;

#define ELSAA_HD __host__ __device__ __forceinline__

// One stored matrix: plain row-major (heads == 0) or head-major.
struct Mat {
    void* p;
    int64_t ld;
    int heads, seq, dh_shift;
};

ELSAA_HD int64_t mat_offset(const Mat& m, int r, int c)
{
    if (m.heads == 0) return (int64_t)r * m.ld + c;
    const int b = r / m.seq, n = r - b * m.seq;
    const int h = c >> m.dh_shift, e = c & ((1 << m.dh_shift) - 1);
    return ((((int64_t)b * m.heads + h) * m.seq + n) << m.dh_shift) + e;
}

// mat_offset as a row part plus a column part.
ELSAA_HD int64_t row_part(const Mat& m, int r)
{
    if (m.heads == 0) return (int64_t)r * m.ld;
    const int b = r / m.seq;
    return ((int64_t)r + (int64_t)b * (m.heads - 1) * m.seq) << m.dh_shift;
}
ELSAA_HD int64_t row_stride(const Mat& m) { return m.heads == 0 ? m.ld : ((int64_t)1 << m.dh_shift); }
ELSAA_HD int64_t col_part(const Mat& m, int c)
{
    if (m.heads == 0) return c;
    return (((int64_t)(c >> m.dh_shift) * m.seq) << m.dh_shift) + (c & ((1 << m.dh_shift) - 1));
}

ELSAA_HD int at_most(int x, int y) { return x < y ? x : y; }

// K-tiles of split sp: [kb, ke) as n tiles of 64 values of k, the first with
// `first` of them (read with a mask), the others whole and ending at ke.
struct KTiles {
    int kb, ke, n, first;
    ELSAA_HD KTiles(int K, int kper, int sp)
    {
        kb = sp * kper;
        ke = kb + at_most(K - kb, kper);
        n = (ke - kb + BK - 1) / BK;
        first = ke - kb - (n - 1) * BK;
    }
    // first k of tile t >= 1; past the end, and where the only tile is the
    // short one, the 64 values that end at ke, so a load without a mask stays
    // in the operand (ke >= 64: gemm_big_kernel, the only one to ask for such
    // tiles, takes no K below 64, and a split that ends before K is at least
    // 64 long)
    ELSAA_HD int whole(int t) const { return ke - (n - at_most(t, n - 1)) * BK; }
};

// Addresses of one operand's K-tiles, rows (or columns) [x0, x0 + XT).
// KMAJOR: the operand is stored [k][x] (x = m or n contiguous), thread tx
// loads k-rows tx / TPR + RPC c at columns x0 + 8 (tx % TPR); else [x][k],
// rows x0 + tx / 8 + 32 c at columns k0 + 8 (tx % 8).  x positions past xlim
// repeat the last ones.  The byte offsets from the tile's first element are
// formed once per thread (32 bits), which needs a K-tile's k-rows in one
// sequence (KMAJOR) or its columns in one head: fast_operand.
template <bool KMAJOR, int XT>
struct StreamIndex {
    static constexpr int C = XT * BK / 8 / kThreads;                    // 16-byte chunks per thread
    static constexpr int TPR = KMAJOR ? XT / 8 : 8, RPC = kThreads / TPR;
    int64_t base;        // byte offset of element (x0, 0) or (0, x0)
    uint32_t off[C];     // from there, or from the K-tile's first element
    ELSAA_HD void init(const Mat& m, int x0, int xlim, int tx)
    {
        const int r = tx / TPR, c8 = 8 * (tx % TPR);
        base = 2 * (KMAJOR ? col_part(m, x0) : row_part(m, x0));
        if (KMAJOR) {
#pragma unroll
            for (int c = 0; c < C; ++c)
                off[c] = (uint32_t)(((r + RPC * c) * row_stride(m) + col_part(m, at_most(x0 + c8, xlim - 8)) - col_part(m, x0)) * 2);
        } else if (m.heads == 0 || x0 / m.seq == (at_most(x0 + XT, xlim) - 1) / m.seq) {
            // rows of one sequence (uniform): equally spaced, without a
            // division for each (about 1 us of a workgroup's start)
#pragma unroll
            for (int c = 0; c < C; ++c)
                off[c] = (uint32_t)(((at_most(x0 + r + RPC * c, xlim - 1) - x0) * row_stride(m) + c8) * 2);
        } else {
#pragma unroll
            for (int c = 0; c < C; ++c)
                off[c] = (uint32_t)((row_part(m, at_most(x0 + r + RPC * c, xlim - 1)) - row_part(m, x0) + c8) * 2);
        }
    }
    // bytes from base to the first element of the K-tile at k0 (uniform)
    ELSAA_HD static int64_t tile(const Mat& m, int k0) { return 2 * (KMAJOR ? row_part(m, k0) : col_part(m, k0)); }
    // value of k, within its K-tile, at which chunk c of thread tx starts
    ELSAA_HD static int k_in_tile(int c, int tx) { return KMAJOR ? tx / TPR + RPC * c : 8 * (tx % TPR); }
};

// The same for 128-row tiles of operands that StreamIndex does not take: 64-bit
// offsets, and a K-tile's rows or columns each in a sequence or head of its
// own.  What does not depend on k is formed once per thread.
template <bool KMAJOR>
struct StreamIndexAny {
    static constexpr int C = BM * BK / 8 / kThreads;
    static constexpr int TPR = KMAJOR ? BM / 8 : 8, RPC = kThreads / TPR;
    int64_t fixed[KMAJOR ? 1 : C];   // elements
    ELSAA_HD void init(const Mat& m, int x0, int xlim, int tx)
    {
        if (KMAJOR) {
            fixed[0] = col_part(m, at_most(x0 + 8 * (tx % TPR), xlim - 8));
        } else {
#pragma unroll
            for (int c = 0; c < C; ++c) fixed[KMAJOR ? 0 : c] = row_part(m, at_most(x0 + tx / TPR + RPC * c, xlim - 1));
        }
    }
    // element offset of chunk c of the K-tile at k0
    ELSAA_HD int64_t at(const Mat& m, int k0, int c, int tx) const
    {
        const int k = k0 + k_in_tile(c, tx);
        return fixed[KMAJOR ? 0 : c] + (KMAJOR ? row_part(m, k) : col_part(m, k));
    }
    ELSAA_HD static int k_in_tile(int c, int tx) { return KMAJOR ? tx / TPR + RPC * c : 8 * (tx % TPR); }
};

#undef ELSAA_HD

struct Plan {
    bool big;                 // 256 x 256 tiles (gemm_big_kernel)
    bool any;                 // 128 x 128 tiles with StreamAny
    int tiles_m, tiles_n, splits, kper;
    size_t ws_bytes;
};

// Whether StreamIndex can address an operand stored as rows x cols: `kmajor`
// ones need every K-tile's 64 rows in one sequence (a single sequence, or
// whole 64-row pieces of several), the others its 64 columns in one head; the
// offsets from a tile's first element (tiles of up to 256 rows or columns
// start at a multiple of their size) must fit 31 bits.  A [x][k] tile spans
// further sequences only where several meet inside 256 rows, a [k][x] one the
// planes of 256 / dh heads (out of reach from 5.6 million tokens a sequence
// at dh 64 and 8.4 million at 128).
inline bool fast_operand(bool kmajor, int rows, int cols, int64_t ld, int heads, int seq)
{
    const int64_t lim = (int64_t)1 << 31;
    if (heads <= 0) return ld >= 0 && ld < lim / 512;
    if (seq < 1 || cols / heads < 8) return false;                     // (refused by check_mat)
    const int64_t dh = cols / heads, plane = (int64_t)seq * dh * 2;     // bytes of one head's rows
    if (kmajor) {
        const int64_t span = dh < kBig ? (kBig / dh - 1) * plane : 0;
        return (seq >= rows || seq % BK == 0) && span + (BK + 1) * dh * 2 + 2 * kBig < lim;
    }
    const int64_t crossings = seq >= rows || seq % kBig == 0 ? 0 : kBig / seq + 1;
    return dh % BK == 0 && crossings * (heads - 1) * plane + kBig * dh * 2 + 2 * BK < lim;
}

inline Plan plan_of(const elsaa_gemm_desc* d)
{
    Plan p;
    const int ar = d->trans_a ? d->K : d->M, ac = d->trans_a ? d->M : d->K;
    const int br = d->trans_b ? d->N : d->K, bc = d->trans_b ? d->K : d->N;
    p.any = !fast_operand(d->trans_a != 0, ar, ac, d->lda, d->a_heads, d->seq) ||
            !fast_operand(d->trans_b == 0, br, bc, d->ldb, d->b_heads, d->seq);
    // (64-bit counts: M, N and K may each be any int)
    auto parts = [](int64_t n, int64_t per) { return (n + per - 1) / per; };
    auto tiles_of = [&](int t) { return parts(d->M, t) * parts(d->N, t); };
    const int64_t ktiles = parts(d->K, BK);
    // Estimated microseconds of a tile size and split count.  A round is the
    // workgroups resident at once on 256 compute units (256 large tiles or
    // 512 small ones); measured per K-tile 1.55 us for a round of large
    // tiles (1040 - 1140 TFLOP/s at M 9000 .. 32768), 1.05 us for a full and
    // 0.8 of that for an at most half full round of small ones (870 TFLOP/s
    // at M 9000 x N 6144 x K 2048; one workgroup a compute unit at M 1000),
    // 1.25 where both operands are read transposed (dW: 670 TFLOP/s), about
    // 2.5 us for a round's first loads and last stores.  Splitting K costs
    // a launch and the partials' way to memory and back (6 TB/s: mostly the
    // memory-side cache).  The lines this
    // draws: M 9000, d_model 2048: QKV 219 us large against 272 small, dX
    // (288 large tiles, a second round of 32) 284 against 273; M 1000 small
    // throughout (16 - 22 us against 28 - 34).
    const double small_us = d->trans_a && !d->trans_b ? 1.25 : 1.05;
    auto estimate = [&](bool big, int splits) {
        const int fill = big ? 256 : 512;
        const int64_t per = parts(ktiles, splits);
        const int64_t wgs = tiles_of(big ? kBig : BM) * parts(ktiles, per), rem = wgs % fill;
        const double rounds = wgs / fill + (rem == 0 ? 0. : !big && 2 * rem <= fill ? 0.8 : 1.);
        const double reduce = splits > 1 ? 5. + 2e-6 * splits * (double)d->M * d->N * 4 / 6. : 0.;
        return rounds * (per * (big ? 1.55 : small_us) + 2.5) + reduce;
    };
    double best = 0.;
    // (the large kernel's unmasked loads need 64 values of k: KTiles::whole)
    for (int kind = 0; kind < (p.any || d->K < BK ? 1 : 2); ++kind) {
        const int64_t tiles = tiles_of(kind ? kBig : BM), fill = kind ? 256 : 512;
        // at least 8 K-tiles per split, at most one round of workgroups
        const int64_t most = tiles < fill ? std::max<int64_t>(1, std::min(fill / tiles, ktiles / 8)) : 1;
        for (int splits = 1; splits <= most; ++splits) {
            const double e = estimate(kind == 1, splits);
            if ((kind == 0 && splits == 1) || e < best) {
                best = e;
                p.big = kind == 1;
                p.splits = splits;
            }
        }
    }
    const int t = p.big ? kBig : BM;
    p.tiles_m = (int)parts(d->M, t);
    p.tiles_n = (int)parts(d->N, t);
    p.kper = (int)std::min<int64_t>(parts(ktiles, p.splits) * BK, INT_MAX - BK + 1);
    p.splits = (int)parts(d->K, p.kper);
    p.ws_bytes = p.splits > 1 ? (size_t)p.splits * d->M * d->N * sizeof(float) : 0;
    return p;
}

}  // namespace gemm
}  // namespace elsaa
