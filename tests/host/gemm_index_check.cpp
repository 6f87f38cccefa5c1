// Host check of the GEMM's operand addresses (gemm_index.hpp): plans products
// of many shapes and walks the loads that the planned kernel issues, thread
// by thread, for the first and last tiles, splits and K-tiles.  Every 16-byte
// load has to lie inside its operand, and every one that brings values the
// product uses has to be at the address of those values.  Built with g++; no
// device is used.
//
// With arguments M N K trans_a trans_b a_heads b_heads c_heads seq it prints
// that product's plan instead ("large" or "small" or "any", splits, K per split).
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>

#include "gemm_index.hpp"

using namespace elsaa::gemm;

namespace {

int g_fail = 0;
long g_loads = 0;

struct Operand {
    Mat m;
    int rows, cols;
    int64_t bytes;
};

Operand operand(int rows, int cols, int64_t ld, int heads, int seq)
{
    Operand o;
    o.m.p = nullptr;
    o.m.ld = ld;
    o.m.heads = heads;
    o.m.seq = seq;
    o.m.dh_shift = 0;
    if (heads > 0)
        while ((1 << o.m.dh_shift) < cols / heads) ++o.m.dh_shift;
    o.rows = rows;
    o.cols = cols;
    o.bytes = 2 * (heads > 0 ? (int64_t)rows * cols : (int64_t)(rows - 1) * ld + cols);
    return o;
}

elsaa_gemm_desc desc(int M, int N, int K, int ta, int tb, int ah, int bh, int ch, int seq)
{
    elsaa_gemm_desc d;
    std::memset(&d, 0, sizeof d);
    d.M = M; d.N = N; d.K = K; d.trans_a = ta; d.trans_b = tb;
    d.lda = ta ? M : K; d.ldb = tb ? K : N; d.ldc = N;
    d.a_heads = ah; d.b_heads = bh; d.c_heads = ch; d.seq = seq;
    d.c_dtype = ELSAA_BF16;
    return d;
}

void fail(const elsaa_gemm_desc& d, char op, const char* what, int64_t at, int64_t bytes)
{
    if (++g_fail <= 20)
        std::printf("FAIL %c of M %d N %d K %d ta %d tb %d heads %d/%d seq %d: %s (byte %lld of %lld)\n", op, d.M, d.N, d.K,
                    d.trans_a, d.trans_b, d.a_heads, d.b_heads, d.seq, what, (long long)at, (long long)bytes);
}

// The loads of one operand's K-tile at k0 with kn valid values of k (masked
// when `mask`), for the tile of rows (or columns) [x0, x0 + XT).
template <bool KMAJOR, int XT>
void check_tile(const elsaa_gemm_desc& d, char op, const Operand& o, int x0, int xlim, int k0, int kn, bool mask, bool used,
                bool any)
{
    using Ix = StreamIndex<KMAJOR, XT>;
    using Any = StreamIndexAny<KMAJOR>;
    for (int tx = 0; tx < kThreads; tx += tx < 64 || tx >= kThreads - 64 ? 1 : 7) {
        Ix ix;
        Any ax;
        if (any) ax.init(o.m, x0, xlim, tx);
        else ix.init(o.m, x0, xlim, tx);
        for (int c = 0; c < Ix::C; ++c) {
            const int k = any ? Any::k_in_tile(c, tx) : Ix::k_in_tile(c, tx);
            if (mask && k >= kn) continue;
            ++g_loads;
            if (!any && ix.off[c] > 0x7fffffffu - 15u) fail(d, op, "offset past the buffer range", ix.off[c], o.bytes);
            const int64_t at = any ? 2 * ax.at(o.m, k0, c, tx) : ix.base + Ix::tile(o.m, k0) + ix.off[c];
            if (at < 0 || at + 16 > o.bytes) fail(d, op, "load outside the operand", at, o.bytes);
            const int x = KMAJOR ? x0 + 8 * (tx % Ix::TPR) : x0 + tx / Ix::TPR + Ix::RPC * c;
            if (!used || x >= xlim) continue;
            const int64_t want = 2 * (KMAJOR ? mat_offset(o.m, k0 + k, x) : mat_offset(o.m, x, k0 + k));
            if (at != want) fail(d, op, "address of other values", at, want);
        }
    }
}

template <bool KMAJOR, int XT>
void check_operand(const elsaa_gemm_desc& d, char op, const Plan& p, const Operand& o, int xlim, int tiles)
{
    const std::set<int> xt = {0, tiles / 2, tiles - 1}, splits = {0, p.splits / 2, p.splits - 1};
    for (int sp : splits) {
        const KTiles kt(d.K, p.kper, sp);
        if (kt.n < 1 || kt.first < 1 || kt.first > BK) fail(d, op, "empty split", sp, p.splits);
        const std::set<int> steps = {1, 2, kt.n / 2, kt.n - 2, kt.n - 1, kt.n, kt.n + 1};
        for (int x : xt) {
            const int x0 = x * XT;
            check_tile<KMAJOR, XT>(d, op, o, x0, xlim, kt.kb, kt.first, true, true, p.any);
            // the large kernel loads tiles 1 .. n + 1, the small one 1 .. n - 1
            for (int t : steps)
                if (t >= 1 && (p.big || t < kt.n)) check_tile<KMAJOR, XT>(d, op, o, x0, xlim, kt.whole(t), BK, false, t < kt.n, p.any);
        }
        // the K-tiles cover the split: one short, then whole ones up to ke
        int k = kt.kb + kt.first;
        for (int t = 1; t < kt.n; ++t, k += BK)
            if (kt.whole(t) != k) fail(d, op, "K-tiles do not follow one another", kt.whole(t), k);
        if (k != kt.ke) fail(d, op, "K-tiles do not end at the split's end", k, kt.ke);
    }
}

template <bool KMAJOR>
void check_operand(const elsaa_gemm_desc& d, char op, const Plan& p, const Operand& o, int xlim, int tiles)
{
    if (p.big) check_operand<KMAJOR, kBig>(d, op, p, o, xlim, tiles);
    else check_operand<KMAJOR, BM>(d, op, p, o, xlim, tiles);
}

void check(const elsaa_gemm_desc& d)
{
    const Plan p = plan_of(&d);
    const Operand A = operand(d.trans_a ? d.K : d.M, d.trans_a ? d.M : d.K, d.lda, d.a_heads, d.seq);
    const Operand B = operand(d.trans_b ? d.N : d.K, d.trans_b ? d.K : d.N, d.ldb, d.b_heads, d.seq);
    if (d.trans_a) check_operand<true>(d, 'A', p, A, d.M, p.tiles_m);
    else check_operand<false>(d, 'A', p, A, d.M, p.tiles_m);
    if (d.trans_b) check_operand<false>(d, 'B', p, B, d.N, p.tiles_n);
    else check_operand<true>(d, 'B', p, B, d.N, p.tiles_n);
}

}  // namespace

int main(int argc, char** argv)
{
    if (argc == 10) {
        int v[9];
        for (int i = 0; i < 9; ++i) v[i] = std::atoi(argv[i + 1]);
        const elsaa_gemm_desc d = desc(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8]);
        const Plan p = plan_of(&d);
        std::printf("%s %d %d\n", p.big ? "large" : p.any ? "any" : "small", p.splits, p.kper);
        return 0;
    }
    // plain operands: short and ragged K on few and many tiles
    const int mn[][2] = {{8, 8}, {200, 136}, {256, 512}, {1016, 3080}, {1024, 1024}, {4096, 4096}, {2048, 6144}, {2840, 3080}};
    for (auto& s : mn)
        for (int K = 8; K <= 9216; K += K < 640 ? 8 : 328)
            for (int t = 0; t < 4; ++t) check(desc(s[0], s[1], K, t & 1, t >> 1, 0, 0, 0, 0));
    // the products of a block over a ragged number of tokens: one sequence of
    // n, whose dW products split a K of n, and several sequences
    for (int dm : {512, 768, 1024, 2048})
        for (int dh : {64, 128})
            for (int n = 1000; n <= 25000; n += n < 13400 || n > 15500 ? 776 : 8) {
                const int H = dm / dh;
                check(desc(n, 3 * dm, dm, 0, 0, 0, 0, 3 * H, n));          // QKV
                check(desc(n, dm, dm, 0, 0, H, 0, 0, n));                  // O W_O
                check(desc(n, dm, dm, 0, 1, 0, 0, H, n));                  // dY W_O'
                check(desc(dm, dm, n, 1, 0, H, 0, 0, n));                  // dW_O
                check(desc(n, dm, 3 * dm, 0, 1, 3 * H, 0, 0, n));          // dQKV W'
                check(desc(dm, 3 * dm, n, 1, 0, 0, 3 * H, 0, n));          // dW_QKV
            }
    for (int seq : {8, 64, 72, 192, 200, 320, 1000, 1024})
        for (int nseq : {2, 5, 9, 31})
            for (int dh : {32, 64, 128}) {
                const int n = seq * nseq, H = 1024 / dh, dm = 1024;
                check(desc(n, 3 * dm, dm, 0, 0, 0, 0, 3 * H, seq));
                check(desc(n, dm, dm, 0, 0, H, 0, 0, seq));
                check(desc(dm, dm, n, 1, 0, H, 0, 0, seq));
                check(desc(n, dm, 3 * dm, 0, 1, 3 * H, 0, 0, seq));
                check(desc(dm, 3 * dm, n, 1, 0, 0, 3 * H, 0, seq));
            }
    // operands of several GiB, up to the offsets' limits, and just past them
    for (int seq : {262144, 1048576, 2097152, 5592320, 5592448, 8388480, 8388736, 16777216})
        for (int nseq : {1, 3})
            for (int dh : {64, 128}) {
                const int64_t rows = (int64_t)seq * nseq;
                if (rows > 33000000) continue;
                const int n = (int)rows, H = 2048 / dh, dm = 2048;
                check(desc(n, dm, dm, 0, 0, H, 0, 0, seq));                // O W_O
                check(desc(dm, dm, n, 1, 0, H, 0, 0, seq));                // dW_O
                check(desc(n, dm, 3 * dm, 0, 1, 3 * H, 0, 0, seq));        // dQKV W'
                check(desc(dm, 3 * dm, n, 1, 0, 0, 3 * H, 0, seq));        // dW_QKV
            }
    for (int seq : {200, 1000, 100000, 524280, 2097160})                   // tiles that cross sequences
        for (int heads : {2, 16, 48}) check(desc(4 * seq, 1024, 64 * heads, 0, 1, heads, 0, 0, seq));
    std::printf("%ld loads\n", g_loads);
    std::printf(g_fail ? "%d FAILED\n" : "ALL OK\n", g_fail);
    return g_fail != 0;
}
