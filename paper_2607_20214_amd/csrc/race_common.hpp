// race_common.hpp -- device helpers of the RACE low-rank kernels (forward and backward).
//
// Features (Alg. 2): for table l, u = W_l x (4 projections), t = tanh(u), and
// for bucket c of the hypercube {+-1}^4 (bit b of c set <-> v_cb = +1)
//   phi_c = exp(beta t.v_c) / sum_c' exp(beta t.v_c') = prod_b sigmoid(2 beta v_cb t_b).
// The projection kernel forms u = W x once per row and stores t = tanh(u)
// in float32 (every pass uses u only through t); chunks are 64 tokens; each
// workgroup is 4 waves,
// wave w handles tokens 16w .. 16w+15 of a chunk when computing features.
#pragma once
#include "common.hpp"
#include "tile.hpp"

namespace elsaa {
namespace race {

constexpr int kC = 64;
constexpr int kThreads = 256;
constexpr int kPad = 8;
constexpr size_t kMaxLds = 160 * 1024;

// The helpers take the thread index as an argument (default threadIdx.x): a
// kernel with several bodies passes each a copy that the compiler cannot
// share between them, so one body's lane addresses are not kept in registers
// through another.

// sigmoid(x) and sigmoid(-x) from one hardware exp and reciprocal: with
// e = exp(-|x|) in (0, 1], sigmoid(|x|) = 1 / (1 + e) and
// sigmoid(-|x|) = e / (1 + e), each within a few ulp and without overflow.
__device__ __forceinline__ void sigmoid_pair(float x, float& sp, float& sn)
{
    const float e = __expf(-fabsf(x));
    const float big = __builtin_amdgcn_rcpf(1.f + e), small = e * big;
    sp = x >= 0.f ? big : small;
    sn = x >= 0.f ? small : big;
}

// tanh(u) = 1 - 2 / (1 + e^{2u}), absolute error about 1e-7 (the features use
// t only through sigmoid(2 beta t) and the chain rule through 1 - t^2)
__device__ __forceinline__ float tanh_abs(float u)
{
    return 1.f - 2.f * __builtin_amdgcn_rcpf(1.f + __expf(2.f * u));
}

// A chunk's 64 rows of W elements in LDS, row-major, the rows in tile.hpp's
// slot order: 16-byte reads of 16 rows, transposed reads and 16-byte stores
// all hit distinct banks, so a chunk is staged once as whole rows and read
// in both orientations (no transposed copy: storing one took about 70 vector
// instructions and twelve 4-byte stores per 16 KB chunk and wave).
template <class T, int W>
struct RowTile {
    using S = typename T::store_t;
    using F = typename T::frag_t;
    static constexpr int LD = W + kPad, ELEMS = kC * LD;
    __device__ static __forceinline__ int row(int r) { return tile::slot_of(r) * LD; }
    // elements [e0, e0 + 8) of row r
    __device__ static __forceinline__ F row8(const S* t, int r, int e0) { return T::ld8(t + row(r) + e0); }
    // elements e0 .. e0 + 3 and e0 + 16 .. e0 + 19 of row r (the k order of
    // two accumulator tiles used as one operand)
    __device__ static __forceinline__ F row44(const S* t, int r, int e0)
    {
        const S* p = t + row(r) + e0;
        return T::ld44(p, p + 16);
    }
    // transposed operand: lane (i = lane % 16, g = lane / 16) receives column
    // c0 + i at rows kb + 8 g + j, j = 0..7
    __device__ static __forceinline__ F col8(const S* t, int kb, int c0, int tx = threadIdx.x)
    {
        const int lane = tx & 63, g = lane >> 4, i = lane & 15;
        const int r = kb + 8 * g;
        if constexpr (T::bytes == 2) {
            const bf16x4 lo = lds_read_tr4((const uint16_t*)(t + row(r + (i >> 2)) + c0 + 4 * (i & 3)));
            const bf16x4 hi = lds_read_tr4((const uint16_t*)(t + row(r + 4 + (i >> 2)) + c0 + 4 * (i & 3)));
            return F{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        } else {
            F f;
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = t[row(r + j) + c0 + i];
            return f;
        }
    }
};

// Sums over 32 of the chunk's tokens on the matrix cores: Phi^T x 1 (every
// entry of the B operand 1), so every lane of the product tile holds the
// sums of its rows' features: lane (g, col) register i += sum over tokens
// kb .. kb + 31 of phi_{f0 + 4g + i} (phit: the tile's col8 at feature f0).
template <class T>
__device__ __forceinline__ f32x4 token_sums(typename T::frag_t phit, f32x4 acc)
{
    float one[8] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
    return T::mma(phit, T::pack(one), acc);
}

// float32 values as matrix-core operands without loss: bf16 storage keeps
// v = p0 + p1 + p2, three bf16 parts (8 mantissa bits each), float32 storage
// keeps v itself.  Split once where the value is produced, then read as
// operand fragments (elements [e0, e0 + 8), the same for every column).
template <class T, int N>
struct Parts {
    using S = typename T::store_t;
    static constexpr int P = T::kSplit ? 3 : 1;
    S v[P][N];
    __device__ __forceinline__ void put(int i, float x)
    {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const S s = T::store(x);
            v[p][i] = s;
            x -= T::load(s);
        }
    }
    __device__ __forceinline__ f32x4 mma_b(typename T::frag_t a, int e0, f32x4 acc) const
    {
#pragma unroll
        for (int p = P - 1; p >= 0; --p) acc = T::mma(a, T::ld8(&v[p][e0]), acc);
        return acc;
    }
    __device__ __forceinline__ f32x4 mma_a(int e0, typename T::frag_t b, f32x4 acc) const
    {
#pragma unroll
        for (int p = P - 1; p >= 0; --p) acc = T::mma(T::ld8(&v[p][e0]), b, acc);
        return acc;
    }
};

// projection count padded to whole 32-wide k-steps (backward du x W)
template <int RP> constexpr int w_kdim() { return RP / 4 < 32 ? 32 : RP / 4; }

// Workgroups per sequence segment in the passes whose feature tables are
// independent (the state sums and the dQ / dK chain rules): each holds
// RP / split consecutive features (whole tables), reads the same chunk rows
// and writes its own state rows or du columns.  256 features split in two,
// so a workgroup's registers and LDS are those of the 128-feature passes.
template <int RP> constexpr int table_split() { return RP == 256 ? 2 : 1; }

// Waves of the passes that hold a segment's whole state (race_out, race_dv):
// each keeps the state's 16 * (D / 16 / waves) columns in registers.  At 256
// features four waves of D = 128 hold 128 state registers each and one wave
// fits a SIMD, so nothing covers its waits; eight hold 64 and two fit
// (8 heads x 65536: race_out 285 -> 239 us, race_dv 251 -> 217).  At 128
// features four waves already fit twice and eight are slower (16384 tokens x
// 16 heads: forward 450 against 465 us).
template <int D, int RP> constexpr int state_waves() { return RP == 256 && D == 128 ? 8 : 4; }

// Rows [t0, t0 + 64) of X (zero past N) into a RowTile, each multiplied by
// scale[row] * mul when SCALED.  load() issues every global load of the
// thread into registers (16 or 8 consecutive lanes cover a row) and store()
// writes them to LDS, so the loads fly while the chunk's features are formed.
// Rows past N are loaded clamped to row N - 1 and zeroed in store(), so the
// loads carry no per-lane branches and later waits count exactly.
// THREADS: threads that share the chunk (tx in [0, THREADS)).
template <class T, int D, bool SCALED, int THREADS = kThreads>
struct StageRows {
    using S = typename T::store_t;
    using Tl = RowTile<T, D>;
    static constexpr int PER = 16 / T::bytes;
    static constexpr int CH = D / PER;
    static constexpr int ITEMS = kC * CH, PT = ITEMS / THREADS;
    static_assert(ITEMS % THREADS == 0, "staging split");
    uint4 v[PT];
    float sc[SCALED ? PT : 1];
    int t0_, n_;
    __device__ __forceinline__ void load(const S* X, int t0, int N, const float* scale = nullptr, int tx = threadIdx.x)
    {
        t0_ = t0;
        n_ = N;
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int it = tx + j * THREADS;
            const int r = min(t0 + it / CH, N - 1);
            v[j] = ldg16(X + (size_t)r * D + (it % CH) * PER);
            if constexpr (SCALED) sc[j] = scale[r];
        }
    }
    __device__ __forceinline__ void store(S* t, float mul = 1.f, int tx = threadIdx.x)
    {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int it = tx + j * THREADS;
            const int r = it / CH;
            if (t0_ + r >= n_) v[j] = make_uint4(0, 0, 0, 0);
            S* dst = t + Tl::row(r) + (it % CH) * PER;
            if constexpr (SCALED) {
                const float f = sc[j] * mul;
                const S* e = (const S*)&v[j];
                float x[PER];
#pragma unroll
                for (int q = 0; q < PER; ++q) x[q] = T::load(e[q]) * f;
                if constexpr (T::bytes == 2) *(typename T::frag_t*)dst = T::pack(x);
                else *(f32x4*)dst = f32x4{x[0], x[1], x[2], x[3]};
            } else {
                *(uint4*)dst = v[j];
            }
        }
    }
};

// Projections t = tanh(u) of the tables this lane handles for chunk tokens
// [t0 + 16w, t0 + 16w + 16) (table tb = g + 4 m of token 16w + col), loaded
// ahead of features_from so that the next chunk's loads overlap this one.
template <int RP>
struct URegs {
    static constexpr int NU = (RP / 16 + 3) / 4;
    f32x4 u[NU];
    // Rows past N and tables past RP / 16 load clamped in-range values
    // (features_from zeroes those rows' features and skips those tables), so
    // the loads carry no per-lane branches.
    // stride: floats per projection row (RP / 4 unless this workgroup holds
    // only some of the row's tables, U then pointing at its first table)
    __device__ __forceinline__ void load(const float* U, int t0, int N, int stride = RP / 4, int tx = threadIdx.x)
    {
        const int lane = tx & 63, wv = tx >> 6;
        const int g = lane >> 4, col = lane & 15;
        const int tok = min(t0 + 16 * wv + col, N - 1);
#pragma unroll
        for (int m = 0; m < NU; ++m) {
            const int tb = min(g + 4 * m, RP / 16 - 1);
            u[m] = *(const f32x4*)(U + (size_t)tok * stride + 4 * tb);
        }
    }
};

// Features of chunk tokens [t0 + 16w, t0 + 16w + 16) for every table, from
// the projections t = tanh(u) in ur (URegs::load of the same chunk), into a
// feature RowTile (zero for padded tables, whose t is 0, and rows past N,
// which repeat row N - 1).  W: row width of
// that tile (RP, or more when ur holds some of the tables, ph then pointing
// at their first column).
template <class T, int RP, int W = RP>
__device__ __forceinline__ void features_from(const URegs<RP>& ur, int t0, int N, int L, float two_beta,
                                              typename T::store_t* ph, int tx = threadIdx.x)
{
    const int lane = tx & 63, wv = tx >> 6;
    const int g = lane >> 4, col = lane & 15;
    const int tl = 16 * wv + col;
#pragma unroll
    for (int m = 0; m < URegs<RP>::NU; ++m) {   // this lane: table tb of token tl
        const int tb = g + 4 * m;
        if (tb >= RP / 16) break;
        const f32x4 t = ur.u[m];                 // t = tanh(W x), formed by the projection pass
        const bool live = tb < L && t0 + tl < N;
        float sp[4], sn[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) sigmoid_pair(two_beta * t[i], sp[i], sn[i]);
        sp[3] = live ? sp[3] : 0.f;              // every product has one of these two factors
        sn[3] = live ? sn[3] : 0.f;
        float phi[16];
#pragma unroll
        for (int c = 0; c < 16; ++c)
            phi[c] = (((c & 1) ? sp[0] : sn[0]) * ((c & 2) ? sp[1] : sn[1])) *
                     (((c & 4) ? sp[2] : sn[2]) * ((c & 8) ? sp[3] : sn[3]));
        using F = typename T::frag_t;
        typename T::store_t* dst = ph + RowTile<T, W>::row(tl) + 16 * tb;
        *(F*)dst = T::pack(phi);
        *(F*)(dst + 8) = T::pack(phi + 8);
    }
}

// t = tanh(u) of the same tokens and tables into ts[token][4 * table + bit]
// (the chain rule's input).
template <int RP>
__device__ __forceinline__ void tanh_rows(const URegs<RP>& ur, float (*ts)[RP / 4], int tx = threadIdx.x)
{
    const int lane = tx & 63, wv = tx >> 6;
    const int g = lane >> 4, tl = 16 * wv + (lane & 15);
#pragma unroll
    for (int m = 0; m < URegs<RP>::NU; ++m)
        if (g + 4 * m < RP / 16) *(f32x4*)&ts[tl][4 * (g + 4 * m)] = ur.u[m];
}

// Chain rule from a transposed feature-gradient tile to the projection
// gradients du.  dphi: accumulator tile of the 16 features of table tb x 16
// rows (lane (g, col) register i holds feature c = 4g + i of row
// 16*qt + col).  phi_c = prod_b s_b(v_cb) with s_b(+1) = sigmoid(2 beta t_b),
// s_b(-1) = sigmoid(-2 beta t_b), so by the product rule
//   du_b = 2 beta s_b(1) s_b(-1) (1 - t_b^2) T_b,
//   T_b  = sum_c v_cb dphi_c prod_{b' != b} s_b'(v_cb').
// Bits 0, 1 of c are i, bits 2, 3 are g: each lane forms its four registers'
// share of the four T_b, and the four lane groups' shares are summed so that
// group b ends with T_b: two swaps of two different values give both halves
// of the sums at once (three exchanges in all).  Lane group g writes
// mul * du_b / (2 beta) into du[row][4 tb + g] (zero for padded tables).
template <class T, int RP>
__device__ __forceinline__ void chain_rule_t(f32x4 dphi, int qt, int tb, int L, float two_beta, float mul,
                                             const float (*ts)[RP / 4],
                                             typename T::store_t (*du)[w_kdim<RP>() + kPad], int tx = threadIdx.x)
{
    const int lane = tx & 63;
    const int g = lane >> 4, col = lane & 15;
    const int row = 16 * qt + col;
    // lane group g evaluates bit g's sigmoid pair; the groups then share them
    const float tg = ts[row][4 * tb + g];
    float spg, sng, sp[4], sn[4];
    sigmoid_pair(two_beta * tg, spg, sng);
    gather16x4(spg, sp);
    gather16x4(sng, sn);
    const float s2 = (g & 1) ? sp[2] : sn[2], s3 = (g & 2) ? sp[3] : sn[3];
    const float e0 = sn[0] * dphi[0] + sp[0] * dphi[1], e1 = sn[0] * dphi[2] + sp[0] * dphi[3];
    const float w = sn[1] * e0 + sp[1] * e1;       // sum over i without bits 2, 3
    const float hi = s2 * s3;
    const float a0 = hi * (sn[1] * (dphi[1] - dphi[0]) + sp[1] * (dphi[3] - dphi[2]));
    const float a1 = hi * (e1 - e0);
    const float a2 = ((g & 1) ? s3 : -s3) * w;
    const float a3 = ((g & 2) ? s2 : -s2) * w;
    // groups 0, 1 take the sums of a0 (group pairs), groups 2, 3 those of a2; a1, a3 alike
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a0), __float_as_uint(a2), false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(a1), __float_as_uint(a3), false, false);
    const float c0 = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    const float c1 = __uint_as_float(y[0]) + __uint_as_float(y[1]);
    const auto z = __builtin_amdgcn_permlane16_swap(__float_as_uint(c0), __float_as_uint(c1), false, false);
    const float tsum = __uint_as_float(z[0]) + __uint_as_float(z[1]);
    const float v = mul * (spg * sng) * (1.f - tg * tg) * tsum;
    du[row][4 * tb + g] = T::store(tb < L ? v : 0.f);
}

// One element of the segment states (base: its address in segment 0, per
// elements apart): mode 0: the total in every segment; 1: exclusive prefix; 2:
// exclusive suffix.  The segments are walked in batches of independent loads.
__device__ __forceinline__ void scan_states(float* base, int nseg, int per, int mode)
{
    constexpr int kBatch = 16;
    float run = 0.f;
    for (int s0 = 0; s0 < nseg; s0 += kBatch) {
        float v[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int s = mode == 2 ? nseg - 1 - (s0 + j) : s0 + j;
            v[j] = (s0 + j < nseg) ? base[(size_t)s * per] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (s0 + j >= nseg) break;
            const int s = mode == 2 ? nseg - 1 - (s0 + j) : s0 + j;
            if (mode != 0) base[(size_t)s * per] = run;
            run += v[j];
        }
    }
    if (mode == 0)
        for (int s = 0; s < nseg; ++s) base[(size_t)s * per] = run;
}

}  // namespace race
}  // namespace elsaa
