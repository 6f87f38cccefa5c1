// race_fwd.hip -- RACE low-rank branch forward (Alg. 2; causal chunked form Alg. 3),
// and the segment-state kernels the backward reuses.
//
// Num = (1/L) sum_l Phi_Q^l B^l, Den = (1/L) sum_l Phi_Q^l A^l with
// A^l = Phi_K^l' 1, B^l = Phi_K^l' V; the causal form restricts both sums to
// keys j <= i.  O_lr = Num / (Den + eps), d_lr = Den.
//
// Features come from t = tanh(W x), stored by the projection kernel.
// The sequence of each (b,h) is cut into segments of whole 64-token chunks:
//   state  one workgroup per segment: S = sum_j phi(x_j) v_j' (r x d) and
//          A = sum_j a_j phi(x_j) over the segment (forward: x = k, v = V,
//          a = 1; the backward reuses it with x = q, v = dNum, a = dDen);
//   scan   per (b,h): exclusive prefix (causal forward), exclusive suffix
//          (causal backward) or the total in every segment (non-causal);
//   out    one workgroup per segment: starting from its prefix state, each
//          chunk computes Num = (1/L) Phi_Q S + tril(Phi_Q Phi_K'/L) V (the
//          masked part only when causal), then adds the chunk to S.
// Each of the 4 waves owns d/4 columns of S, held as float32 matrix-core
// accumulators for the whole segment; the intra-chunk kernel matrix and every
// contraction run on MFMA (bf16 or float32 operands, float32 accumulation).
#include <type_traits>

#include "bwd_rows.hpp"
#include "internal.hpp"
#include "race_common.hpp"

namespace elsaa {

using namespace race;

namespace {

template <class T, int D, int RP>
struct StateSmem {
    using S = typename T::store_t;
    S v[RowTile<T, D>::ELEMS];    // value rows
    S ph[RowTile<T, RP>::ELEMS];  // feature rows
    Parts<T, kC> aw;              // weights of A (backward)
};

template <class T, int D, int RP>
struct OutSmem {
    using S = typename T::store_t;
    S v[RowTile<T, D>::ELEMS];    // V chunk
    S phq[RowTile<T, RP>::ELEMS]; // Phi_Q chunk
    S phk[RowTile<T, RP>::ELEMS]; // Phi_K chunk
    S mm[kC][kC + kPad];          // tril(Phi_Q Phi_K') / L
    Parts<T, RP> a_state;
    float den[state_waves<D, RP>() / 4][kC];  // parts of Den
};

struct StateArgs {
    const float* U;       // projections of the feature rows [BH][N][RP/4]
    const void* Val;      // value rows [BH][N][D]
    const float* vscale;  // per-row value scale [BH][N] (backward; else null)
    const float* aw;      // per-row weight of A [BH][N] (backward; else null: 1)
    float* states;        // [BH][nseg][RP*D + RP]
    int H, N, L, seg_len, nseg;
    float two_beta, mul;
    RowArgs rows;         // kStateRows
};

// What a state pass sums: the forward's key rows, the backward's query rows
// with given scalars (vscale, aw), or the same with the rows' scalars formed on
// the way from dO (Val), O_s and O_lr and written out.
enum StateKind { kStateFwd = 0, kStateBwd = 1, kStateRows = 2 };

// A chunk's rows of dO, O_s and O_lr and the row inputs of the scalars: loads
// one chunk ahead (as StageRows), then the two dot products per row (CH lanes
// cover a row), the row's scalars, and sc_lr dO into the value tile.
template <class T, int D>
struct StageDots {
    using S = typename T::store_t;
    static constexpr int PER = 16 / T::bytes, CH = D / PER, PT = kC * CH / kThreads;
    static_assert(CH == 8 || CH == 16, "lanes per row");
    uint4 u[PT], ol[PT];
    f32x4 os[PT][PER / 4];
    RowIn in[PT];
    __device__ __forceinline__ void load(const S* dO, const RowArgs& r, size_t bh, int t0, int N)
    {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int it = threadIdx.x + j * kThreads;
            const size_t row = bh * N + min(t0 + it / CH, N - 1);
            const size_t at = row * D + (it % CH) * PER;
            u[j] = ldg16(dO + at);
            ol[j] = ldg16((const S*)r.Olr + at);
#pragma unroll
            for (int e = 0; e < PER / 4; ++e) os[j][e] = *(const f32x4*)(r.Os + at + 4 * e);
            in[j].load(r, row);
        }
    }
    __device__ static __forceinline__ float dpp(float v, const int ctrl_sel)
    {
        const uint32_t x = __float_as_uint(v);
        const uint32_t y = ctrl_sel == 0   ? __builtin_amdgcn_mov_dpp(x, 0xb1, 0xf, 0xf, true)     // lane ^ 1
                           : ctrl_sel == 1 ? __builtin_amdgcn_mov_dpp(x, 0x4e, 0xf, 0xf, true)     // lane ^ 2
                           : ctrl_sel == 2 ? __builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true)    // the row half mirrored
                                           : __builtin_amdgcn_mov_dpp(x, 0x140, 0xf, 0xf, true);   // the row mirrored
        return v + __uint_as_float(y);
    }
    // sum over the CH consecutive lanes of a row, in each of them
    __device__ static __forceinline__ float lanes_sum(float v)
    {
        v = dpp(dpp(dpp(v, 0), 1), 2);
        if constexpr (CH == 16) v = dpp(v, 3);
        return v;
    }
    __device__ __forceinline__ void store(const RowArgs& r, size_t bh, int t0, int N, S* t, Parts<T, kC>& aw) const
    {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int it = threadIdx.x + j * kThreads, rl = it / CH, e0 = (it % CH) * PER;
            const bool live = t0 + rl < N;
            const S* ue = (const S*)&u[j];
            const S* le = (const S*)&ol[j];
            float x[PER], uos = 0.f, uol = 0.f;
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                x[e] = T::load(ue[e]);
                uos += x[e] * os[j][e / 4][e % 4];
                uol += x[e] * T::load(le[e]);
            }
            uos = lanes_sum(uos);
            uol = lanes_sum(uol);
            const float f = live ? in[j].gl * (1.f / (in[j].den + r.eps)) : 0.f;
#pragma unroll
            for (int e = 0; e < PER; ++e) x[e] *= f;
            S* dst = t + RowTile<T, D>::row(rl) + e0;
            if constexpr (T::bytes == 2) *(typename T::frag_t*)dst = T::pack(x);
            else *(f32x4*)dst = f32x4{x[0], x[1], x[2], x[3]};
            if (e0 == 0) {
                float dden = 0.f;
                if (live) dden = row_scalars(r, bh * N + t0 + rl, in[j], uos, uol);
                aw.put(rl, dden);
            }
        }
    }
};

template <class T, int D, int RP, int KIND>
__global__ __launch_bounds__(kThreads, KIND == kStateRows && T::bytes == 2 ? 2 : 1) void race_state_kernel(StateArgs a)
{
    constexpr bool BWD = KIND != kStateFwd, ROWS = KIND == kStateRows;   // A is weighted; scalars formed here
    static_assert(!ROWS || table_split<RP>() == 1, "one workgroup per row");
    using St = typename T::store_t;
    using F = typename T::frag_t;
    constexpr int DW = D / 64;
    constexpr int SPLIT = table_split<RP>(), RPW = RP / SPLIT;   // features of this workgroup
    constexpr int FT = RPW / 16, NFA = (FT + 3) / 4;
    using TV = RowTile<T, D>;
    using TP = RowTile<T, RPW>;
    __shared__ __attribute__((aligned(16))) StateSmem<T, D, RPW> sm;
    const int seg = blockIdx.x / SPLIT, part = blockIdx.x % SPLIT, h = blockIdx.y, b = blockIdx.z;
    const int F0 = part * RPW, L = a.L - F0 / 16;                  // first feature; tables from here on
    const size_t bh = (size_t)b * a.H + h;
    const float* U = a.U + bh * a.N * (RP / 4) + F0 / 4;
    const St* Vl = (const St*)a.Val + bh * a.N * D;
    const float* vs = KIND == kStateBwd ? a.vscale + bh * a.N : nullptr;
    const float* aw = KIND == kStateBwd ? a.aw + bh * a.N : nullptr;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int g = lane >> 4, col = lane & 15;

    f32x4 S[FT][DW];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int j = 0; j < DW; ++j) S[ft][j] = f32x4{0, 0, 0, 0};
    // A of the feature tiles ft = w, w + 4, ...: bf16 on the matrix cores
    // (every column alike), float32 in the vector units (lane (g, col): feature
    // 16 ft + col over the tokens of lane group g, Aacc[j][0]; a float32 product
    // takes eight matrix instructions of 32 cycles)
    f32x4 Aacc[NFA];
#pragma unroll
    for (int j = 0; j < NFA; ++j) Aacc[j] = f32x4{0, 0, 0, 0};

    const int t_beg = seg * a.seg_len, t_end = min(a.N, t_beg + a.seg_len);
    // projections, value rows and A weights of the chunk, loaded one chunk ahead
    URegs<RPW> ur;
    typename std::conditional<ROWS, StageDots<T, D>, StageRows<T, D, KIND == kStateBwd>>::type vr;
    float awv = 0.f;
    auto load_chunk = [&](int c0) {
        ur.load(U, c0, a.N, RP / 4);
        if constexpr (ROWS) vr.load((const St*)a.Val, a.rows, bh, c0, a.N);
        else vr.load(Vl, c0, a.N, vs);
        if constexpr (KIND == kStateBwd) awv = aw[min(c0 + (int)threadIdx.x, a.N - 1)];   // masked to the chunk's rows where stored
    };
    load_chunk(t_beg);
    for (int t0 = t_beg; t0 < t_end; t0 += kC) {
        __syncthreads();
        if constexpr (ROWS) vr.store(a.rows, bh, t0, a.N, sm.v, sm.aw);
        else vr.store(sm.v);
        if (KIND == kStateBwd && threadIdx.x < kC) sm.aw.put(threadIdx.x, t0 + (int)threadIdx.x < a.N ? awv : 0.f);
        features_from<T, RPW>(ur, t0, a.N, L, a.two_beta, sm.ph);
        __syncthreads();
        load_chunk(t0 + kC < t_end ? t0 + kC : t0);   // the last chunk reloads its own (unconditional loads)
        // S[f][cols of wave] += Phi'[f][rows] V[rows][cols]
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            F bv[DW];
#pragma unroll
            for (int j = 0; j < DW; ++j) bv[j] = TV::col8(sm.v, 32 * kk, 16 * (w * DW + j));
#pragma unroll
            for (int ft = 0; ft < FT; ++ft) {
                const F af = TP::col8(sm.ph, 32 * kk, 16 * ft);
#pragma unroll
                for (int j = 0; j < DW; ++j) S[ft][j] = T::mma(af, bv[j], S[ft][j]);
                if (ft % 4 == w) {
                    if constexpr (!T::kSplit) {
                        float s = 0.f;           // (eight tokens first: a shorter chain of sums)
#pragma unroll
                        for (int i = 0; i < 8; ++i) s += BWD ? af[i] * sm.aw.v[0][32 * kk + 8 * g + i] : af[i];
                        Aacc[ft / 4][0] += s;
                    } else if constexpr (BWD) {
                        Aacc[ft / 4] = sm.aw.mma_b(af, 32 * kk + 8 * g, Aacc[ft / 4]);
                    } else {
                        Aacc[ft / 4] = token_sums<T>(af, Aacc[ft / 4]);
                    }
                }
            }
        }
    }
    float* out = a.states + (bh * a.nseg + seg) * (size_t)(RP * D + RP);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int j = 0; j < DW; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[(size_t)(F0 + 16 * ft + 4 * g + i) * D + 16 * (w * DW + j) + col] = S[ft][j][i] * a.mul;
#pragma unroll
    for (int j = 0; j < NFA; ++j) {
        const int ft = w + 4 * j;
        if (ft >= FT) break;
        if constexpr (!T::kSplit) {
            const float s = wave_sum16(Aacc[j][0]);
            if (g == 0) out[RP * D + F0 + 16 * ft + col] = s * a.mul;
        } else if (col == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) out[RP * D + F0 + 16 * ft + 4 * g + i] = Aacc[j][i] * a.mul;
        }
    }
}

__global__ __launch_bounds__(256) void race_scan_kernel(float* states, int nseg, int per, int mode)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < per) scan_states(states + blockIdx.y * (size_t)nseg * per + e, nseg, per, mode);
}

struct OutArgs {
    const float* Uq;      // projections of Q rows [BH][N][RP/4]
    const float* Uk;      // projections of K rows
    const void* V;
    const float* states;
    void* O_lr;           // storage dtype [BH][N][D]
    float* d_lr;
    int H, N, L, seg_len, nseg, causal;
    float two_beta, inv_L, eps;
};

template <class T, int D, int RP>
__global__ __launch_bounds__((state_waves<D, RP>() * 64), 2) void race_out_kernel(OutArgs a)
{
    using St = typename T::store_t;
    using F = typename T::frag_t;
    // WS groups of four waves: a chunk's feature tables and the key tiles of
    // its kernel matrix are dealt over the groups
    constexpr int NW = state_waves<D, RP>(), WS = NW / 4, RW = RP / WS;
    constexpr int DW = D / (16 * NW);
    constexpr int FS = RP / 32;
    using TV = RowTile<T, D>;
    using TP = RowTile<T, RP>;
    __shared__ __attribute__((aligned(16))) OutSmem<T, D, RP> sm;
    const int seg = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const size_t bh = (size_t)b * a.H + h;
    const float* Uq = a.Uq + bh * a.N * (RP / 4);
    const float* Uk = a.Uk + bh * a.N * (RP / 4);
    const St* V = (const St*)a.V + bh * a.N * D;
    St* Olr = (St*)a.O_lr + bh * a.N * D;
    float* dlr = a.d_lr + bh * a.N;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);   // wave-uniform, as in race_state
    const int g = lane >> 4, col = lane & 15;
    const int grp = WS > 1 ? w >> 2 : 0, wq = w - 4 * grp, tx = threadIdx.x - kThreads * grp;   // group, place in it

    const float* st_in = a.states + (bh * a.nseg + seg) * (size_t)(RP * D + RP);
    f32x4 S[RP / 16][DW];
#pragma unroll
    for (int ft = 0; ft < RP / 16; ++ft)
#pragma unroll
        for (int j = 0; j < DW; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                S[ft][j][i] = st_in[(size_t)(16 * ft + 4 * g + i) * D + 16 * (w * DW + j) + col];
    for (int f = threadIdx.x; f < RP; f += NW * 64) sm.a_state.put(f, st_in[RP * D + f]);
    // A runs on the matrix cores (causal): wave w keeps the feature tiles
    // ft = w, w + NW, ... in accumulator tiles (every column holds the sums;
    // column 0 starts from the segment's prefix state and is published to
    // a_state after each chunk)
    constexpr int FT = RP / 16, NFA = (FT + NW - 1) / NW;
    f32x4 Aacc[NFA];
#pragma unroll
    for (int j = 0; j < NFA; ++j) {
        const int ft = w + NW * j;
#pragma unroll
        for (int i = 0; i < 4; ++i) Aacc[j][i] = ft < FT && col == 0 ? st_in[RP * D + 16 * ft + 4 * g + i] : 0.f;
    }

    const int t_beg = seg * a.seg_len, t_end = min(a.N, t_beg + a.seg_len);
    URegs<RW> uq, uk;                    // projections and V rows of the chunk, loaded one chunk ahead
    StageRows<T, D, false, NW * 64> vr;
    uq.load(Uq + grp * (RW / 4), t_beg, a.N, RP / 4, tx);
    if (a.causal) {
        uk.load(Uk + grp * (RW / 4), t_beg, a.N, RP / 4, tx);
        vr.load(V, t_beg, a.N);
    }
    for (int t0 = t_beg; t0 < t_end; t0 += kC) {
        __syncthreads();
        features_from<T, RW, RP>(uq, t0, a.N, a.L - grp * (RW / 16), a.two_beta, sm.phq + grp * RW, tx);
        if (a.causal) {
            vr.store(sm.v);
            features_from<T, RW, RP>(uk, t0, a.N, a.L - grp * (RW / 16), a.two_beta, sm.phk + grp * RW, tx);
        }
        __syncthreads();
        {
            // next chunk's rows (the last chunk reloads its own: unconditional loads)
            const int tn = t0 + kC < t_end ? t0 + kC : t0;
            uq.load(Uq + grp * (RW / 4), tn, a.N, RP / 4, tx);
            if (a.causal) {
                uk.load(Uk + grp * (RW / 4), tn, a.N, RP / 4, tx);
                vr.load(V, tn, a.N);
            }
        }
        // the wave's 16 queries: Den (with two groups, the group's half of it), inter part (1/L) Phi_Q . A (every row of
        // the product tile alike), and the rows [16wq, 16wq + 16) of the
        // intra-chunk kernel matrix (causal), formed transposed: lane (g, col)
        // holds keys 16 kt + 4 g + i of query 16 wq + col, so a row's four
        // entries leave in one store and its sum is in-lane plus one exchange
        // over the lane groups
        {
            const int qi = 16 * wq + col;
            F qf[FS];
            f32x4 da = {0, 0, 0, 0};
#pragma unroll
            for (int fs = 0; fs < FS; ++fs) {
                qf[fs] = TP::row8(sm.phq, qi, 32 * fs + 8 * g);
                if (fs / (FS / WS) == grp) {
                    if constexpr (T::kSplit) {
                        da = sm.a_state.mma_a(32 * fs + 8 * g, qf[fs], da);
                    } else {
                        // float32: each lane group sums its own features, two
                        // at a time, and the four parts are added in pairs
                        // (the matrix cores' one chain of RP products is less
                        // accurate: d_lr of 784 tokens, 64 features, off by
                        // 1.43e-7 against 0.91e-7)
                        const float* as = &sm.a_state.v[0][32 * fs + 8 * g];
#pragma unroll
                        for (int i = 0; i < 4; ++i) da[0] += qf[fs][i] * as[i] + qf[fs][4 + i] * as[4 + i];
                    }
                }
            }
            if constexpr (!T::kSplit) da[0] = wave_sum16(da[0]);
            float rs = 0.f;
            if (a.causal) {
                for (int kt = grp; kt < 4; kt += WS) {
                    f32x4 mt = {0, 0, 0, 0};
                    if (kt <= wq) {
#pragma unroll
                        for (int fs = 0; fs < FS; ++fs)
                            mt = T::mma(TP::row8(sm.phk, 16 * kt + col, 32 * fs + 8 * g), qf[fs], mt);
                    }
                    f32x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int kj = 16 * kt + 4 * g + i;
                        v[i] = (kj <= qi) ? mt[i] * a.inv_L : 0.f;
                        rs += v[i];
                    }
                    store4<T>(&sm.mm[qi][16 * kt + 4 * g], v);
                }
                rs = wave_sum16(rs);
            }
            if (g == 0) {
                const float den = da[0] * a.inv_L + rs;
                sm.den[grp][qi] = den;
                if (WS == 1 && t0 + qi < a.N) dlr[t0 + qi] = den;
            }
        }
        __syncthreads();
        // Num^T for the wave's d columns, all 64 queries (lane (g, col) holds
        // d = 16 (w DW + j) + 4 g + i of query 16 qt + col): inter-chunk part
        // with S rounded to the storage dtype once per chunk (the forward
        // sums positive features against it, no cancellation), then the
        // masked intra-chunk part
        f32x4 num[4][DW];
#pragma unroll
        for (int qt = 0; qt < 4; ++qt)
#pragma unroll
            for (int j = 0; j < DW; ++j) num[qt][j] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int fs = 0; fs < FS; ++fs) {
            F sf[DW];
#pragma unroll
            for (int j = 0; j < DW; ++j) {
                float sv[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sv[i] = S[2 * fs][j][i];
                    sv[4 + i] = S[2 * fs + 1][j][i];
                }
                sf[j] = T::pack(sv);
            }
#pragma unroll
            for (int qt = 0; qt < 4; ++qt) {
                const F af = TP::row44(sm.phq, 16 * qt + col, 32 * fs + 4 * g);
#pragma unroll
                for (int j = 0; j < DW; ++j) num[qt][j] = T::mma(sf[j], af, num[qt][j]);
            }
        }
#pragma unroll
        for (int qt = 0; qt < 4; ++qt)
#pragma unroll
            for (int j = 0; j < DW; ++j) num[qt][j] *= a.inv_L;
        F bv[2][DW];                     // V^T operands: the intra-chunk part and the state update
        if (a.causal) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int j = 0; j < DW; ++j) bv[kk][j] = TV::col8(sm.v, 32 * kk, 16 * (w * DW + j));
#pragma unroll
                for (int qt = 0; qt < 4; ++qt) {
                    const F bf = T::ld8(&sm.mm[16 * qt + col][32 * kk + 8 * g]);
#pragma unroll
                    for (int j = 0; j < DW; ++j) num[qt][j] = T::mma(bv[kk][j], bf, num[qt][j]);
                }
            }
        }
#pragma unroll
        for (int qt = 0; qt < 4; ++qt) {
            const int ql = 16 * qt + col;
            const int tok = t0 + ql;
            float den = sm.den[0][ql];
            if constexpr (WS > 1) {
                den += sm.den[WS - 1][ql];
                if (w == 0 && g == 0 && tok < a.N) dlr[tok] = den;
            }
            const float inv = 1.f / (den + a.eps);
            if (tok < a.N) {
#pragma unroll
                for (int j = 0; j < DW; ++j)
                    store4<T>(Olr + (size_t)tok * D + 16 * (w * DW + j) + 4 * g, num[qt][j] * inv);
            }
        }
        if (a.causal) {
            // S += Phi_K' V (chunk), A += Phi_K' 1
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int ft = 0; ft < FT; ++ft) {
                    const F af = TP::col8(sm.phk, 32 * kk, 16 * ft);
#pragma unroll
                    for (int j = 0; j < DW; ++j) S[ft][j] = T::mma(af, bv[kk][j], S[ft][j]);
                    if (ft % NW == w) Aacc[ft / NW] = token_sums<T>(af, Aacc[ft / NW]);
                }
            }
            // the den of the next chunk reads a_state after its first barrier
#pragma unroll
            for (int j = 0; j < NFA; ++j) {
                const int ft = w + NW * j;
                if (ft < FT && col == 0)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sm.a_state.put(16 * ft + 4 * g + i, Aacc[j][i]);
            }
        }
    }
}

template <class T, int D, int RP>
constexpr bool fits()
{
    return sizeof(StateSmem<T, D, RP / table_split<RP>()>) <= kMaxLds && sizeof(OutSmem<T, D, RP>) <= kMaxLds;
}

// The row scalars in the state pass: one launch and one reading of dO less.
// At d_h 64 that is a gain for short calls (whole steps: 65536 rows, 64
// features 112 -> 106 us, encoder step 123 -> 118; float32 25088 rows 140 ->
// 137, 65536 rows 189 -> 185; 262144 rows, past the line, 324 -> 314).  At d_h 128 the pass's registers leave two
// workgroups a compute unit in bf16 and one in float32, too few to stream O_s
// at the row pass's rate: up to 64 features and 65536 rows it is still the
// faster one or equal (32768 rows 128 -> 126, 65536 175 -> 174; 131072 rows
// 312 -> 315), at 128 features (32768 rows 164 -> 166, 131072 368 -> 378) and
// in float32 (4096 rows 87 -> 91, 65536 341 -> 354) it loses throughout.
// With the tables split over two workgroups every row would be read twice.
template <class T, int D, int RP>
constexpr bool rows_can_fuse()
{
    return table_split<RP>() == 1 && (D == 64 || (T::bytes == 2 && RP <= 64));
}
template <class T, int D, int RP>
bool fused_rows(const Shape& s)
{
    return rows_can_fuse<T, D, RP>() && (int64_t)s.B * s.H * s.N <= (D == 64 ? 131072 : 65536);
}

template <class T, int D, int RP>
hipError_t launch_states_t(const Shape& s, const StateArgs& a, bool bwd, const SortJob* sort, hipStream_t st)
{
    if constexpr (!fits<T, D, RP>()) {
        return hipErrorInvalidConfiguration;
    } else {
        dim3 grid(s.nseg * table_split<RP>(), s.H, s.B);
        hipError_t e;
        if (!bwd) ELSAA_LAUNCH("race_state_fwd", (race_state_kernel<T, D, RP, kStateFwd>), grid, dim3(kThreads), 0, st, a);
        else if (fused_rows<T, D, RP>(s)) {
            if constexpr (rows_can_fuse<T, D, RP>())
                ELSAA_LAUNCH("race_rows_bwd", (race_state_kernel<T, D, RP, kStateRows>), grid, dim3(kThreads), 0, st, a);
        } else {
            if ((e = launch_bwd_rows(s, a.Val, a.rows, st)) != hipSuccess) return e;
            ELSAA_LAUNCH("race_state_bwd", (race_state_kernel<T, D, RP, kStateBwd>), grid, dim3(kThreads), 0, st, a);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const int per = RP * D + RP, scan_mode = !s.causal ? 0 : bwd ? 2 : 1;
        if (sort && sort_tasks(s) > 0) return launch_sort(s, *sort, ScanJob{a.states, s.nseg, per, scan_mode}, st);
        ELSAA_LAUNCH(bwd ? "race_scan_bwd" : "race_scan_fwd", race_scan_kernel, dim3((per + 255) / 256, s.B * s.H), dim3(256), 0, st,
                           a.states, s.nseg, per, scan_mode);
        return hipGetLastError();
    }
}

template <class T, int D, int RP>
hipError_t launch_out_t(const Shape& s, const OutArgs& a, hipStream_t st)
{
    if constexpr (!fits<T, D, RP>()) {
        return hipErrorInvalidConfiguration;
    } else {
        dim3 grid(s.nseg, s.H, s.B);
        ELSAA_LAUNCH("race_out", (race_out_kernel<T, D, RP>), grid, dim3(state_waves<D, RP>() * 64), 0, st, a);
        return hipGetLastError();
    }
}

template <template <class, int, int> class Fn, class... A>
hipError_t dispatch(const Shape& s, A&&... args)
{
    const int rp = race_padded_features(s.r);
#define ELSAA_RP(T_, D_)                                                        \
    switch (rp) {                                                               \
        case 32: return Fn<T_, D_, 32>::run(s, args...);                        \
        case 64: return Fn<T_, D_, 64>::run(s, args...);                        \
        case 128: return Fn<T_, D_, 128>::run(s, args...);                      \
        default: return Fn<T_, D_, 256>::run(s, args...);                       \
    }
    if (s.bf16) {
        if (s.D == 64) { ELSAA_RP(BF16, 64) }
        ELSAA_RP(BF16, 128)
    }
    if (s.D == 64) { ELSAA_RP(F32, 64) }
    ELSAA_RP(F32, 128)
#undef ELSAA_RP
}

template <class T, int D, int RP>
struct StatesFn {
    static hipError_t run(const Shape& s, const StateArgs& a, bool bwd, const SortJob* sort, hipStream_t st)
    {
        return launch_states_t<T, D, RP>(s, a, bwd, sort, st);
    }
};

template <class T, int D, int RP>
struct OutFn {
    static hipError_t run(const Shape& s, const OutArgs& a, hipStream_t st) { return launch_out_t<T, D, RP>(s, a, st); }
};

template <class T, int D, int RP>
struct FitsFn {
    static hipError_t run(const Shape&) { return fits<T, D, RP>() ? hipSuccess : hipErrorInvalidConfiguration; }
};

}  // namespace

// Padded feature count of the GPU path: r rounded up to 32, 64, 128 or 256.
int race_padded_features(int r) { return r <= 32 ? 32 : r <= 64 ? 64 : r <= 128 ? 128 : 256; }

size_t race_state_floats(const Shape& s)
{
    const int rp = race_padded_features(s.r);
    return (size_t)s.B * s.H * s.nseg * ((size_t)rp * s.D + rp);
}

bool race_fwd_fits(const Shape& s) { return dispatch<FitsFn>(s) == hipSuccess; }

int race_proj_stride(const Shape& s) { return race_padded_features(s.r) / 4; }

hipError_t launch_race_bwd_states(const Shape& s, const float* Uq, const void* dO, const RowArgs& rows,
                                  float* states_b, hipStream_t st)
{
    StateArgs a;
    a.U = Uq; a.Val = dO; a.vscale = rows.rs + 3 * rows.BHN; a.aw = rows.rs + 4 * rows.BHN; a.states = states_b;
    a.H = s.H; a.N = s.N; a.L = s.L; a.seg_len = s.seg_len; a.nseg = s.nseg;
    a.two_beta = 2.f * s.beta; a.mul = 1.f / (float)s.L;
    a.rows = rows;
    return dispatch<StatesFn>(s, a, true, (const SortJob*)nullptr, st);
}

hipError_t launch_race_fwd(const Shape& s, const float* Uq, const float* Uk, const void* V,
                           float* states, void* O_lr, float* d_lr, const SortJob* sort, hipStream_t st)
{
    StateArgs sa = {};
    sa.U = Uk; sa.Val = V; sa.states = states;
    sa.H = s.H; sa.N = s.N; sa.L = s.L; sa.seg_len = s.seg_len; sa.nseg = s.nseg;
    sa.two_beta = 2.f * s.beta; sa.mul = 1.f;
    hipError_t e = dispatch<StatesFn>(s, sa, false, sort, st);
    if (e != hipSuccess) return e;
    OutArgs a;
    a.Uq = Uq; a.Uk = Uk; a.V = V; a.states = states;
    a.O_lr = O_lr; a.d_lr = d_lr;
    a.H = s.H; a.N = s.N; a.L = s.L; a.seg_len = s.seg_len; a.nseg = s.nseg; a.causal = s.causal;
    a.two_beta = 2.f * s.beta; a.inv_L = 1.f / (float)s.L; a.eps = s.eps;
    return dispatch<OutFn>(s, a, st);
}

}  // namespace elsaa
