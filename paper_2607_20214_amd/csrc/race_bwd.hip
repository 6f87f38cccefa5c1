// race_bwd.hip -- backward of the RACE low-rank branch (Alg. 2 / Alg. 3 differentiated).
//
// With dNum_i = g_lr dO_i / (Den_i + eps) and dDen_i (row scalars of the
// backward preprocess), and V~_j = [V_j, 1], dN~_i = [dNum_i, dDen_i]:
//   dphi(q_i) = (1/L) sum_{j <= i} <dN~_i, V~_j> phi(k_j)          (pass LB1, forward time)
//   dphi(k_j) = (1/L) sum_{i >= j} <dN~_i, V~_j> phi(q_i)          (pass LB2, reverse time)
//   dV_j      = (1/L) sum_{i >= j} <phi(q_i), phi(k_j)> dNum_i      (pass LB3, reverse time)
// (non-causal: all i, j).  Each is a linear-attention pass over 64-token
// chunks with a running state: LB1 reads S = sum phi(k) V', A = sum phi(k)
// (the forward's segment prefix states); LB2 and LB3 read the suffix states
// dS = (1/L) sum phi(q) dNum', dA = (1/L) sum phi(q) dDen.  LB1 and LB2
// contract their state over d, so each wave owns a quarter of the features;
// LB3 contracts over the features, so each wave owns a share of d.
// dphi is chained through phi = prod sigmoid(2 beta v t), t = tanh(W x) to
// du, the gradient of the projections u = W x.  LB1 and LB2 store du (storage
// dtype, [BH][N][wk], wk = 4L padded to 32) and the sparse backward forms
// dQ (dK) += du W on MFMA where it adds its own part, so only wk values per
// row cross HBM instead of d float32 ones; this pass provides W' = W_hi' +
// W_lo' ([H][D][wk], bf16 parts of float32 accuracy).  The running states
// enter the MFMAs split the same way: their products cancel against the dDen
// terms.  LB3 writes dV in the storage dtype [BH][N][D]; the sparse backward
// adds it to its float32 dV before the final rounding.
#include <type_traits>

#include "internal.hpp"
#include "race_common.hpp"

namespace elsaa {

using namespace race;

namespace {

struct LbArgs {
    const float* Uq;        // projections of Q rows [BH][N][RP/4]
    const float* Uk;        // projections of K rows
    const void* V;
    const void* dO;
    const float* rs;        // row scalars (sc_lr at 3*BHN, dDen at 4*BHN)
    const float* states_f;  // forward prefix states (LB1)
    const float* states_b;  // backward suffix states (LB2, LB3)
    void* du_q;             // du rows [BH][N][wk] (storage dtype)
    void* du_k;
    void* dv;               // dV rows [BH][N][D] (storage dtype)
    const float* W;         // W_race [H][4L][D]
    void* wt_hi;            // W' parts [H][D][wk] (storage dtype)
    void* wt_lo;
    int H, N, L, seg_len, nseg, causal;
    int items;              // B H nseg
    size_t BHN;
    float two_beta, inv_L;
};

// Non-causal passes only apply the total states: their workgroups hold no
// intra-chunk operands, so more of them fit a compute unit (C = 0: short
// arrays in their place). Instantiated apart, r = 64: bf16 d_h 64 takes 84
// registers and 19 KB (was 136 and 47 KB: 3 -> 5 workgroups a compute unit),
// float32 121 and 34 KB (220 and 89 KB: 1 -> 4); the float32 training step of
// 32 heads x 784 tokens, with two workgroups of the block kernel a compute
// unit as well, 137 -> 114 us.
template <class T, int D, int RP, bool C>
struct Lb1Smem {
    using S = typename T::store_t;
    S dn[RowTile<T, D>::ELEMS];            // dO chunk (dNum_i = sc_lr,i dO_i: the products apply sc_lr)
    S v[C ? RowTile<T, D>::ELEMS : 8];     // V chunk
    S pk[C ? RowTile<T, RP>::ELEMS : 8];   // Phi_K chunk
    S gg[C ? kC : 1][kC + kPad];           // G[i][j] = <dNum_i, V_j> + dDen_i, j <= i
    float ts[kC][RP / 4];                  // tanh(W q) of the chunk's queries
    S du[kC][w_kdim<RP>() + kPad];
    float dden[kC];
    float sc[kC];                          // sc_lr of the chunk's queries
};

template <class T, int D, int RP, bool C>
struct Lb2Smem {
    using S = typename T::store_t;
    S v[RowTile<T, D>::ELEMS];             // V chunk
    S dn[C ? RowTile<T, D>::ELEMS : 8];    // dNum / L chunk
    S pq[C ? RowTile<T, RP>::ELEMS : 8];   // Phi_Q chunk
    S ggt[C ? kC : 1][kC + kPad];          // G'[j][i] / L, i >= j
    float ts[kC][RP / 4];                  // tanh(W k) of the chunk's keys
    S du[kC][w_kdim<RP>() + kPad];
    Parts<T, kC> ddp;                      // dDen / L as operand parts
    float dden[kC];                        // dDen / L
};

template <class T, int D, int RP, bool C>
struct Lb3Smem {
    using S = typename T::store_t;
    S pk[RowTile<T, RP>::ELEMS];           // Phi_K chunk
    S dn[C ? RowTile<T, D>::ELEMS : 8];    // dNum / L chunk
    S pq[C ? RowTile<T, RP>::ELEMS : 8];   // Phi_Q chunk
    S mt[C ? kC : 1][kC + kPad];           // M'[j][i] = <phi(k_j), phi(q_i)>, i >= j
};

template <class T, int D, int RP>
constexpr bool bwd_fits()
{
    return sizeof(Lb1Smem<T, D, RP / table_split<RP>(), true>) <= kMaxLds &&
           sizeof(Lb2Smem<T, D, RP / table_split<RP>(), true>) <= kMaxLds &&
           sizeof(Lb3Smem<T, D, RP, true>) <= kMaxLds;
}

// du rows [t0, t0 + 64) of the chunk (LDS, storage dtype) -> rows of out
// [N][WK], 16 bytes per thread and store.
template <class T, int RPW, int RP>
__device__ __forceinline__ void store_du(const typename T::store_t (*du)[w_kdim<RPW>() + kPad],
                                         typename T::store_t* out, int t0, int N, int tx)
{
    // a workgroup holding all the features writes whole (padded) rows,
    // one holding some of the tables their RPW / 4 columns
    constexpr int WK = w_kdim<RP>(), COLS = RPW == RP ? WK : RPW / 4;
    constexpr int PER = 16 / T::bytes, CH = COLS / PER;
    static_assert(COLS % PER == 0, "du row of whole 16-byte pieces");
    for (int it = tx; it < kC * CH; it += kThreads) {
        const int r = it / CH, c = it % CH;
        if (t0 + r < N) stg16(out + (size_t)(t0 + r) * WK + c * PER, *(const uint4*)&du[r][c * PER]);
    }
}

// W' = W_hi' + W_lo' of every head, [H][D][WK] (rows 4l + b, zero past 4L):
// kWtPer elements per workgroup of the passes' launch.
constexpr int kWtPer = 8 * kThreads;
template <class T>
__device__ __forceinline__ void wt_body(const LbArgs& a, int blk, int D, int WK)
{
    using St = typename T::store_t;
    const int per = D * WK, n = a.H * per;
    for (int j = 0; j < kWtPer / kThreads; ++j) {
        const int it = blk * kWtPer + j * kThreads + threadIdx.x;
        if (it >= n) return;
        const int h = it / per, d = it % per / WK, p = it % WK;
        const float w = p < 4 * a.L ? a.W[((size_t)h * 4 * a.L + p) * D + d] : 0.f;
        const St vh = T::store(w);
        ((St*)a.wt_hi)[it] = vh;
        ((St*)a.wt_lo)[it] = T::store(T::kSplit ? w - T::load(vh) : 0.f);
    }
}

// The state part of dphi' for the wave's feature tile in St (rows d, its
// columns the tile's features) against the 64 rows of x: acc[t] = S' x_t for
// the 16-row tiles t.  The state enters as hi + lo bf16 parts, split once per
// chunk and k-step.
template <class T, int D>
__device__ __forceinline__ void state_product(const f32x4 (&St)[D / 16], const typename T::store_t* x, f32x4 (&acc)[4],
                                              int tx)
{
    using F = typename T::frag_t;
    const int lane = tx & 63, g = lane >> 4, col = lane & 15;
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int ds = 0; ds < D / 32; ++ds) {
        float sv[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sv[i] = St[2 * ds][i];
            sv[4 + i] = St[2 * ds + 1][i];
        }
        F shi, slo;
        T::split(sv, shi, slo);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const F bf = RowTile<T, D>::row44(x, 16 * t + col, 32 * ds + 4 * g);
            acc[t] = T::mma(shi, bf, acc[t]);
            if (T::kSplit) acc[t] = T::mma(slo, bf, acc[t]);
        }
    }
}

// ---------------------------------------------------------------- LB1: dQ
template <class T, int D, int RP, bool CAUSAL>
__device__ __forceinline__ void race_dq_body(const LbArgs& a, size_t bh, int seg, int part,
                                             Lb1Smem<T, D, RP / table_split<RP>(), CAUSAL>& sm)
{
    using St = typename T::store_t;
    using F = typename T::frag_t;
    constexpr int RPW = RP / table_split<RP>();                    // features of this workgroup
    constexpr int DT = D / 16, KS = D / 32, FT = RPW / 16, NFT = (FT + 3) / 4;
    using TV = RowTile<T, D>;
    using TP = RowTile<T, RPW>;
    const int F0 = part * RPW, L = a.L - F0 / 16;                  // first feature; tables from here on
    const float* Uq = a.Uq + bh * a.N * (RP / 4) + F0 / 4;
    const float* Uk = a.Uk + bh * a.N * (RP / 4) + F0 / 4;
    const St* V = (const St*)a.V + bh * a.N * D;
    const St* dO = (const St*)a.dO + bh * a.N * D;
    const float* sclr = a.rs + 3 * a.BHN + bh * a.N;
    const float* dden = a.rs + 4 * a.BHN + bh * a.N;
    St* du_out = (St*)a.du_q + bh * a.N * w_kdim<RP>() + F0 / 4;
    int tx = threadIdx.x;
    asm volatile("" : "+v"(tx));                                  // this body's own copy (race_common.hpp)
    const int lane = tx & 63, w = __builtin_amdgcn_readfirstlane(tx >> 6);
    const int g = lane >> 4, col = lane & 15;

    for (int it = tx; it < kC * (w_kdim<RPW>() + kPad); it += kThreads)
        (&sm.du[0][0])[it] = T::store(0.f);
    // state S'[d][f] for the wave's features f = 16 (w + 4j) + col, and
    // A[f] of the same feature tiles (lane (g, col) register i: feature
    // 16 (w + 4j) + 4 g + i, every column alike; token_sums keeps it so)
    f32x4 St_[NFT][DT], Aacc[NFT];
    const float* st_in = a.states_f + (bh * a.nseg + seg) * (size_t)(RP * D + RP);
#pragma unroll
    for (int j = 0; j < NFT; ++j) {
        const int ft = w + 4 * j;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                St_[j][dt][i] = ft < FT ? st_in[(size_t)(F0 + 16 * ft + col) * D + 16 * dt + 4 * g + i] : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) Aacc[j][i] = ft < FT ? st_in[RP * D + F0 + 16 * ft + 4 * g + i] : 0.f;
    }

    const int t_beg = seg * a.seg_len, t_end = min(a.N, t_beg + a.seg_len);
    URegs<RPW> uq, uk;                    // projections of the chunk, loaded one chunk ahead
    uq.load(Uq, t_beg, a.N, RP / 4, tx);
    if constexpr (CAUSAL) uk.load(Uk, t_beg, a.N, RP / 4, tx);
    for (int t0 = t_beg; t0 < t_end; t0 += kC) {
        __syncthreads();
        // every global load of the chunk is issued first; the features (vector
        // work) run while they are in flight, then the rows go to LDS
        StageRows<T, D, false> sdn, sv;
        sdn.load(dO, t0, a.N, nullptr, tx);
        if constexpr (CAUSAL) sv.load(V, t0, a.N, nullptr, tx);
        const bool in = tx < kC && t0 + tx < a.N;
        const float ddv = in ? dden[t0 + tx] : 0.f, scv = in ? sclr[t0 + tx] : 0.f;
        tanh_rows<RPW>(uq, sm.ts, tx);
        if constexpr (CAUSAL) features_from<T, RPW>(uk, t0, a.N, L, a.two_beta, sm.pk, tx);
        sdn.store(sm.dn, 1.f, tx);
        if constexpr (CAUSAL) sv.store(sm.v, 1.f, tx);
        if (tx < kC) {
            sm.dden[tx] = ddv;
            sm.sc[tx] = scv;
        }
        __syncthreads();
        {
            // next chunk's projections (the last chunk reloads its own, so
            // the loads are unconditional)
            const int tn = t0 + kC < t_end ? t0 + kC : t0;
            uq.load(Uq, tn, a.N, RP / 4, tx);
            if constexpr (CAUSAL) uk.load(Uk, tn, a.N, RP / 4, tx);
        }
        if constexpr (CAUSAL) {
            // G rows [16w, 16w + 16): sc_lr,i <dO_i, V_j> + dDen_i for j <= i,
            // formed transposed (lane (g, col): keys 16 kt + 4 g + i of query
            // 16 w + col) so each lane stores four entries of its row at once
            const int qi = 16 * w + col;
            const float scq = sm.sc[qi], ddq = sm.dden[qi];
            F df[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) df[ks] = TV::row8(sm.dn, qi, 32 * ks + 8 * g);
            for (int kt = 0; kt < 4; ++kt) {
                f32x4 acc = {0, 0, 0, 0};
                if (kt <= w) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
                        acc = T::mma(TV::row8(sm.v, 16 * kt + col, 32 * ks + 8 * g), df[ks], acc);
                }
                f32x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = 16 * kt + 4 * g + i <= qi ? acc[i] * scq + ddq : 0.f;
                store4<T>(&sm.gg[qi][16 * kt + 4 * g], v);
            }
        }
        __syncthreads();
        // dphi(q)' tiles [features of table ft] x [16 queries]: sc_lr S dO + A dDen + intra
#pragma unroll
        for (int j = 0; j < NFT; ++j) {
            const int ft = w + 4 * j;
            if (ft >= FT) break;
            f32x4 acc[4];
            state_product<T, D>(St_[j], sm.dn, acc, tx);
#pragma unroll
            for (int qt = 0; qt < 4; ++qt) {
                const float ddq = sm.dden[16 * qt + col], scq = sm.sc[16 * qt + col];
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[qt][i] = acc[qt][i] * scq + Aacc[j][i] * ddq;
            }
            if constexpr (CAUSAL) {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const F pf = TP::col8(sm.pk, 32 * kk, 16 * ft, tx);
#pragma unroll
                    for (int qt = 0; qt < 4; ++qt)
                        acc[qt] = T::mma(pf, T::ld8(&sm.gg[16 * qt + col][32 * kk + 8 * g]), acc[qt]);
                }
            }
            // the four tiles' chain rules side by side: their exchanges overlap
#pragma unroll
            for (int qt = 0; qt < 4; ++qt)
                chain_rule_t<T, RPW>(acc[qt], qt, ft, L, a.two_beta, a.two_beta * a.inv_L, sm.ts, sm.du, tx);
        }
        __syncthreads();
        store_du<T, RPW, RP>(sm.du, du_out, t0, a.N, tx);
        if constexpr (CAUSAL) {
            // S' += V' Phi_K (chunk), A += Phi_K' 1
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                F pf[NFT];
#pragma unroll
                for (int j = 0; j < NFT; ++j) {
                    const int ft = w + 4 * j;
                    if (ft >= FT) break;
                    pf[j] = TP::col8(sm.pk, 32 * kk, 16 * ft, tx);
                    Aacc[j] = token_sums<T>(pf[j], Aacc[j]);
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const F vf = TV::col8(sm.v, 32 * kk, 16 * dt, tx);
#pragma unroll
                    for (int j = 0; j < NFT; ++j) {
                        if (w + 4 * j >= FT) break;
                        St_[j][dt] = T::mma(vf, pf[j], St_[j][dt]);
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------- LB2: dK
template <class T, int D, int RP, bool CAUSAL>
__device__ __forceinline__ void race_dk_body(const LbArgs& a, size_t bh, int seg, int part,
                                             Lb2Smem<T, D, RP / table_split<RP>(), CAUSAL>& sm)
{
    using St = typename T::store_t;
    using F = typename T::frag_t;
    constexpr int RPW = RP / table_split<RP>();                    // features of this workgroup
    constexpr int DT = D / 16, KS = D / 32, FT = RPW / 16, NFT = (FT + 3) / 4;
    using TV = RowTile<T, D>;
    using TP = RowTile<T, RPW>;
    const int F0 = part * RPW, L = a.L - F0 / 16;                  // first feature; tables from here on
    const float* Uq = a.Uq + bh * a.N * (RP / 4) + F0 / 4;
    const float* Uk = a.Uk + bh * a.N * (RP / 4) + F0 / 4;
    const St* V = (const St*)a.V + bh * a.N * D;
    const St* dO = (const St*)a.dO + bh * a.N * D;
    const float* sclr = a.rs + 3 * a.BHN + bh * a.N;
    const float* dden = a.rs + 4 * a.BHN + bh * a.N;
    St* du_out = (St*)a.du_k + bh * a.N * w_kdim<RP>() + F0 / 4;
    int tx = threadIdx.x;
    asm volatile("" : "+v"(tx));                                  // this body's own copy (race_common.hpp)
    const int lane = tx & 63, w = __builtin_amdgcn_readfirstlane(tx >> 6);
    const int g = lane >> 4, col = lane & 15;

    for (int it = tx; it < kC * (w_kdim<RPW>() + kPad); it += kThreads)
        (&sm.du[0][0])[it] = T::store(0.f);
    // the suffix state of the wave's feature tiles, as in the dQ pass:
    // dS'[d][f], and dA[f] = (1/L) sum phi(q) dDen of the queries after the chunk
    f32x4 St_[NFT][DT], Aacc[NFT];
    const float* st_in = a.states_b + (bh * a.nseg + seg) * (size_t)(RP * D + RP);
#pragma unroll
    for (int j = 0; j < NFT; ++j) {
        const int ft = w + 4 * j;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                St_[j][dt][i] = ft < FT ? st_in[(size_t)(F0 + 16 * ft + col) * D + 16 * dt + 4 * g + i] : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) Aacc[j][i] = ft < FT ? st_in[RP * D + F0 + 16 * ft + 4 * g + i] : 0.f;
    }

    const int t_beg = seg * a.seg_len, t_end = min(a.N, t_beg + a.seg_len);
    const int nch = (t_end - t_beg + kC - 1) / kC;
    URegs<RPW> uq, uk;                    // projections of the chunk, loaded one chunk ahead
    uk.load(Uk, t_beg + (nch - 1) * kC, a.N, RP / 4, tx);
    if constexpr (CAUSAL) uq.load(Uq, t_beg + (nch - 1) * kC, a.N, RP / 4, tx);
    for (int c = nch - 1; c >= 0; --c) {
        const int t0 = t_beg + c * kC;
        __syncthreads();
        // loads first, features under them, then the LDS stores
        StageRows<T, D, false> svr;
        StageRows<T, D, true> sdn;
        svr.load(V, t0, a.N, nullptr, tx);
        if constexpr (CAUSAL) sdn.load(dO, t0, a.N, sclr, tx);
        const bool in = tx < kC && t0 + tx < a.N;
        const float ddv = in ? dden[t0 + tx] * a.inv_L : 0.f;
        tanh_rows<RPW>(uk, sm.ts, tx);
        if constexpr (CAUSAL) features_from<T, RPW>(uq, t0, a.N, L, a.two_beta, sm.pq, tx);
        svr.store(sm.v, 1.f, tx);
        if constexpr (CAUSAL) {
            sdn.store(sm.dn, a.inv_L, tx);
            if (tx < kC) {
                sm.dden[tx] = ddv;
                sm.ddp.put(tx, ddv);
            }
        }
        __syncthreads();
        {
            // previous chunk's projections (unconditional: chunk 0 reloads its own)
            const int tn = c > 0 ? t0 - kC : t0;
            uk.load(Uk, tn, a.N, RP / 4, tx);
            if constexpr (CAUSAL) uq.load(Uq, tn, a.N, RP / 4, tx);
        }
        if constexpr (CAUSAL) {
            // G' rows j in [16w, 16w + 16): (<V_j, dNum_i> + dDen_i) / L for
            // i >= j, formed transposed (lane (g, col): queries 16 it + 4 g + i
            // of key 16 w + col) so each lane stores four entries of its row at once
            const int kj = 16 * w + col;
            F vf[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) vf[ks] = TV::row8(sm.v, kj, 32 * ks + 8 * g);
            for (int it = 0; it < 4; ++it) {
                f32x4 acc = {0, 0, 0, 0};
                if (it >= w) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
                        acc = T::mma(TV::row8(sm.dn, 16 * it + col, 32 * ks + 8 * g), vf[ks], acc);
                }
                const f32x4 dd = *(const f32x4*)&sm.dden[16 * it + 4 * g];
                f32x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = 16 * it + 4 * g + i >= kj ? acc[i] + dd[i] : 0.f;
                store4<T>(&sm.ggt[kj][16 * it + 4 * g], v);
            }
        }
        __syncthreads();
        // dphi(k)' tiles [features of table ft] x [16 keys]: dS V + dA + intra
#pragma unroll
        for (int j = 0; j < NFT; ++j) {
            const int ft = w + 4 * j;
            if (ft >= FT) break;
            f32x4 acc[4];
            state_product<T, D>(St_[j], sm.v, acc, tx);
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) acc[kt] += Aacc[j];
            if constexpr (CAUSAL) {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const F pf = TP::col8(sm.pq, 32 * kk, 16 * ft, tx);
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt)
                        acc[kt] = T::mma(pf, T::ld8(&sm.ggt[16 * kt + col][32 * kk + 8 * g]), acc[kt]);
                }
            }
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
                chain_rule_t<T, RPW>(acc[kt], kt, ft, L, a.two_beta, a.two_beta, sm.ts, sm.du, tx);
        }
        __syncthreads();
        store_du<T, RPW, RP>(sm.du, du_out, t0, a.N, tx);
        if constexpr (CAUSAL) {
            // dS' += (dNum / L)' Phi_Q (chunk), dA += (1/L) Phi_Q' dDen
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                F pf[NFT];
#pragma unroll
                for (int j = 0; j < NFT; ++j) {
                    const int ft = w + 4 * j;
                    if (ft >= FT) break;
                    pf[j] = TP::col8(sm.pq, 32 * kk, 16 * ft, tx);
                    Aacc[j] = sm.ddp.mma_b(pf[j], 32 * kk + 8 * g, Aacc[j]);
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const F df = TV::col8(sm.dn, 32 * kk, 16 * dt, tx);
#pragma unroll
                    for (int j = 0; j < NFT; ++j) {
                        if (w + 4 * j >= FT) break;
                        St_[j][dt] = T::mma(df, pf[j], St_[j][dt]);
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------- LB3: dV
template <class T, int D, int RP, bool CAUSAL>
__device__ __forceinline__ void race_dv_body(const LbArgs& a, size_t bh, int seg, Lb3Smem<T, D, RP, CAUSAL>& sm)
{
    using St = typename T::store_t;
    using F = typename T::frag_t;
    constexpr int NW = state_waves<D, RP>(), WS = NW / 4, RW = RP / WS;   // as in race_out
    constexpr int DW = D / (16 * NW), FS = RP / 32;
    using TV = RowTile<T, D>;
    using TP = RowTile<T, RP>;
    const float* Uq = a.Uq + bh * a.N * (RP / 4);
    const float* Uk = a.Uk + bh * a.N * (RP / 4);
    const St* dO = (const St*)a.dO + bh * a.N * D;
    const float* sclr = a.rs + 3 * a.BHN + bh * a.N;
    St* out = (St*)a.dv + bh * a.N * D;
    int tx = threadIdx.x;
    asm volatile("" : "+v"(tx));                                  // this body's own copy (race_common.hpp)
    const int lane = tx & 63, w = __builtin_amdgcn_readfirstlane(tx >> 6);
    const int g = lane >> 4, col = lane & 15;
    const int grp = WS > 1 ? w >> 2 : 0, wq = w - 4 * grp, tg = tx - kThreads * grp;   // group, place in it

    const float* st_in = a.states_b + (bh * a.nseg + seg) * (size_t)(RP * D + RP);
    f32x4 S[RP / 16][DW];
#pragma unroll
    for (int ft = 0; ft < RP / 16; ++ft)
#pragma unroll
        for (int j = 0; j < DW; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                S[ft][j][i] = st_in[(size_t)(16 * ft + 4 * g + i) * D + 16 * (w * DW + j) + col];

    const int t_beg = seg * a.seg_len, t_end = min(a.N, t_beg + a.seg_len);
    const int nch = (t_end - t_beg + kC - 1) / kC;
    URegs<RW> uq, uk;                    // projections of the chunk, loaded one chunk ahead
    uk.load(Uk + grp * (RW / 4), t_beg + (nch - 1) * kC, a.N, RP / 4, tg);
    if constexpr (CAUSAL) uq.load(Uq + grp * (RW / 4), t_beg + (nch - 1) * kC, a.N, RP / 4, tg);
    for (int c = nch - 1; c >= 0; --c) {
        const int t0 = t_beg + c * kC;
        __syncthreads();
        // loads first, features under them, then the LDS stores
        StageRows<T, D, true, NW * 64> sdn;
        if constexpr (CAUSAL) sdn.load(dO, t0, a.N, sclr, tx);
        features_from<T, RW, RP>(uk, t0, a.N, a.L - grp * (RW / 16), a.two_beta, sm.pk + grp * RW, tg);
        if constexpr (CAUSAL) {
            features_from<T, RW, RP>(uq, t0, a.N, a.L - grp * (RW / 16), a.two_beta, sm.pq + grp * RW, tg);
            sdn.store(sm.dn, a.inv_L, tx);
        }
        __syncthreads();
        {
            // previous chunk's projections (unconditional: chunk 0 reloads its own)
            const int tn = c > 0 ? t0 - kC : t0;
            uk.load(Uk + grp * (RW / 4), tn, a.N, RP / 4, tg);
            if constexpr (CAUSAL) uq.load(Uq + grp * (RW / 4), tn, a.N, RP / 4, tg);
        }
        if constexpr (CAUSAL) {
            // M' rows j in [16wq, 16wq + 16): <phi(k_j), phi(q_i)> for i >= j,
            // formed transposed (lane (g, col): queries 16 it + 4 g + i of key
            // 16 wq + col) so each lane stores four entries of its row at once
            const int kj = 16 * wq + col;
            F kf[FS];
#pragma unroll
            for (int fs = 0; fs < FS; ++fs) kf[fs] = TP::row8(sm.pk, kj, 32 * fs + 8 * g);
            for (int it = grp; it < 4; it += WS) {
                f32x4 acc = {0, 0, 0, 0};
                if (it >= wq) {
#pragma unroll
                    for (int fs = 0; fs < FS; ++fs)
                        acc = T::mma(TP::row8(sm.pq, 16 * it + col, 32 * fs + 8 * g), kf[fs], acc);
                }
                f32x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = 16 * it + 4 * g + i >= kj ? acc[i] : 0.f;
                store4<T>(&sm.mt[kj][16 * it + 4 * g], v);
            }
        }
        __syncthreads();
        f32x4 accs[4][DW];
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int j = 0; j < DW; ++j) accs[kt][j] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int fs = 0; fs < FS; ++fs) {
            F shi[DW], slo[DW];
#pragma unroll
            for (int j = 0; j < DW; ++j) {
                float sv[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sv[i] = S[2 * fs][j][i];
                    sv[4 + i] = S[2 * fs + 1][j][i];
                }
                T::split(sv, shi[j], slo[j]);
            }
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                const F bf = TP::row44(sm.pk, 16 * kt + col, 32 * fs + 4 * g);
#pragma unroll
                for (int j = 0; j < DW; ++j) {
                    accs[kt][j] = T::mma(shi[j], bf, accs[kt][j]);
                    if (T::kSplit) accs[kt][j] = T::mma(slo[j], bf, accs[kt][j]);
                }
            }
        }
        // dV^T: lane (g, col) holds d = 16 (w DW + j) + 4 g + i of key 16 kt + col
        F bv[2][DW];                     // (dNum / L)^T operands: the intra-chunk part and the state update
        if constexpr (CAUSAL) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int j = 0; j < DW; ++j) bv[kk][j] = TV::col8(sm.dn, 32 * kk, 16 * (w * DW + j), tx);
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) {
                    const F bf = T::ld8(&sm.mt[16 * kt + col][32 * kk + 8 * g]);
#pragma unroll
                    for (int j = 0; j < DW; ++j) accs[kt][j] = T::mma(bv[kk][j], bf, accs[kt][j]);
                }
            }
        }
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            const int tok = t0 + 16 * kt + col;
            if (tok < a.N)
#pragma unroll
                for (int j = 0; j < DW; ++j) store4<T>(out + (size_t)tok * D + 16 * (w * DW + j) + 4 * g, accs[kt][j]);
        }
        if constexpr (CAUSAL) {
            // dS += Phi_Q' (dNum / L) (chunk)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int ft = 0; ft < RP / 16; ++ft) {
                    const F af = TP::col8(sm.pq, 32 * kk, 16 * ft, tx);
#pragma unroll
                    for (int j = 0; j < DW; ++j) S[ft][j] = T::mma(af, bv[kk][j], S[ft][j]);
                }
            }
        }
    }
}

// The three passes in one launch: they depend on the states only, so one
// pass's workgroups start in the places the previous one's leave (three
// launches left three partly filled last rounds and two gaps: 16K 243 + 7 us
// with W' apart, 223 us together; 4096 tokens x 16 heads 37 + 8 against 24).
// Pass after pass, not interleaved: with the passes of a segment side by side
// the compute units fetch three loops' instructions in turn (253 us at 16K),
// which costs more than their shared rows in L2 save.  W' for the sparse
// epilogues is formed by a few workgroups at the end of the grid.
// 256 features keep dV on its own: its state takes a whole compute unit's
// registers, which would halve the dQ and dK workgroups in flight.
template <int RP> constexpr bool dv_joins() { return RP < 256; }

template <class T, int D, int RP, bool CAUSAL>
__global__ __launch_bounds__(kThreads, 2) void race_bwd_kernel(LbArgs a)
{
    constexpr int SPLIT = table_split<RP>(), ROLES = 2 * SPLIT + (dv_joins<RP>() ? 1 : 0);
    constexpr bool DV = dv_joins<RP>();
    __shared__ __attribute__((aligned(16))) union {
        Lb1Smem<T, D, RP / SPLIT, CAUSAL> q;
        Lb2Smem<T, D, RP / SPLIT, CAUSAL> k;
        typename std::conditional<DV, Lb3Smem<T, D, RP, CAUSAL>, char>::type v;
    } sm;
    const int role = blockIdx.x / a.items, item = blockIdx.x - role * a.items;
    if (role >= ROLES) {
        wt_body<T>(a, blockIdx.x - ROLES * a.items, D, w_kdim<RP>());
        return;
    }
    const int seg = item % a.nseg;
    const size_t bh = item / a.nseg;
    if (role < SPLIT) race_dq_body<T, D, RP, CAUSAL>(a, bh, seg, role, sm.q);
    else if (role < 2 * SPLIT) race_dk_body<T, D, RP, CAUSAL>(a, bh, seg, role - SPLIT, sm.k);
    else if constexpr (DV) race_dv_body<T, D, RP, CAUSAL>(a, bh, seg, sm.v);
}

template <class T, int D, int RP, bool CAUSAL>
__global__ __launch_bounds__((state_waves<D, RP>() * 64), (state_waves<D, RP>() / 4)) void race_dv_kernel(LbArgs a)
{
    __shared__ __attribute__((aligned(16))) Lb3Smem<T, D, RP, CAUSAL> sm;
    race_dv_body<T, D, RP, CAUSAL>(a, blockIdx.y, blockIdx.x, sm);
}

template <class T, int D, int RP>
struct BwdFn {
    static hipError_t run(const Shape& s, const LbArgs& a, hipStream_t st)
    {
        if constexpr (!bwd_fits<T, D, RP>()) {
            return hipErrorInvalidConfiguration;
        } else {
            constexpr int ROLES = 2 * table_split<RP>() + (dv_joins<RP>() ? 1 : 0);
            const int wt = (s.H * D * w_kdim<RP>() + kWtPer - 1) / kWtPer;   // W' rides along
            if (a.causal) ELSAA_LAUNCH("race_bwd", (race_bwd_kernel<T, D, RP, true>), dim3(a.items * ROLES + wt), dim3(kThreads), 0, st, a);
            else ELSAA_LAUNCH("race_bwd", (race_bwd_kernel<T, D, RP, false>), dim3(a.items * ROLES + wt), dim3(kThreads), 0, st, a);
            hipError_t e = hipGetLastError();
            if constexpr (!dv_joins<RP>()) {
                if (e != hipSuccess) return e;
                if (a.causal) ELSAA_LAUNCH("race_dv", (race_dv_kernel<T, D, RP, true>), dim3(s.nseg, s.H * s.B), dim3(state_waves<D, RP>() * 64), 0, st, a);
                else ELSAA_LAUNCH("race_dv", (race_dv_kernel<T, D, RP, false>), dim3(s.nseg, s.H * s.B), dim3(state_waves<D, RP>() * 64), 0, st, a);
                e = hipGetLastError();
            }
            return e;
        }
    }
};

template <class T, int D, int RP>
struct BwdFitsFn {
    static hipError_t run(const Shape&) { return bwd_fits<T, D, RP>() ? hipSuccess : hipErrorInvalidConfiguration; }
};

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

}  // namespace

bool race_bwd_fits(const Shape& s) { return dispatch<BwdFitsFn>(s) == hipSuccess; }

size_t race_wt_bytes(const Shape& s)
{
    const int rp = race_padded_features(s.r);
    const size_t wk = rp / 4 < 32 ? 32 : rp / 4;
    return (size_t)s.H * s.D * wk * (s.bf16 ? 2 : 4);
}

int race_wk(const Shape& s)
{
    const int rp = race_padded_features(s.r);
    return rp / 4 < 32 ? 32 : rp / 4;
}

hipError_t launch_race_bwd(const Shape& s, const float* Uq, const float* Uk, const void* V,
                           const void* dO, const float* W_race, const float* rs,
                           const float* states_f, const float* states_b, void* wt_hi, void* wt_lo,
                           void* du_q, void* du_k, void* dv_lr, hipStream_t st)
{
    const size_t BHN = (size_t)s.B * s.H * s.N;
    LbArgs a;
    a.Uq = Uq; a.Uk = Uk; a.V = V; a.dO = dO; a.rs = rs;
    a.W = W_race; a.wt_hi = wt_hi; a.wt_lo = wt_lo; a.items = s.B * s.H * s.nseg;
    a.H = s.H; a.N = s.N; a.L = s.L; a.seg_len = s.seg_len; a.nseg = s.nseg; a.causal = s.causal;
    a.BHN = BHN;
    a.two_beta = 2.f * s.beta; a.inv_L = 1.f / (float)s.L;
    a.states_f = states_f; a.states_b = states_b;
    a.du_q = du_q; a.du_k = du_k; a.dv = dv_lr;
    return dispatch<BwdFn>(s, a, st);
}

}  // namespace elsaa
