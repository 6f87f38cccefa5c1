// bwd_rows.hpp -- per-row scalars of the backward.
//
// For u = dO_i, with O = g_s m O_s + g_lr O_lr, m = d_s / D, D = d_s + lambda Den + eps,
// O_s = N_s / (d_s + eps), O_lr = Num / (Den + eps):
//   dm    = g_s <O_s, u>                      (dm / d log d_s = m (1 - m))
//   sc_s  = g_s m                             (dO_s = sc_s u)
//   Delta = sc_s <u, O_s> - dm m (1 - m)(d_s + eps) / d_s
//   sc_lr = g_lr / (Den + eps)                (dNum = sc_lr u)
//   dDen  = -g_lr <u, O_lr> / (Den + eps) - dm m lambda / D
//   dg_s  = m <O_s, u>,  dg_lr = <O_lr, u>,  dlambda = -dm m Den / D
// (lambda per token when given; with m fixed to 1 every dm term is zero).
// Stored as rs[f][BHN] with f = 0: log2(d_s + eps), 1: Delta, 2: sc_s,
// 3: sc_lr, 4: dDen.
#pragma once
#include "common.hpp"

namespace elsaa {

struct RowArgs {
    const float* Os;        // float32 [BHN][D]
    const void* Olr;        // storage dtype [BHN][D]
    const float* m;
    const float* lse;
    const float* dlr;
    const float* gates;     // [BHN][2] or null
    const float* lam_rows;  // or null
    float* rs;
    float* dg;              // [BHN][2] or null
    float* dlam;            // or null
    size_t BHN;
    float lambda, eps;
    int m_one;
};

// The row's inputs besides the two dot products.
struct RowIn {
    float gs, gl, m, lse, den, lam;
    __device__ __forceinline__ void load(const RowArgs& a, size_t row)
    {
        gs = a.gates ? a.gates[row * 2] : 1.f;
        gl = a.gates ? a.gates[row * 2 + 1] : 1.f;
        m = a.m[row];
        lse = a.lse[row];
        den = a.dlr[row];
        lam = a.lam_rows ? a.lam_rows[row] : a.lambda;
    }
};

// Writes the scalars of `row` from uos = <u, O_s> and uol = <u, O_lr>; returns dDen.
__device__ __forceinline__ float row_scalars(const RowArgs& a, size_t row, const RowIn& in, float uos, float uol)
{
    const float mi = in.m, ls = in.lse, den = in.den;
    const float rel = a.eps * __expf(fminf(-ls, 80.f));   // eps / d_s
    const float dm = a.m_one ? 0.f : in.gs * uos;
    const float scs = in.gs * mi;
    const float delta = scs * uos - dm * mi * (1.f - mi) * (1.f + rel);
    const float inv_den = 1.f / (den + a.eps);
    const float Dtot = __expf(fminf(ls, 80.f)) + in.lam * den + a.eps;
    const float dden = -in.gl * uol * inv_den - dm * mi * in.lam / Dtot;
    a.rs[row] = (ls + log1pf(rel)) * kLog2e;
    a.rs[a.BHN + row] = delta;
    a.rs[2 * a.BHN + row] = scs;
    a.rs[3 * a.BHN + row] = in.gl * inv_den;
    a.rs[4 * a.BHN + row] = dden;
    if (a.dg) {
        a.dg[row * 2] = mi * uos;
        a.dg[row * 2 + 1] = uol;
    }
    if (a.dlam) a.dlam[row] = -dm * mi * den / Dtot;
    return dden;
}

}  // namespace elsaa
