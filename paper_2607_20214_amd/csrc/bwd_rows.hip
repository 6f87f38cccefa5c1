// bwd_rows.hip -- the backward's per-row scalars (bwd_rows.hpp) as a pass of
// their own, 16 lanes per row (short calls form them in the backward's state
// pass, race_fwd.hip).
#include "bwd_rows.hpp"
#include "internal.hpp"

namespace elsaa {

namespace {

template <class T, int D>
__global__ __launch_bounds__(256) void bwd_rows_kernel(const typename T::store_t* __restrict__ dO, RowArgs a)
{
    constexpr int PL = D / 16;   // elements per lane
    const size_t row = (size_t)blockIdx.x * 16 + threadIdx.x / 16;
    const int sub = threadIdx.x & 15;
    if (row >= a.BHN) return;   // whole 16-lane groups leave together
    float uos = 0.f, uol = 0.f;
    const size_t base = row * D + sub * PL;
    const typename T::store_t* Olr = (const typename T::store_t*)a.Olr;
#pragma unroll
    for (int e = 0; e < PL; e += 4) {
        const f32x4 u = load4<T>(dO + base + e), xs = *(const f32x4*)(a.Os + base + e), xl = load4<T>(Olr + base + e);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uos += u[i] * xs[i];
            uol += u[i] * xl[i];
        }
    }
    uos = row_sum16(uos);
    uol = row_sum16(uol);
    if (sub != 0) return;
    RowIn in;
    in.load(a, row);
    row_scalars(a, row, in, uos, uol);
}

}  // namespace

hipError_t launch_bwd_rows(const Shape& s, const void* dO, const RowArgs& a, hipStream_t st)
{
    dim3 grid((unsigned)((a.BHN + 15) / 16));
#define ELSAA_ROWS(T_, D_)                                                                       \
    ELSAA_LAUNCH("bwd_rows", (bwd_rows_kernel<T_, D_>), grid, dim3(256), 0, st, (const T_::store_t*)dO, a)
    if (s.bf16) {
        if (s.D == 64) ELSAA_ROWS(BF16, 64);
        else ELSAA_ROWS(BF16, 128);
    } else {
        if (s.D == 64) ELSAA_ROWS(F32, 64);
        else ELSAA_ROWS(F32, 128);
    }
#undef ELSAA_ROWS
    return hipGetLastError();
}

}  // namespace elsaa
