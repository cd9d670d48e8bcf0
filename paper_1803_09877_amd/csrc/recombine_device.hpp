// The recombination u = R_{.,U} b (Algorithm 1, line 4) of one lane's columns, for the kernels that run it.
#pragma once

#include "device_util.hpp"
#include "wave_reduce.hpp"

namespace draco {
namespace {

// sum += sum over q < cnt of b_q * (row idx_q) at the lane's two complex columns: honest rows in ascending node order, in
// fp64.  Lane l of the wavefront holds the index and the coefficient of the l-th of at most 64 rows (a scalar load for each
// row would be waited for one by one, half of the time on short rows).  UN rows in flight; no load is under a
// condition (cyc_project_body): with the last round's under one, rows of no more than two rounds, a dozen nodes, had all of
// theirs there ((12, 2, 2 M), one word: 21.2 us, 18.0 so).
template <bool FULL, int LO, int UN, bool NT>
__device__ __forceinline__ void add_rows(const float* __restrict__ Rm, const float* __restrict__ Rlo, int64_t ldm, int my_row,
                                         double2 my_b, int cnt, int64_t c0, int nin, double (&sum)[4]) {
    float4 x[UN];
    lo_raw_t<LO> xl[LO != kLoNone ? UN : 1];
    auto fetch = [&](int slot, int q) {
        const int64_t off = (int64_t)__builtin_amdgcn_readlane(my_row, q) * ldm + c0;
        x[slot] = ldx<FULL, NT>(Rm + off, nin);
        if constexpr (LO != kLoNone) xl[slot] = ld_lo<FULL, LO, NT>(Rlo, off, nin);
    };
    auto use = [&](int slot, int q) {
        const double br = lane_value(my_b.x, q), bi = lane_value(my_b.y, q);
        const wire4 v = wire_value<LO>(x[slot], xl[LO != kLoNone ? slot : 0]);
        cmac(br, bi, v.x, v.y, sum[0], sum[1]);
        cmac(br, bi, v.z, v.w, sum[2], sum[3]);
    };
#pragma unroll
    for (int i = 0; i < UN; ++i) fetch(i, min(i, cnt - 1));
    int q = 0;
    for (; q + UN < cnt; q += UN) {   // (behind the last row it is read again)
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            use(i, q + i);
            fetch(i, min(q + UN + i, cnt - 1));
        }
    }
#pragma unroll
    for (int i = 0; i < UN; ++i) {
        if (q + i < cnt) use(i, q + i);
    }
}

// One rounding to fp32.  realout: unpacked wire, the sum is the real part, one float per complex entry.
template <bool FULL>
__device__ __forceinline__ void store_sum(float* __restrict__ u, bool realout, int64_t d, int64_t c0, const double (&sum)[4]) {
    if (realout) {
        const int64_t c = c0 / 2;
        if (FULL || 2 * c < d) u[c] = (float)sum[0];
        if (FULL || 2 * c + 2 < d) u[c + 1] = (float)sum[2];
    } else {
        stx<FULL>(u + c0, make_float4((float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]), FULL ? 4 : clamp4(d - c0));
    }
}

}  // namespace
}  // namespace draco
