// Cross-lane sums and maxima of doubles on a 64-lane wavefront without LDS: DPP moves inside a
// row of 16 lanes, v_permlane16/32_swap between rows.  All 64 lanes must be active.
#pragma once

#include <hip/hip_runtime.h>

namespace draco {
namespace {

// The value that lane q (the same in every lane) holds.
__device__ __forceinline__ double lane_value(double v, int q) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), q), __builtin_amdgcn_readlane(__double2loint(v), q));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    // every lane reads a lane of its own row of 16, or 0 behind its end, so no previous value is kept (mov_dpp): one
    // instruction per word
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
constexpr int kDppXor1 = 0xB1;         // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7 - i within each 8 lanes
constexpr int kDppRor8 = 0x128;        // lane i <-> i ^ 8 within each 16 lanes
constexpr int kDppShl1 = 0x101;        // lane i <- i + 1 within each 16 lanes, 0 into the last

// Swaps lanes 32-63 of a with lanes 0-31 of b (WIDTH = 32), or the odd rows of 16 lanes of a with
// the even rows of b (WIDTH = 16).
template <int WIDTH>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
    static_assert(WIDTH == 32 || WIDTH == 16, "lane halves or rows");
    const unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
    const unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
    if constexpr (WIDTH == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
        a = __hiloint2double((int)h[0], (int)l[0]);
        b = __hiloint2double((int)h[1], (int)l[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
        a = __hiloint2double((int)h[0], (int)l[0]);
        b = __hiloint2double((int)h[1], (int)l[1]);
    }
}
// Lanes whose bit WIDTH is clear receive a + (a of the lane with that bit set), the others the
// same of b.
template <int WIDTH>
__device__ __forceinline__ double swap_add(double a, double b) {
    lane_swap<WIDTH>(a, b);
    return a + b;
}

// Sum and maximum over aligned groups of N lanes; every lane of a group receives the result,
// bit-identical across the group.
template <int N>
__device__ __forceinline__ double group_sum(double v) {
    if constexpr (N >= 2) v += dpp_move<kDppXor1>(v);
    if constexpr (N >= 4) v += dpp_move<kDppXor2>(v);
    if constexpr (N >= 8) v += dpp_move<kDppHalfMirror>(v);   // quads are uniform by now
    if constexpr (N >= 16) v += dpp_move<kDppRor8>(v);
    if constexpr (N >= 32) v = swap_add<16>(v, v);
    if constexpr (N >= 64) v = swap_add<32>(v, v);
    return v;
}
// The same for several values, a step of all of them before the next: one wavefront issues in order, and a step is three
// dependent instructions.
template <int N, int M>
__device__ __forceinline__ void group_sums(double (&v)[M]) {
    if constexpr (N >= 2) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += dpp_move<kDppXor1>(v[i]);
    }
    if constexpr (N >= 4) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += dpp_move<kDppXor2>(v[i]);
    }
    if constexpr (N >= 8) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += dpp_move<kDppHalfMirror>(v[i]);
    }
    if constexpr (N >= 16) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += dpp_move<kDppRor8>(v[i]);
    }
    if constexpr (N >= 32) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] = swap_add<16>(v[i], v[i]);
    }
    if constexpr (N >= 64) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] = swap_add<32>(v[i], v[i]);
    }
}
template <int N>
__device__ __forceinline__ double group_max(double v) {
    if constexpr (N >= 2) v = fmax(v, dpp_move<kDppXor1>(v));
    if constexpr (N >= 4) v = fmax(v, dpp_move<kDppXor2>(v));
    if constexpr (N >= 8) v = fmax(v, dpp_move<kDppHalfMirror>(v));
    if constexpr (N >= 16) v = fmax(v, dpp_move<kDppRor8>(v));
    if constexpr (N >= 32) {
        double w = v;
        lane_swap<16>(v, w);
        v = fmax(v, w);
    }
    if constexpr (N >= 64) {
        double w = v;
        lane_swap<32>(v, w);
        v = fmax(v, w);
    }
    return v;
}

// Sums N values (a power of two, 2 .. 16) over the 64 lanes together; lane l returns the sum of
// value l / (64 / N).  A step that halves the lanes a sum is spread over also halves the sums a
// lane holds, so N sums cost about N + 6 exchanges instead of 6 N.
template <int N>
__device__ __forceinline__ double reduce_over_wave(const double (&v)[N]) {
    static_assert(N == 2 || N == 4 || N == 8 || N == 16, "a power of two up to 16");
    const int lane = threadIdx.x & 63;
    double w[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) w[i] = swap_add<32>(v[i], v[i + N / 2]);
    if constexpr (N >= 4) {
#pragma unroll
        for (int i = 0; i < N / 4; ++i) w[i] = swap_add<16>(w[i], w[i + N / 4]);
    } else {
        w[0] = swap_add<16>(w[0], w[0]);
    }
    if constexpr (N >= 8) {   // lanes with bit 3 keep the upper half of the values
        const bool up = (lane & 8) != 0;
#pragma unroll
        for (int i = 0; i < N / 8; ++i) {
            const double give = up ? w[i] : w[i + N / 8], keep = up ? w[i + N / 8] : w[i];
            w[i] = keep + dpp_move<kDppRor8>(give);
        }
    } else {
        w[0] += dpp_move<kDppRor8>(w[0]);
    }
    if constexpr (N >= 16) {
        const bool up = (lane & 4) != 0;
        const double give = up ? w[0] : w[1], keep = up ? w[1] : w[0];
        w[0] = keep + dpp_move<kDppHalfMirror>(give);
        w[0] += dpp_move<kDppXor1>(w[0]);
        w[0] += dpp_move<kDppXor2>(w[0]);
    } else {
        w[0] += dpp_move<kDppXor1>(w[0]);
        w[0] += dpp_move<kDppXor2>(w[0]);
        w[0] += dpp_move<kDppHalfMirror>(w[0]);   // quads are uniform by now
    }
    return w[0];
}

}  // namespace
}  // namespace draco
