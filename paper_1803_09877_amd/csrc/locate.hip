// phi and the recombination vector on the device: the kernels around locate_device.hpp.
#include "locate_device.hpp"

#include <cmath>

namespace draco {

namespace {

constexpr int kSumWaves = 8;   // wavefronts that add partial sums before the first one locates

// sm.gam <- sums[P] (tiles == 0, one wavefront), or the sum over t < tiles of sums[t][P] (kSumWaves of them): each
// wavefront adds every kSumWaves-th tile, then their sums are added in order.
__device__ __forceinline__ void load_projections(LocateSmem& sm, double2 (*part)[kMaxNodes],
                                                 const double2* __restrict__ sums, int tiles,
                                                 const double2* __restrict__ roots, int P) {
    const int wave = threadIdx.x / kW, lane = threadIdx.x % kW;
    if (tiles == 0) {
        for (int j = lane; j < P; j += kW) {
            sm.gam[j] = sums[j];
            sm.root[j] = roots[j];
        }
        wave_sync();
        return;
    }
    for (int j = lane; j < P; j += kW) {
        double2 a = make_double2(0.0, 0.0);
#pragma unroll 8
        for (int t = wave; t < tiles; t += kSumWaves) {
            const double2 p = sums[(int64_t)t * P + j];
            a.x += p.x;
            a.y += p.y;
        }
        part[wave][j] = a;
    }
    for (int j = threadIdx.x; j < P; j += kW * kSumWaves) sm.root[j] = roots[j];
    __syncthreads();
    for (int j = threadIdx.x; j < P; j += kW * kSumWaves) {
        double2 a = part[0][j];
#pragma unroll
        for (int w = 1; w < kSumWaves; ++w) {
            a.x += part[w][j].x;
            a.y += part[w][j].y;
        }
        sm.gam[j] = a;
    }
    __syncthreads();
}

}  // namespace

// One kernel for the sample's locator and the last one, so that the second of a decode finds the code
// in the instruction cache (0.3 to 0.5 % of a step with a sample, little more than runs differ; the rest is its chain of
// dependent steps, locate_device.hpp).
// CH: chunks of 64 nodes.
template <int CH>
__global__ __launch_bounds__(kW * kSumWaves) void cyc_locate_kernel(
    const double2* __restrict__ sums, int tiles, const double2* __restrict__ roots, int P, int s, double tau,
    double isq, const double2* __restrict__ b0, const CycSpec spec, const LocateOut out, int sample) {
    if (sample != 0 && !takes_sample(spec)) return;
    __shared__ LocateSmem sm;
    __shared__ double2 part[kSumWaves][kMaxNodes];
    load_projections(sm, part, sums, tiles, roots, P);
    if (threadIdx.x >= kW) return;
    const int lane = threadIdx.x;
    NodeSet<CH> flagged;
    const bool clean = locate_wave<CH>(sm, P, s, tau, isq, b0, out, lane, flagged);
    if (sample == 0 && spec.state != nullptr) {
        // the flagged nodes are the ones speculated on
        const int now = spec.state[kSpecNow];
        bool same = now != 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (c * kW < P) same &= flagged.word[c] == (now == kSpecOnSample ? spec.mask[c] : 0ull);
        }
        if (lane == 0) {
            spec.state[kSpecDone] = same ? 1 : 0;
            if (spec.mask != nullptr) {
                const int skip = spec.state[kSpecSkip];
                if (takes_sample(spec)) {
                    if (!same) {   // misled (or its locator failed): project only, longer each time
                        const int misses = min(spec.state[kSpecMisses] + 1, kMaxMisses);
                        spec.state[kSpecMisses] = misses;
                        spec.state[kSpecSkip] = (1 << misses) - 1;
                    } else if (!clean) {
                        spec.state[kSpecMisses] = 0;
                    }
                } else if (skip > 0) {
                    spec.state[kSpecSkip] = skip - 1;
                }
            }
            spec.state[kSpecClean] = clean ? min(spec.state[kSpecClean] + 1, kCleanRun) : 0;
        }
    }
}

static void launch(int threads, const double2* sums, int tiles, const double2* roots, int P, int s, double tau,
                   const double2* b0, const CycSpec& spec, const LocateOut& out, bool sample, hipStream_t stream) {
    const double isq = 1.0 / std::sqrt((double)P);
    auto go = [&](auto chunks) {
        hipLaunchKernelGGL((cyc_locate_kernel<decltype(chunks)::value>), dim3(1), dim3(threads), 0, stream, sums, tiles, roots, P,
                           s, tau, isq, b0, spec, out, sample ? 1 : 0);
    };
    if (P <= kW) go(std::integral_constant<int, 1>());
    else go(std::integral_constant<int, kMaxNodes / kW>());
}

hipError_t launch_cyc_locate(const double2* sums, int64_t tiles, const double2* roots, int P, int s, double tau,
                             const double2* b0, uint64_t* mask_out, int32_t* status_out, double2* b_out,
                             int32_t* idx_out, int32_t* nu_out, const CycSpec& spec, hipStream_t stream) {
    const LocateOut out{mask_out, status_out, b_out, idx_out, nu_out, nullptr};
    launch(tiles > 0 ? kW * kSumWaves : kW, sums, (int)tiles, roots, P, s, tau, b0, spec, out, false, stream);
    return hipGetLastError();
}

hipError_t launch_cyc_locate_sample(const double2* partial, const double2* roots, int P, int s, double tau,
                                    const double2* b0, double2* b_out, int32_t* idx_out, int32_t* nu_out,
                                    const CycSpec& spec, hipStream_t stream) {
    const LocateOut out{spec.mask, spec.state + kSpecStatus, b_out, idx_out, nu_out, spec.b};
    launch(kW * kSumWaves, partial, (int)kSampleTiles, roots, P, s, tau, b0, spec, out, true, stream);
    return hipGetLastError();
}

}  // namespace draco
