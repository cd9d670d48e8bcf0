// phi and the recombination vector on the device: the kernels around locate_device.hpp.
#include "device_util.hpp"
#include "locate_device.hpp"
#include "recombine_device.hpp"

#include <algorithm>
#include <cmath>

namespace draco {

namespace {

constexpr int kSumWaves = 8;   // wavefronts that add partial sums before the first one locates

// Where a located set goes.
struct LocateOut {
    uint64_t* mask;      // ceil(P/64) words
    int32_t* status;
    double2* b;          // honest nodes' coefficients, one behind the other
    int32_t* idx;        // and their indices
    int32_t* nu;         // how many
    double2* dense;      // the coefficients by node (flagged ones untouched), or nullptr
};

// sm.gam <- sums[P] (tiles == 0, one wavefront), or the sum over t < tiles of sums[t][P] (W wavefronts): each adds every
// W-th tile, then their sums are added in order.
template <int W>
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
#pragma unroll 16
        for (int t = wave; t < tiles; t += W) {
            const double2 p = sums[(int64_t)t * P + j];
            a.x += p.x;
            a.y += p.y;
        }
        part[wave][j] = a;
    }
    for (int j = threadIdx.x; j < P; j += kW * W) sm.root[j] = roots[j];
    __syncthreads();
    for (int j = threadIdx.x; j < P; j += kW * W) {
        double2 a = part[0][j];
#pragma unroll
        for (int w = 1; w < W; ++w) {
            a.x += part[w][j].x;
            a.y += part[w][j].y;
        }
        sm.gam[j] = a;
    }
    __syncthreads();
}

}  // namespace

// Whether the flagged nodes are the ones that the projection speculated on: the output then holds the sum already.
template <int CH>
__device__ __forceinline__ bool holds_speculation(const CycSpec& spec, const Located<CH>& found, int P) {
    const int now = spec.state[kSpecNow];
    bool same = now != 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (c * kW < P) same &= found.flagged.word[c] == (now == kSpecOnSample ? spec.mask[c] : 0ull);
    }
    return same;
}
// What the next call expects.
template <int CH>
__device__ __forceinline__ void note_outcome(const CycSpec& spec, const Located<CH>& found, bool same, int lane) {
    if (lane != 0) return;
    const bool clean = found.clean();
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
    load_projections<kSumWaves>(sm, part, sums, tiles, roots, P);
    if (threadIdx.x >= kW) return;
    const int lane = threadIdx.x;
    const Located<CH> found = locate_wave<CH>(sm, P, s, tau, isq, b0, lane);
    int nu = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {   // the honest nodes, one behind the other in ascending order
        if (c * kW >= P) break;
        const int j = c * kW + lane;
        const bool honest = j < P && !found.flagged.has(c, lane);
        const unsigned long long bal = __ballot(honest);
        if (honest) {
            const int pos = nu + __popcll(bal & ((1ull << lane) - 1ull));
            out.idx[pos] = j;
            out.b[pos] = found.b[c];
            if (out.dense != nullptr) out.dense[j] = found.b[c];
        }
        if (lane == 0) out.mask[c] = found.flagged.word[c];
        nu += __popcll(bal);
    }
    if (lane == 0) {
        *out.nu = nu;
        *out.status = found.status;
    }
    if (sample == 0 && spec.state != nullptr) note_outcome(spec, found, holds_speculation(spec, found, P), lane);
}

// The locator and the recombination of short rows in one launch (a launch behind another is 4 us): every
// workgroup runs the locator for itself, with its first rows already in flight, and adds its columns with the coefficients
// out of LDS.  A workgroup owns 1 KiB of the rows, its eight wavefronts take every eighth row, kAhead in flight,
// and their sums are added in order.  Decodes in us, two launches and one: (45, 3, 30 000) on the 5-byte wire, nobody and
// three lie, 13.9 / 11.6 and 17.3 / 14.8, (20, 4, 10 001) 13.8 / 11.0 and 15.8 / 14.3, (45, 7, 65 000) on the 6-byte one 18.6 /
// 14.2 and 26.9 / 23.3.  Beyond 64 tiles, more KiB than CUs, it gains nothing ((45, 3, 180 000): 24.5 and 24.6 us).
constexpr int kAhead = 6;
template <int LO>
struct ShortRows {
    float4 x[kAhead];
    lo_raw_t<LO> xl[LO != kLoNone ? kAhead : 1];
    template <bool FULL>
    __device__ __forceinline__ void load(const float* __restrict__ Rm, const float* __restrict__ Rlo, int64_t ldm, int64_t c0,
                                         int nin, int first, int P) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {   // (behind the last row it is read again)
            const int64_t off = (int64_t)min(first + i * kSumWaves, P - 1) * ldm + c0;
            x[i] = ldx<FULL, false>(Rm + off, nin);
            if constexpr (LO != kLoNone) xl[i] = ld_lo<FULL, LO, false>(Rlo, off, nin);
        }
    }
    __device__ __forceinline__ void add(const double2* b, const uint64_t* flagged, int first, int P, double (&sum)[4]) const {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const int j = first + i * kSumWaves;
            if (j < P && ((flagged[j >> 6] >> (j & 63)) & 1ull) == 0) {   // (a liar's words may be no numbers)
                const double2 bj = b[j];
                const wire4 v = wire_value<LO>(x[i], xl[LO != kLoNone ? i : 0]);
                cmac(bj.x, bj.y, v.x, v.y, sum[0], sum[1]);
                cmac(bj.x, bj.y, v.z, v.w, sum[2], sum[3]);
            }
        }
    }
};
template <int LO, int CH>
__global__ __launch_bounds__(kW * kSumWaves) void cyc_locate_recombine_kernel(
    const double2* __restrict__ sums, int tiles, const double2* __restrict__ roots, int P, int s, double tau, double isq,
    const double2* __restrict__ b0, uint64_t* __restrict__ mask, int32_t* __restrict__ status, const float* __restrict__ Rm,
    const float* __restrict__ Rlo, int64_t ldm, float* __restrict__ u, int realout, int64_t d) {
    __shared__ LocateSmem sm;
    __shared__ union {
        double2 tile_sums[kSumWaves][kMaxNodes];
        double row_sums[kSumWaves][4][kW];
    } part;
    __shared__ double2 b[kMaxNodes];
    __shared__ uint64_t flagged[kMaskWords];
    const int lane = threadIdx.x % kW, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kW);
    const int64_t mlen = 2 * ((d + 1) / 2), c0 = ((int64_t)blockIdx.x * kW + lane) * 4;
    ShortRows<LO> rows;
    auto fetch = [&](int first) {
        if ((int64_t)(blockIdx.x + 1) * (kW * 4) <= d) rows.template load<true>(Rm, Rlo, ldm, c0, 4, first, P);
        else rows.template load<false>(Rm, Rlo, ldm, c0, clamp4(mlen - c0), first, P);
    };
    if constexpr (CH == 1) fetch(wave);   // (four chunks leave no registers for them)
    load_projections<kSumWaves>(sm, part.tile_sums, sums, tiles, roots, P);
    if (wave == 0) {
        const Located<CH> found = locate_wave<CH>(sm, P, s, tau, isq, b0, lane);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (c * kW + lane < P) b[c * kW + lane] = found.b[c];
            if (lane == 0) flagged[c] = found.flagged.word[c];
            if (lane == 0 && blockIdx.x == 0 && c * kW < P) mask[c] = found.flagged.word[c];
        }
        if (lane == 0 && blockIdx.x == 0) *status = found.status;
    }
    __syncthreads();
    if constexpr (CH != 1) fetch(wave);
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    rows.add(b, flagged, wave, P, sum);
    for (int first = wave + kAhead * kSumWaves; first < P; first += kAhead * kSumWaves) {
        fetch(first);
        rows.add(b, flagged, first, P, sum);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) part.row_sums[wave][i][lane] = sum[i];
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < kSumWaves; ++w) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] += part.row_sums[w][i][lane];
    }
    store_sum<false>(u, realout != 0, d, c0, sum);
}

// The same for longer rows of messages that stay in the memory-side cache: every workgroup runs the locator, and if the output
// does not hold the sum yet, they walk over the rows together, two of them per CU.  Decodes in us, two launches and one: (45, 3, 500 000) on the 5-byte wire, nobody and three
// lie, 30.2 / 29.0 and 51.1 / 49.4; (15, 2, 1 M) on one word 21.7 / 20.1 and 33.7 / 30.9, unpacked 48.6 / 45.6; (45, 3,
// 1 M) on the 6-byte wire 51.8 / 50.9 and 93.5 / 89.7.
template <int LO, int UN>
__global__ __launch_bounds__(kBlock, 2) void cyc_locate_walk_kernel(
    const double2* __restrict__ sums, int tiles, const double2* __restrict__ roots, int P, int s, double tau, double isq,
    const double2* __restrict__ b0, uint64_t* __restrict__ mask, int32_t* __restrict__ status, const CycSpec spec,
    const float* __restrict__ Rm, const float* __restrict__ Rlo, int64_t ldm, float* __restrict__ u, int realout,
    unsigned blocks, int64_t d) {
    __shared__ LocateSmem sm;
    __shared__ double2 part[kBlock / kW][kMaxNodes];
    __shared__ double2 b[kW];
    __shared__ int idx[kW];
    __shared__ int honest_rows;   // -1: the output holds their sum already
    const int lane = threadIdx.x % kW;
    load_projections<kBlock / kW>(sm, part, sums, tiles, roots, P);
    if (threadIdx.x < kW) {
        const Located<1> found = locate_wave<1>(sm, P, s, tau, isq, b0, lane);
        const bool honest = lane < P && !found.flagged.has(0, lane);
        const unsigned long long bal = __ballot(honest);
        if (honest) {
            const int pos = __popcll(bal & ((1ull << lane) - 1ull));
            idx[pos] = lane;
            b[pos] = found.b[0];
        }
        const bool done = spec.state != nullptr && holds_speculation(spec, found, P);
        if (lane == 0) honest_rows = done ? -1 : __popcll(bal);
        if (blockIdx.x == 0) {
            if (lane == 0) {
                mask[0] = found.flagged.word[0];
                *status = found.status;
            }
            if (spec.state != nullptr) note_outcome(spec, found, done, lane);
        }
    }
    __syncthreads();
    const int cnt = __builtin_amdgcn_readfirstlane(honest_rows);
    if (cnt < 0) return;
    if (cnt == 0) {   // every message is broken: a sum of nothing
        const double none[4] = {0.0, 0.0, 0.0, 0.0};
        for (unsigned block = blockIdx.x; block < blocks; block += gridDim.x)
            store_sum<false>(u, realout != 0, d, lane_column<kSpreadRecombine>(d, blocks, block), none);
        return;
    }
    const int mine = min(lane, cnt - 1), my_row = idx[mine];
    const double2 my_b = b[mine];
    for (unsigned block = blockIdx.x; block < blocks; block += gridDim.x) {
        const int64_t c0 = lane_column<kSpreadRecombine>(d, blocks, block);
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
        if (block_is_full<kSpreadRecombine>(d, d, blocks, block)) {
            add_rows<true, LO, UN, false>(Rm, Rlo, ldm, my_row, my_b, cnt, c0, 4, sum);
            store_sum<true>(u, realout != 0, d, c0, sum);
        } else {
            add_rows<false, LO, UN, false>(Rm, Rlo, ldm, my_row, my_b, cnt, c0, clamp4(2 * ((d + 1) / 2) - c0), sum);
            store_sum<false>(u, realout != 0, d, c0, sum);
        }
    }
}

// One, two or four chunks of 64 nodes: in four, 65 to 128 nodes carried two empty ones through every sum.  Decodes with 8 liars, us,
// four chunks / two: (70, 8, 7 000) on the 5-byte wire 45.1 / 41.6, (70, 8, 300 000) on two fp32 words 112 / 110.
template <class F>
static void with_chunks(int P, F&& f) {
    static_assert(kMaxNodes == 4 * kW, "four chunks at most");
    if (P <= kW) f(std::integral_constant<int, 1>());
    else if (P <= 2 * kW) f(std::integral_constant<int, 2>());
    else f(std::integral_constant<int, 4>());
}

static void launch(int threads, const double2* sums, int tiles, const double2* roots, int P, int s, double tau,
                   const double2* b0, const CycSpec& spec, const LocateOut& out, bool sample, hipStream_t stream) {
    const double isq = 1.0 / std::sqrt((double)P);
    auto go = [&](auto chunks) {
        hipLaunchKernelGGL((cyc_locate_kernel<decltype(chunks)::value>), dim3(1), dim3(threads), 0, stream, sums, tiles, roots, P,
                           s, tau, isq, b0, spec, out, sample ? 1 : 0);
    };
    with_chunks(P, go);
}

hipError_t load_locator() {
    hipFuncAttributes of{};
    return hipFuncGetAttributes(&of, reinterpret_cast<const void*>(&cyc_locate_walk_kernel<kLoNone, 6>));
}

hipError_t launch_cyc_locate_recombine(const double2* sums, int64_t tiles, const double2* roots, int P, int s, double tau,
                                       const double2* b0, uint64_t* mask_out, int32_t* status_out, const CycSpec& spec,
                                       const float* R, const float* Rlo, int lo, int64_t ldm, float* u, bool realout, int64_t d,
                                       hipStream_t stream) {
    const double isq = 1.0 / std::sqrt((double)P);
    with_format(Rlo, lo, [&](auto fmt) {
        constexpr int LO = decltype(fmt)::value;
        if (one_chunk_per_cu(d)) {
            const dim3 grid((unsigned)((d + kW * 4 - 1) / (kW * 4)));
            auto go = [&](auto chunks) {
                hipLaunchKernelGGL((cyc_locate_recombine_kernel<LO, decltype(chunks)::value>), grid, dim3(kW * kSumWaves), 0,
                                   stream, sums, (int)tiles, roots, P, s, tau, isq, b0, mask_out, status_out, R, Rlo, ldm, u,
                                   realout ? 1 : 0, d);
            };
            with_chunks(P, go);
            return;
        }
        // As many workgroups as take the same number of 4 KiB pieces each, two per CU at most (bf16 second words, (40, 5,
        // 800 001): 70.3 us, 72.5 with 512 of them), and few rows in flight, whose place eight wavefronts per CU take.
        const unsigned blocks = grid_cols<kSpreadRecombine>(d), rounds = (blocks + 511) / 512;
        constexpr int UN = LO == kLoNone ? 6 : LO == kLoF32 ? 2 : 3;
        hipLaunchKernelGGL((cyc_locate_walk_kernel<LO, UN>), dim3((blocks + rounds - 1) / rounds), dim3(kBlock), 0, stream, sums,
                           (int)tiles, roots, P, s, tau, isq, b0, mask_out, status_out, spec, R, Rlo, ldm, u, realout ? 1 : 0,
                           blocks, d);
    });
    return hipGetLastError();
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
