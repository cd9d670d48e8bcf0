// Cyclic code: the two streaming passes of the decoder D^Cyc (Algorithm 1) -- the
// projection f R of phi and the recombination R_{.,U} b -- and the plain copy kernel
// used for calibration.
#include "device_util.hpp"
#include "projection_rng.hpp"
#include "recombine_device.hpp"
#include "wave_reduce.hpp"

#include <algorithm>
#include <type_traits>

namespace draco {

// The set that the projection pass speculates on (run after the sample's locator).
__device__ __forceinline__ int speculates_on(const CycSpec& spec) {
    if (spec.mask == nullptr) return spec.state[kSpecClean] != 0 ? kSpecOnNobody : 0;
    if (takes_sample(spec)) return spec.state[kSpecStatus] == 0 ? kSpecOnSample : 0;
    return spec.state[kSpecClean] >= kCleanRun ? kSpecOnNobody : 0;
}

// phi step 1: gamma'_j = sum_i f_i * r_j[i].  A lane owns K float4 (two complex numbers each) of
// every row, keeps its slice of f in registers and has the next D rows in flight: a row's registers
// are loaded again as soon as it is summed.  The 2 D fp64 sums of D rows are reduced over the
// wavefront together (reduce_over_wave).  The four wavefront sums are added in fixed order and stored
// per tile.
//
// Speculation (SPEC): while a row is in registers the kernel also accumulates
// u0 = sum_j b_j r_j with b the recombination vector for a predicted set of adversaries, and
// writes it to the output.  If the locator then finds that set, u0 IS the decoded sum (b depends on
// the set alone; same coefficients, same order, same instruction sequence as the recombination
// kernel) and the second pass over the messages is skipped.  Rows of predicted adversaries stay out
// of u0.
// ONCE: at most D rows, nothing is fetched again (a kernel of a few us waits for its instructions too: the
// fewer the better).
// F: whether f is stored (f != nullptr).  Left to run time the compiler starts to make an f ahead of the branch, which a
// short kernel with a stored one notices.
enum { kFEither, kFStored, kFMade };
template <int LO, int K, int D, bool NT, bool SPEC, bool FULL, bool ONCE = false, int F = kFEither>
__device__ __forceinline__ void cyc_project_body(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                 int64_t ldm, const float* __restrict__ f, uint64_t f_seed,
                                                 const double2* __restrict__ b, const uint64_t* __restrict__ flagged,
                                                 float* __restrict__ u, bool realout, const int64_t (&col)[K], int j0,
                                                 int j1, int64_t d, double2 (*wsum)[kMaxNodes]) {
    const int64_t h = (d + 1) / 2;                                   // complex numbers per row
    int nflt[K];  // message floats that exist in my k-th float4 (4, 2 or 0)
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t c = col[k] / 2;   // first complex index
        nflt[k] = (FULL || c + 1 < h) ? 4 : (c < h ? 2 : 0);
    }
    float4 x[D][K];
    lo_raw_t<LO> xl[D][LO != kLoNone ? K : 1];
    auto fetch = [&](int slot, int j) {
        const int64_t row = (int64_t)j * ldm;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            x[slot][k] = ldx<FULL, NT>(Rm + row + col[k], nflt[k]);
            if constexpr (LO != kLoNone) xl[slot][k] = ld_lo<FULL, LO, NT>(Rlo, row + col[k], nflt[k]);
        }
    };
    // in flight while f is read or made.  (Fewer rows than D: the last one again, unused.  Under a condition the
    // compiler moves a row's conversion to fp64 up to its load and waits for each row in turn.)
#pragma unroll
    for (int i = 0; i < D; ++i) fetch(i, min(j0 + i, j1 - 1));
    double f0[K], f1[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t c = col[k] / 2;
        if (F == kFStored || (F == kFEither && f != nullptr)) {
            f0[k] = (FULL || c < h) ? (double)f[c] : 0.0;
            f1[k] = (FULL || c + 1 < h) ? (double)f[c + 1] : 0.0;
        } else {  // no stored vector: make the two entries (once per tile, reused for all P rows)
            f0[k] = (FULL || c < h) ? (double)projection_entry(f_seed, (uint64_t)c) : 0.0;
            f1[k] = (FULL || c + 1 < h) ? (double)projection_entry(f_seed, (uint64_t)(c + 1)) : 0.0;
        }
    }
    double ure0[SPEC ? K : 1], uim0[SPEC ? K : 1], ure1[SPEC ? K : 1], uim1[SPEC ? K : 1];
    uint64_t out_of_u[SPEC ? kMaskWords : 1];   // rows of predicted adversaries
    if constexpr (SPEC) {
#pragma unroll
        for (int k = 0; k < K; ++k) ure0[k] = uim0[k] = ure1[k] = uim1[k] = 0.0;
#pragma unroll
        for (int w = 0; w < kMaskWords; ++w) out_of_u[w] = flagged != nullptr && 64 * w < j1 ? table_entry(flagged, w) : 0ull;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // Rows j .. j+D-1 from the ring.  WHOLE: all of them exist and so do the D rows behind them, which
    // are fetched.  No load is then under a condition: behind one the compiler cannot count the loads
    // in flight and waits for all of them.
    auto round = [&](auto whole, int j) {
        constexpr bool WHOLE = decltype(whole)::value;
        double sums[2 * D];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int at = j + i;
            double are = 0.0, aim = 0.0;
            if (WHOLE || ONCE || at < j1) {
                auto row = [&](auto joint) {   // the projection of row `at`, with its share of u if joint
                    double2 bj = make_double2(0.0, 0.0);
                    if constexpr (decltype(joint)::value) bj = table_entry(b, at);
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const wire4 v = wire_value<LO>(x[i][k], xl[i][LO != kLoNone ? k : 0]);
                        are = fma(f0[k], v.x, are);
                        aim = fma(f0[k], v.y, aim);
                        are = fma(f1[k], v.z, are);
                        aim = fma(f1[k], v.w, aim);
                        if constexpr (decltype(joint)::value) {
                            cmac(bj.x, bj.y, v.x, v.y, ure0[k], uim0[k]);
                            cmac(bj.x, bj.y, v.z, v.w, ure1[k], uim1[k]);
                        }
                    }
                };
                if constexpr (SPEC) {
                    const uint64_t word = at < 64 ? out_of_u[0] : at < 128 ? out_of_u[1] : at < 192 ? out_of_u[2] : out_of_u[3];
                    if (((word >> (at & 63)) & 1ull) != 0) row(std::false_type{});
                    else row(std::true_type{});
                } else {
                    row(std::false_type{});
                }
                if constexpr (!ONCE) {
                    if (WHOLE || at + D < j1) fetch(i, at + D);
                }
            }
            sums[2 * i] = are;
            sums[2 * i + 1] = aim;
        }
        const double t = reduce_over_wave<2 * D>(sums);
        constexpr int G = 64 / (2 * D);   // lanes that share a sum
        const int v = lane / G;           // 2 * row + component
        if (lane % G == 0 && (WHOLE || j + v / 2 < j1)) reinterpret_cast<double*>(&wsum[wave][j - j0])[v] = t;
    };
    if constexpr (ONCE) {
        round(std::false_type{}, j0);
    } else {
        int j = j0;
        for (; j + 2 * D <= j1; j += D) round(std::true_type{}, j);
        for (; j < j1; j += D) round(std::false_type{}, j);
    }
    if constexpr (SPEC) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t c0 = col[k];
            if (realout) {  // unpacked wire: the sum is the real part, one float per complex entry
                const int64_t c = c0 / 2;
                if (FULL || c < h) u[c] = (float)ure0[k];
                if (FULL || c + 1 < h) u[c + 1] = (float)ure1[k];
            } else {
                const int nout = clamp4(d - c0);
                const float4 out = make_float4((float)ure0[k], (float)uim0[k], (float)ure1[k], (float)uim1[k]);
                if (nout == 4) st4(u + c0, out);
                else st4_partial(u + c0, out, nout);
            }
        }
    }
}
// partial[j] <- the sum of the four wavefronts' sums of row j, for the rows j0 .. j1-1 of this workgroup.
__device__ __forceinline__ void store_wave_sums(const double2 (*wsum)[kMaxNodes], double2* __restrict__ partial, int j0, int j1) {
    __syncthreads();
    if ((int)threadIdx.x < j1 - j0) {
        double2 a = wsum[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) {
            a.x += wsum[w][threadIdx.x].x;
            a.y += wsum[w][threadIdx.x].y;
        }
        partial[j0 + threadIdx.x] = a;
    }
}

// The projection of short rows: 4 KiB tiles (blockIdx.x), groups of 8 nodes (blockIdx.y), no speculation.  A launch
// of a few us is bound by latency: all rows of a group are loaded at once.  For second words of 8 and 16 bits straight through,
// under no condition ((45, 3, 20 000), 5-byte wire: 6.1 us, 7.6 as bursts); the others gain from a row's
// arithmetic standing behind the row's condition, where its wait is for that row alone (8-byte wire: 7.6 us, 9.5
// straight through; one word: 6.4 and 6.5; 6-byte wire, (250, 1, 10 000): 7.9 us as bursts, 7.4 straight through).
template <int LO, int F>
__global__ __launch_bounds__(kBlock) void cyc_project_short_kernel(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                                   int64_t ldm, const float* __restrict__ f, uint64_t f_seed,
                                                                   double2* __restrict__ partial, int P, int64_t d) {
    __shared__ double2 wsum[kBlock / 64][kMaxNodes];
    const int j0 = (int)blockIdx.y * 8, j1 = min(P, j0 + 8);
    const int64_t col[1] = {((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4};
    if ((int64_t)(blockIdx.x + 1) * (kBlock * 4) <= (d + 1) / 2 * 2)
        cyc_project_body<LO, 1, 8, false, false, true, true, F>(Rm, Rlo, ldm, f, f_seed, nullptr, nullptr, nullptr, false, col, j0, j1, d, wsum);
    else
        cyc_project_body<LO, 1, 8, false, false, false, true, F>(Rm, Rlo, ldm, f, f_seed, nullptr, nullptr, nullptr, false, col, j0, j1, d, wsum);
    store_wave_sums(wsum, partial + (int64_t)blockIdx.x * P, j0, j1);
}

// Rows in bursts of 8.  (A group of 8 nodes is one burst.  As cyc_project_body with its rows under conditions these kernels
// take 107 registers for 82 and 10 to 40 % longer: the loop is what keeps a row's conversions behind its load.)
template <int LO, bool FULL>
__device__ __forceinline__ void cyc_project_burst_body(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                       int64_t ldm, const float* __restrict__ f, uint64_t f_seed, int64_t col,
                                                       int j0, int j1, int64_t d, double2 (*wsum)[kMaxNodes]) {
    constexpr int D = 8;
    const int64_t h = (d + 1) / 2, c = col / 2;
    const int n = (FULL || c + 1 < h) ? 4 : (c < h ? 2 : 0);
    float4 x[D];
    lo_raw_t<LO> xl[D];
    auto fetch = [&](int j) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
            if (j + i < j1) {
                const int64_t off = (int64_t)(j + i) * ldm + col;
                x[i] = ldx<FULL, false>(Rm + off, n);
                if constexpr (LO != kLoNone) xl[i] = ld_lo<FULL, LO, false>(Rlo, off, n);
            }
        }
    };
    fetch(j0);
    double f0, f1;
    if (f != nullptr) {
        f0 = (FULL || c < h) ? (double)f[c] : 0.0;
        f1 = (FULL || c + 1 < h) ? (double)f[c + 1] : 0.0;
    } else {
        f0 = (FULL || c < h) ? (double)projection_entry(f_seed, (uint64_t)c) : 0.0;
        f1 = (FULL || c + 1 < h) ? (double)projection_entry(f_seed, (uint64_t)(c + 1)) : 0.0;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int j = j0; j < j1; j += D) {
        if (j != j0) fetch(j);
        double sums[2 * D];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            double are = 0.0, aim = 0.0;
            if (j + i < j1) {
                const wire4 v = wire_value<LO>(x[i], xl[i]);
                are = fma(f0, v.x, are);
                aim = fma(f0, v.y, aim);
                are = fma(f1, v.z, are);
                aim = fma(f1, v.w, aim);
            }
            sums[2 * i] = are;
            sums[2 * i + 1] = aim;
        }
        const double t = reduce_over_wave<2 * D>(sums);
        constexpr int G = 64 / (2 * D);
        const int v = lane / G;
        if (lane % G == 0 && j + v / 2 < j1) reinterpret_cast<double*>(&wsum[wave][j - j0])[v] = t;
    }
}
template <int LO>
__global__ __launch_bounds__(kBlock) void cyc_project_burst_kernel(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                                   int64_t ldm, const float* __restrict__ f, uint64_t f_seed,
                                                                   double2* __restrict__ partial, int P, int rows, int64_t d) {
    __shared__ double2 wsum[kBlock / 64][kMaxNodes];
    const int j0 = (int)blockIdx.y * rows, j1 = min(P, j0 + rows);
    const int64_t col = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
    if ((int64_t)(blockIdx.x + 1) * (kBlock * 4) <= (d + 1) / 2 * 2)
        cyc_project_burst_body<LO, true>(Rm, Rlo, ldm, f, f_seed, col, j0, j1, d, wsum);
    else
        cyc_project_burst_body<LO, false>(Rm, Rlo, ldm, f, f_seed, col, j0, j1, d, wsum);
    store_wave_sums(wsum, partial + (int64_t)blockIdx.x * P, j0, j1);
}
// blockIdx.x: tile of all P nodes.
// What it speculates on is up to spec (kernels.hpp); spec.state == nullptr: nothing.
// The first `rest` tiles take what is left of the rows behind their last whole window, 4 KiB contiguously each, the
// others K * 4 pieces of 1 KiB spread over a window (device_util.hpp, "workgroup footprint"): at (45, 3, 25.6 M) on
// the 5-byte wire the joint pass takes 885 us so and 955 with K * 4 KiB contiguously.  Rows off the line grid
// are read contiguously all the same (windows: K * 4 KiB), because both ends of every piece are parts of lines that
// another die reads too ((32, 4, 3 000 003) on the 6-byte wire: 134 us against 140).
// NT: streaming loads; NT_JOINT: in the joint pass.
template <int LO, int K, int D, bool NT, bool NT_JOINT>
__global__ __launch_bounds__(kBlock) void cyc_project_kernel(const float* __restrict__ Rm,
                                                             const float* __restrict__ Rlo, int64_t ldm,
                                                             const float* __restrict__ f, uint64_t f_seed,
                                                             double2* __restrict__ partial,
                                                             const double2* __restrict__ b0, float* __restrict__ u,
                                                             int realout, const CycSpec spec, int P,
                                                             unsigned rest, int contiguous, int64_t d) {
    __shared__ double2 wsum[kBlock / 64][kMaxNodes];
    constexpr int j0 = 0;
    const int j1 = P;
    const double2* b = nullptr;
    const uint64_t* flagged = nullptr;
    if (spec.state != nullptr) {
        const int now = speculates_on(spec);
        if (now == kSpecOnSample) {
            b = spec.b;
            flagged = spec.mask;
        } else if (now == kSpecOnNobody) {
            b = b0;
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) spec.state[kSpecNow] = now;
    }
    const int64_t mlen = (d + 1) / 2 * 2;
    if (blockIdx.x < rest) {
        const int64_t unit = contiguous != 0 ? kBlock * 4 * K : kWindow, first = mlen / unit * unit;
        const int64_t c1[1] = {first + ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4};
        if (b != nullptr) cyc_project_body<LO, 1, 8, NT_JOINT, true, false>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, realout != 0, c1, j0, j1, d, wsum);
        else cyc_project_body<LO, 1, 8, NT, false, false>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, false, c1, j0, j1, d, wsum);
    } else {
        constexpr unsigned per = kWindow / (kBlock * 4 * K);   // tiles per window
        const unsigned tile = blockIdx.x - rest;
        int64_t c[K];
        if (contiguous == 0) {
            const int64_t base = (int64_t)(tile / per) * kWindow + (tile % per) * 256 + (threadIdx.x >> 6) * (per * 256) + (threadIdx.x & 63) * 4;
#pragma unroll
            for (int k = 0; k < K; ++k) c[k] = base + (int64_t)k * (4 * per * 256);
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) c[k] = ((int64_t)tile * K * kBlock + k * kBlock + threadIdx.x) * 4;
        }
        if (b != nullptr) cyc_project_body<LO, K, D, NT_JOINT, true, true>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, realout != 0, c, j0, j1, d, wsum);
        else cyc_project_body<LO, K, D, NT, false, true>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, false, c, j0, j1, d, wsum);
    }
    store_wave_sums(wsum, partial + (int64_t)blockIdx.x * P, j0, j1);
}

// The projection of a sample: kSampleTiles tiles of 1024 floats, `step` tiles apart, rows in groups
// of 8 (blockIdx.y).  The first one is drawn from f, which is new in every call and unknown to the
// adversaries, so that no column (but a row's last, partial tile) is safe from the sample.
template <int LO>
__global__ __launch_bounds__(kBlock) void cyc_sample_kernel(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                            int64_t ldm, const float* __restrict__ f, uint64_t f_seed,
                                                            double2* __restrict__ partial, const CycSpec spec,
                                                            int P, unsigned step, unsigned firsts, int64_t d) {
    if (!takes_sample(spec)) return;
    __shared__ double2 wsum[kBlock / 64][kMaxNodes];
    const int j0 = (int)blockIdx.y * 8, j1 = min(P, j0 + 8);
    uint64_t draw = f_seed;
    if (f != nullptr) draw = ((uint64_t)__float_as_uint(f[0]) << 32) | __float_as_uint(f[1]);
    draw = (draw ^ (draw >> 29)) * 0x9E3779B97F4A7C15ull;
    const int64_t first = (unsigned)(draw >> 32) % firsts;
    const int64_t col[1] = {((first + (int64_t)blockIdx.x * step) * kBlock + threadIdx.x) * 4};
    cyc_project_body<LO, 1, 8, true, false, true, true>(Rm, Rlo, ldm, f, f_seed, nullptr, nullptr, nullptr, false, col, j0, j1, d,
                                                     wsum);
    store_wave_sums(wsum, partial + (int64_t)blockIdx.x * P, j0, j1);
}

// sums[part][j] = sum over the part's tiles of partial[tile][j], in a fixed order, UN entries in flight per lane.  A
// workgroup touches every line of its part for 16 bytes of it, so a long table is read in kReduceParts parts, each by one
// die (workgroup b runs on die b mod 8): 6256 tiles of 45 nodes 5.0 us, 7.5 with the parts spread over the dies, 11.2 in
// one part, 11 to 19 in one part with two to eight nodes per workgroup.
template <int UN>
__global__ __launch_bounds__(kBlock) void cyc_project_reduce_kernel(const double2* __restrict__ partial,
                                                                    double2* __restrict__ sums, int P, int tiles) {
    __shared__ double2 sm[kBlock];
    const int j = blockIdx.y, per = (tiles + (int)gridDim.x - 1) / (int)gridDim.x;
    const int begin = (int)blockIdx.x * per, end = min(tiles, begin + per);
    double2 a = make_double2(0.0, 0.0);
    for (int t0 = begin + (int)threadIdx.x; t0 < end; t0 += UN * kBlock) {
        double2 p[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) p[i] = partial[(int64_t)min(t0 + i * kBlock, end - 1) * P + j];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            if (t0 + i * kBlock < end) {
                a.x += p[i].x;
                a.y += p[i].y;
            }
        }
    }
    sm[threadIdx.x] = a;
    __syncthreads();
    for (int off = kBlock / 2; off >= 1; off >>= 1) {
        if ((int)threadIdx.x < off) {
            sm[threadIdx.x].x += sm[threadIdx.x + off].x;
            sm[threadIdx.x].y += sm[threadIdx.x + off].y;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[(int64_t)blockIdx.x * P + j] = sm[0];
}

// u = R_{.,U} b on packed complex messages, unpacked to reals (recombine_device.hpp): 64 honest rows at a time.
template <bool FULL, int LO, int UN, bool NT>
__device__ __forceinline__ void cyc_recombine_body(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                   int64_t ldm,
                                                   const double2* __restrict__ b, const int32_t* __restrict__ idx,
                                                   const int32_t* __restrict__ nu_ptr, float* __restrict__ u,
                                                   bool realout, int64_t d, int64_t c0) {
    const int nu = *nu_ptr;  // honest nodes; written by the locator (device) or copied in by the host path
    const int lane = threadIdx.x & 63;
    const int nin = FULL ? 4 : clamp4(2 * ((d + 1) / 2) - c0);   // (all lanes stay: the others read their indices)
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int base = 0; base < nu; base += 64) {
        const int cnt = min(64, nu - base), mine = base + min(lane, cnt - 1);
        add_rows<FULL, LO, UN, NT>(Rm, Rlo, ldm, idx[mine], b[mine], cnt, c0, nin, sum);
    }
    store_sum<FULL>(u, realout, d, c0, sum);
}

// If the projection pass speculated on the set that the locator found, the output already holds the
// answer: nothing to do.
template <int LO, int UN, bool NT>
__global__ __launch_bounds__(kBlock) void cyc_recombine_kernel(const float* __restrict__ Rm,
                                                               const float* __restrict__ Rlo, int64_t ldm,
                                                               const double2* __restrict__ b,
                                                               const int32_t* __restrict__ idx,
                                                               const int32_t* __restrict__ nu,
                                                               const int32_t* __restrict__ state,
                                                               float* __restrict__ u, int realout, int64_t d) {
    if (state != nullptr && state[kSpecDone] != 0) return;
    const int64_t c0 = lane_column<kSpreadRecombine>(d);
    if (block_is_full<kSpreadRecombine>(d, d)) cyc_recombine_body<true, LO, UN, NT>(Rm, Rlo, ldm, b, idx, nu, u, realout != 0, d, c0);
    else cyc_recombine_body<false, LO, UN, NT>(Rm, Rlo, ldm, b, idx, nu, u, realout != 0, d, c0);
}

// The same for rows too short to fill the chip, where all of it is latency: a workgroup owns 1 KiB of the
// rows, its wavefronts take every fourth honest row, six in flight, and their sums are added in order.  (More
// rows in flight per wavefront are more instructions, which a kernel of a few us waits for as well.)
template <bool FULL, int LO>
__device__ __forceinline__ void cyc_recombine_few_body(const float* __restrict__ Rm, const float* __restrict__ Rlo, int64_t ldm,
                                                       const double2* __restrict__ b, const int32_t* __restrict__ idx, int nu,
                                                       int64_t c0, int nin, double (&sum)[4]) {
    constexpr int UN = 6, W = kBlock / 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int base = wave; base < nu; base += W * 64) {   // lane l holds row base + W l
        const int cnt = min(64, (nu - base + W - 1) / W), mine = base + W * min(lane, cnt - 1);
        const int my_row = idx[mine];
        const double2 my_b = b[mine];
        for (int q = 0; q < cnt; q += UN) {
            float4 x[UN];
            lo_raw_t<LO> xl[LO != kLoNone ? UN : 1];
#pragma unroll
            for (int i = 0; i < UN; ++i) {   // (behind the last row it is read again)
                const int64_t off = (int64_t)__builtin_amdgcn_readlane(my_row, min(q + i, cnt - 1)) * ldm + c0;
                x[i] = ldx<FULL, false>(Rm + off, nin);
                if constexpr (LO != kLoNone) xl[i] = ld_lo<FULL, LO, false>(Rlo, off, nin);
            }
#pragma unroll
            for (int i = 0; i < UN; ++i) {
                if (q + i < cnt) {
                    const double br = lane_value(my_b.x, q + i), bi = lane_value(my_b.y, q + i);
                    const wire4 v = wire_value<LO>(x[i], xl[LO != kLoNone ? i : 0]);
                    cmac(br, bi, v.x, v.y, sum[0], sum[1]);
                    cmac(br, bi, v.z, v.w, sum[2], sum[3]);
                }
            }
        }
    }
}
template <int LO>
__global__ __launch_bounds__(kBlock) void cyc_recombine_few_kernel(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                                   int64_t ldm, const double2* __restrict__ b,
                                                                   const int32_t* __restrict__ idx,
                                                                   const int32_t* __restrict__ nu, float* __restrict__ u,
                                                                   int realout, int64_t d) {
    __shared__ double part[kBlock / 64][4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c0 = ((int64_t)blockIdx.x * 64 + lane) * 4;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    if (((int64_t)blockIdx.x + 1) * 256 <= d) cyc_recombine_few_body<true, LO>(Rm, Rlo, ldm, b, idx, *nu, c0, 4, sum);
    else cyc_recombine_few_body<false, LO>(Rm, Rlo, ldm, b, idx, *nu, c0, clamp4(2 * ((d + 1) / 2) - c0), sum);
#pragma unroll
    for (int i = 0; i < 4; ++i) part[wave][i][lane] = sum[i];
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < kBlock / 64; ++w) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] += part[w][i][lane];
    }
    if (realout != 0) {
        const int64_t c = c0 / 2;
        if (2 * c < d) u[c] = (float)sum[0];
        if (2 * c + 2 < d) u[c + 1] = (float)sum[2];
    } else {
        stx<false>(u + c0, make_float4((float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]), clamp4(d - c0));
    }
}

// Plain copy of a [rows][row_len] slab (row stride ld): the fastest copy of a row-major
// slab found on MI355X.  A workgroup moves one 4 KiB piece of one row and ends; column
// tiles vary fastest across the grid, so at any moment the chip streams one or two rows.
// Calibration kernel for bandwidth figures and for scaling hardware byte counters.
__global__ __launch_bounds__(kBlock) void copy_probe_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                                            int rows, int64_t row_len, int64_t ld) {
    const int64_t c0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
    if (c0 + 4 > row_len || (int)blockIdx.y >= rows) return;
    const int64_t off = (int64_t)blockIdx.y * ld + c0;
    st4(dst + off, ld4(src + off));
}


// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

// float4 per lane and row (K) of the projection: as many as still give about two workgroups per CU, one on many rows,
// which live longer (more columns per lane share the sums over the wavefront).  Project and sample in us, K = 4, 2 and 1:
// 45 rows of the 5-byte wire 25.6 M floats 926, 950 and 983; 1.9 M 99, 106 and 111; 1.2 M 70, 63 and 65; 500 000 35, 34
// and 38; 15 rows of one word 4 M 46, 49 and 53; 2 M 29.4, 28.1 and 29.9; 500 000 16, 14.4 and 13.6.
// But one where the wider lanes' last workgroups leave that many more of the CUs idle: decodes over states in turn, K = 2 and
// 1, (45, 3) on the 5-byte wire 1 200 001, 586 workgroups and 1172, 63.6 and 60.2 us, 600 001, 293 and 586, 40.2 and 38.9.
static int project_width(int64_t d, int P) {
    const int64_t nvec = ((d + 1) / 2 + 1) / 2;
    const int wide = nvec >= (P >= 24 ? 440 : 880) * kBlock * 4 ? 4 : nvec >= 240 * kBlock * 2 ? 2 : 1;
    auto turns = [&](int k) { return (nvec + 256ll * kBlock * k - 1) / (256ll * kBlock * k) * k; };   // of one float4 per lane
    return 5 * turns(wide) >= 6 * turns(1) ? 1 : wide;
}
// Tiles of whole windows, and of 4 KiB contiguously for the rest of a row (see cyc_project_kernel).
struct ProjectTiles {
    int64_t whole, rest;
};
static ProjectTiles tiles_of(int64_t d, int P, bool contiguous) {
    const int64_t mlen = (d + 1) / 2 * 2, per = kBlock * 4 * project_width(d, P), unit = contiguous ? per : kWindow;
    return {mlen / unit * unit / per, grid_for((mlen % unit + 3) / 4)};
}
int64_t project_tiles(int64_t d, int P, int64_t ldm) {
    const ProjectTiles t = tiles_of(d, P, ldm % 32 != 0);
    return t.whole + t.rest;
}
int64_t project_tiles_at_most(int64_t d, int P) { return std::max(project_tiles(d, P, 0), project_tiles(d, P, 4)); }
// Rows of fewer 4 KiB tiles than CUs are short: a workgroup takes 8 nodes of a tile, and nothing is speculated on.  Of 8 nodes
// or fewer only those that the locator's kernel also recombines: beyond, a speculation that holds saves a launch there.
bool short_rows(int64_t d, int P) {
    return (d + 1) / 2 * 2 <= (P > 8 ? kShortTiles : kFusedTiles) * (kBlock * 4);
}


hipError_t launch_cyc_project(const float* R, const float* Rlo, int lo, int64_t ldm, const float* f, uint64_t f_seed,
                              double2* partial, const double2* b0, float* u, bool realout, const CycSpec& spec, int P,
                              int64_t d, hipStream_t stream) {
    const int K = project_width(d, P);
    const bool contiguous = ldm % 32 != 0;
    const ProjectTiles t = tiles_of(d, P, contiguous);
    const dim3 grid((unsigned)(t.whole + t.rest));
    // A second pass finds messages of this size in the memory-side cache (kernels.hpp); a joint pass expects none.
    const int64_t bytes = P * d * word_bytes(Rlo, lo);
    const bool stay = bytes <= kSmallMessages, stay_joint = bytes <= kCachedMessages;
    with_format(Rlo, lo, [&](auto fmt) {
        constexpr int LO = decltype(fmt)::value;
        auto go = [&](auto k, auto ahead, auto nt, auto nt_joint) {
            constexpr int N = decltype(k)::value, D = decltype(ahead)::value;
            constexpr bool NT = decltype(nt)::value, NTJ = decltype(nt_joint)::value;
            constexpr size_t fixed = (kBlock / 64) * kMaxNodes * sizeof(double2);   // wsum
            // four pieces: two workgroups per CU ((15, 2, 4 M): 46 us, 49 unlimited)
            size_t lds = 0;
            if constexpr (N == 4) {
                allow_large_lds<cyc_project_kernel<LO, N, D, NT, NTJ>>(fixed);
                lds = throttle_lds(2, fixed, 0);
            }
            hipLaunchKernelGGL((cyc_project_kernel<LO, N, D, NT, NTJ>), grid, dim3(kBlock), lds, stream, R, Rlo, ldm, f, f_seed,
                               partial, b0, u, realout ? 1 : 0, spec, P, (unsigned)t.rest, contiguous ? 1 : 0, d);
        };
        // rows in flight: two of K = 4 or 2 pieces (four gain nothing), four of one
        auto shape = [&](auto nt, auto nt_joint) {
            if (K == 4) go(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{}, nt, nt_joint);
            else if (K == 2) go(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{}, nt, nt_joint);
            else go(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{}, nt, nt_joint);
        };
        if (short_rows(d, P)) {
            constexpr int rows = 8;   // (45, 3, 30 000) on the 5-byte wire: 18 us with all rows in one group, 9 in groups of 8
            const dim3 groups(grid.x, (unsigned)((P + rows - 1) / rows));
            if constexpr (LO == kLoI8 || LO == kLoBf16) {
                auto go = [&](auto where) {
                    hipLaunchKernelGGL((cyc_project_short_kernel<LO, decltype(where)::value>), groups, dim3(kBlock), 0, stream, R,
                                       Rlo, ldm, f, f_seed, partial, P, d);
                };
                if (f != nullptr) go(std::integral_constant<int, kFStored>{});
                else go(std::integral_constant<int, kFMade>{});
            } else {
                hipLaunchKernelGGL(cyc_project_burst_kernel<LO>, groups, dim3(kBlock), 0, stream, R, Rlo, ldm, f, f_seed, partial,
                                   P, rows, d);
            }
            return;
        }
        if (stay_joint) shape(std::false_type{}, std::false_type{});
        else if (stay) shape(std::false_type{}, std::true_type{});
        else shape(std::true_type{}, std::true_type{});
    });
    return hipGetLastError();
}

hipError_t launch_cyc_sample(const float* R, const float* Rlo, int lo, int64_t ldm, const float* f, uint64_t f_seed,
                             double2* partial, const CycSpec& spec, int P, int64_t d, hipStream_t stream) {
    const int64_t tiles = (d + 1) / 2 * 2 / (kBlock * 4);   // whole ones
    if (tiles < kSampleTiles) return hipErrorInvalidValue;
    const int64_t step = tiles / kSampleTiles, firsts = tiles - (kSampleTiles - 1) * step;   // first tile < firsts
    with_format(Rlo, lo, [&](auto fmt) {
        hipLaunchKernelGGL((cyc_sample_kernel<decltype(fmt)::value>), dim3(kSampleTiles, (unsigned)((P + 7) / 8)),
                           dim3(kBlock), 0, stream, R, Rlo, ldm, f, f_seed, partial, spec, P, (unsigned)step,
                           (unsigned)firsts, d);
    });
    return hipGetLastError();
}

hipError_t launch_cyc_reduce(const double2* partial, double2* sums, int parts, int P, int64_t tiles, hipStream_t stream) {
    const dim3 grid((unsigned)parts, (unsigned)P);
    if (tiles <= (int64_t)4 * kBlock * parts)
        hipLaunchKernelGGL(cyc_project_reduce_kernel<4>, grid, dim3(kBlock), 0, stream, partial, sums, P, (int)tiles);
    else
        hipLaunchKernelGGL(cyc_project_reduce_kernel<8>, grid, dim3(kBlock), 0, stream, partial, sums, P, (int)tiles);
    return hipGetLastError();
}

hipError_t launch_copy_probe(const float* src, float* dst, int rows, int64_t row_len, int64_t ld,
                             hipStream_t stream) {
    hipLaunchKernelGGL(copy_probe_kernel, dim3(grid_for(row_len / 4), (unsigned)rows), dim3(kBlock), 0, stream, src,
                       dst, rows, row_len, ld);
    return hipGetLastError();
}

hipError_t launch_cyc_recombine(const float* R, const float* Rlo, int lo, int64_t ldm, const double2* b, const int32_t* idx,
                                const int32_t* nu, const int32_t* state, int P, float* u, bool realout,
                                int64_t d, hipStream_t stream) {
    const dim3 grid(grid_cols<kSpreadRecombine>(d)), block(kBlock);
    // Short rows: only where the projection does not speculate, whose joint pass adds the rows in another order; with
    // a full second word or none only the shorter half of those, on enough rows to share.  Kernel in us, this form
    // against the other: 5-byte wire, 250 000 floats, 45 nodes 17 and 30, 12 nodes 9.8 and 10.8; 6-byte, 45 nodes 22 and
    // 32; two fp32 words, 45 nodes 20 000 floats 13 and 18, 250 000 25 and 21, 12 nodes 60 000 9.2 and 8.3; one word, 18
    // nodes 20 000 6.7 and 7.7.
    const int bytes = word_bytes(Rlo, lo);
    const bool few = short_rows(d, P) && (bytes == 5 || bytes == 6 || (d <= 65536 && P >= 16));
    const bool stay = P * d * bytes <= kSmallMessages;   // see launch_cyc_project
    with_format(Rlo, lo, [&](auto fmt) {
        constexpr int LO = decltype(fmt)::value;
        // Rows in flight and workgroups per CU at (45, 3, 25.6 M): with an 8-bit second word 0.81 of the
        // HBM peak with 4 workgroups x 2 rows (also 2 x 6 and 6 x 1); a 16-bit one wants more wavefronts
        // for its 8-byte loads (four workgroups 0.82, two 0.69-0.76).  Two fp32 words of
        // short rows, which do not fill the chip, want five rows ((45, 3, 150 000): 15.3 us, 16.3 with three; 22.0 and 21.5 at
        // 300 000).
        constexpr int UN = LO == kLoNone ? 6 : LO == kLoI8 ? 2 : 3;
        const size_t lds = throttle_lds(LO == kLoBf16 || LO == kLoI8 ? 4 : 2, 0, 0);
        auto go = [&](auto un, auto nt, size_t bytes) {
            constexpr int N = decltype(un)::value;
            constexpr bool NT = decltype(nt)::value;
            allow_large_lds<cyc_recombine_kernel<LO, N, NT>>();
            hipLaunchKernelGGL((cyc_recombine_kernel<LO, N, NT>), grid, block, bytes, stream, R, Rlo, ldm, b, idx, nu, state,
                               u, realout ? 1 : 0, d);
        };
        if (few)
            hipLaunchKernelGGL(cyc_recombine_few_kernel<LO>, dim3((unsigned)((d + 255) / 256)), block, 0, stream, R, Rlo, ldm, b,
                               idx, nu, u, realout ? 1 : 0, d);
        else if (LO == kLoF32 && short_rows(d, P)) go(std::integral_constant<int, LO == kLoF32 ? 5 : UN>{}, std::false_type{}, lds);
        else if (stay) go(std::integral_constant<int, UN>{}, std::false_type{}, lds);
        else go(std::integral_constant<int, UN>{}, std::true_type{}, lds);
    });
    return hipGetLastError();
}


}  // namespace draco
