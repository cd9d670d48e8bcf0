// Cyclic code: the two streaming passes of the decoder D^Cyc (Algorithm 1) -- the
// projection f R of phi and the recombination R_{.,U} b -- and the plain copy kernel
// used for calibration.
#include "device_util.hpp"
#include "projection_rng.hpp"
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

// phi step 1: gamma'_j = sum_i f_i * r_j[i].  A workgroup owns a tile of kBlock * K float4
// (two complex numbers each) of every row and keeps its slice of f in registers.  RB rows are
// taken at a time (8 loads of 16 bytes in flight per lane; 16, or a second buffer for the next
// round, gain nothing), and their 2 RB fp64 sums
// are reduced over the wavefront together (reduce_over_wave).  The four wavefront sums are added
// in fixed order and stored per tile.
//
// Speculation (SPEC): while a row is in registers the kernel also accumulates
// u0 = sum_j b_j r_j with b the recombination vector for a predicted set of adversaries, and
// writes it to the output.  If the locator then finds that set, u0 IS the decoded sum (b depends on
// the set alone; same coefficients, same order, same instruction sequence as the recombination
// kernel) and the second pass over the messages is skipped.  Rows of predicted adversaries stay out
// of u0.
template <int LO, int K, int RB, bool NT, bool SPEC, bool FULL>
__device__ __forceinline__ void cyc_project_body(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                 int64_t ldm, const float* __restrict__ f, uint64_t f_seed,
                                                 const double2* __restrict__ b, const uint64_t* __restrict__ flagged,
                                                 float* __restrict__ u, bool realout, int64_t tile, int j0, int j1,
                                                 int64_t d, double2 (*wsum)[kMaxNodes]) {
    const int64_t h = (d + 1) / 2;                                   // complex numbers per row
    const int64_t q0 = tile * (kBlock * K) + threadIdx.x;            // my first float4
    int nflt[K];  // message floats that exist in my k-th float4 (4, 2 or 0)
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t c = 2 * (q0 + (int64_t)k * kBlock);   // first complex index
        nflt[k] = (FULL || c + 1 < h) ? 4 : (c < h ? 2 : 0);
    }
    float4 x[RB][K];
    lo_raw_t<LO> xl[RB][LO != kLoNone ? K : 1];
    auto fetch = [&](int j) {   // rows j .. j+RB-1, those below j1
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            if (j + i < j1) {
                const int64_t off = (int64_t)(j + i) * ldm + q0 * 4;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    x[i][k] = ldx<FULL, NT>(Rm + off + (int64_t)k * kBlock * 4, nflt[k]);
                    if constexpr (LO != kLoNone)
                        xl[i][k] = ld_lo<FULL, LO, NT>(Rlo, off + (int64_t)k * kBlock * 4, nflt[k]);
                }
            }
        }
    };
    fetch(j0);   // in flight while f is read or made
    double f0[K], f1[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t c = 2 * (q0 + (int64_t)k * kBlock);
        if (f != nullptr) {
            f0[k] = (FULL || c < h) ? (double)f[c] : 0.0;
            f1[k] = (FULL || c + 1 < h) ? (double)f[c + 1] : 0.0;
        } else {  // no stored vector: make the two entries (once per tile, reused for all P rows)
            f0[k] = (FULL || c < h) ? (double)projection_entry(f_seed, (uint64_t)c) : 0.0;
            f1[k] = (FULL || c + 1 < h) ? (double)projection_entry(f_seed, (uint64_t)(c + 1)) : 0.0;
        }
    }
    double ure0[SPEC ? K : 1], uim0[SPEC ? K : 1], ure1[SPEC ? K : 1], uim1[SPEC ? K : 1];
    if constexpr (SPEC) {
#pragma unroll
        for (int k = 0; k < K; ++k) ure0[k] = uim0[k] = ure1[k] = uim1[k] = 0.0;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int j = j0; j < j1; j += RB) {
        if (j != j0) fetch(j);
        double sums[2 * RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            double are = 0.0, aim = 0.0;
            if (j + i < j1) {
                auto row = [&](auto joint) {   // the projection of row j + i, with its share of u if joint
                    double2 bj = make_double2(0.0, 0.0);
                    if constexpr (decltype(joint)::value) bj = b[j + i];
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
                    if (flagged != nullptr && ((flagged[(j + i) >> 6] >> ((j + i) & 63)) & 1ull) != 0)
                        row(std::false_type{});
                    else
                        row(std::true_type{});
                } else {
                    row(std::false_type{});
                }
            }
            sums[2 * i] = are;
            sums[2 * i + 1] = aim;
        }
        const double t = reduce_over_wave<2 * RB>(sums);
        constexpr int G = 64 / (2 * RB);   // lanes that share a sum
        const int v = lane / G;            // 2 * row + component
        if (lane % G == 0 && j + v / 2 < j1) reinterpret_cast<double*>(&wsum[wave][j - j0])[v] = t;
    }
    if constexpr (SPEC) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t c0 = (q0 + (int64_t)k * kBlock) * 4;
            if (realout) {  // unpacked wire: the sum is the real part, one float per complex entry
                const int64_t c = c0 / 2;
                if (c < h) u[c] = (float)ure0[k];
                if (c + 1 < h) u[c + 1] = (float)ure1[k];
            } else {
                const int nout = clamp4(d - c0);
                const float4 out = make_float4((float)ure0[k], (float)uim0[k], (float)ure1[k], (float)uim1[k]);
                if (nout == 4) st4(u + c0, out);
                else st4_partial(u + c0, out, nout);
            }
        }
    }
}

// blockIdx.x: tile, blockIdx.y: group of `rows` nodes (one group of all P if it may speculate).
// What it speculates on is up to spec (kernels.hpp); spec.state == nullptr: nothing.
template <int LO, int K, int RB, bool NT>
__global__ __launch_bounds__(kBlock) void cyc_project_kernel(const float* __restrict__ Rm,
                                                             const float* __restrict__ Rlo, int64_t ldm,
                                                             const float* __restrict__ f, uint64_t f_seed,
                                                             double2* __restrict__ partial,
                                                             const double2* __restrict__ b0, float* __restrict__ u,
                                                             int realout, const CycSpec spec, int P, int rows,
                                                             int64_t d) {
    __shared__ double2 wsum[kBlock / 64][kMaxNodes];
    const int j0 = (int)blockIdx.y * rows, j1 = min(P, j0 + rows);
    const int64_t tile = blockIdx.x;
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
    const bool full = (tile + 1) * (kBlock * K) * 2 <= (d + 1) / 2;
    if (b != nullptr) {
        if (full) cyc_project_body<LO, K, RB, NT, true, true>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, realout != 0, tile, j0, j1, d, wsum);
        else cyc_project_body<LO, K, RB, NT, true, false>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, realout != 0, tile, j0, j1, d, wsum);
    } else {
        if (full) cyc_project_body<LO, K, RB, NT, false, true>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, false, tile, j0, j1, d, wsum);
        else cyc_project_body<LO, K, RB, NT, false, false>(Rm, Rlo, ldm, f, f_seed, b, flagged, u, false, tile, j0, j1, d, wsum);
    }
    __syncthreads();
    if ((int)threadIdx.x < j1 - j0) {
        double2 a = wsum[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) {
            a.x += wsum[w][threadIdx.x].x;
            a.y += wsum[w][threadIdx.x].y;
        }
        partial[tile * P + j0 + threadIdx.x] = a;
    }
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
    cyc_project_body<LO, 1, 8, true, false, true>(Rm, Rlo, ldm, f, f_seed, nullptr, nullptr, nullptr, false,
                                                  first + (int64_t)blockIdx.x * step, j0, j1, d, wsum);
    __syncthreads();
    if ((int)threadIdx.x < j1 - j0) {
        double2 a = wsum[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) {
            a.x += wsum[w][threadIdx.x].x;
            a.y += wsum[w][threadIdx.x].y;
        }
        partial[(int64_t)blockIdx.x * P + j0 + threadIdx.x] = a;
    }
}

// gamma[j] = sum over tiles of partial[tile][j], in a fixed order.
__global__ __launch_bounds__(kBlock) void cyc_project_reduce_kernel(const double2* __restrict__ partial,
                                                                    double2* __restrict__ gamma, int P,
                                                                    int64_t tiles) {
    __shared__ double2 sm[kBlock];
    const int j = blockIdx.x;
    double2 a = make_double2(0.0, 0.0);
    for (int64_t t = threadIdx.x; t < tiles; t += kBlock) {
        const double2 p = partial[t * P + j];
        a.x += p.x;
        a.y += p.y;
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
    if (threadIdx.x == 0) gamma[j] = sm[0];
}

// u = R_{.,U} b on packed complex messages, unpacked to reals: honest rows in
// ascending node order, fp64 accumulation, one rounding to fp32.
template <bool FULL, int LO, int UN, bool NT>
__device__ __forceinline__ void cyc_recombine_body(const float* __restrict__ Rm, const float* __restrict__ Rlo,
                                                   int64_t ldm,
                                                   const double2* __restrict__ b, const int32_t* __restrict__ idx,
                                                   const int32_t* __restrict__ nu_ptr, float* __restrict__ u,
                                                   bool realout, int64_t d) {
    const int nu = *nu_ptr;  // honest nodes; written by the locator (device) or copied in by the host path
    const int64_t c0 = lane_column<kSpreadRecombine>(d);
    if (!FULL && c0 >= d) return;
    const int64_t mlen = 2 * ((d + 1) / 2);
    const int nin = FULL ? 4 : clamp4(mlen - c0);
    const int nout = FULL ? 4 : clamp4(d - c0);
    double are0 = 0.0, aim0 = 0.0, are1 = 0.0, aim1 = 0.0;
    for (int q0 = 0; q0 < nu; q0 += UN) {
        float4 x[UN];
        lo_raw_t<LO> xl[LO != kLoNone ? UN : 1];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            if (q0 + i < nu) {
                x[i] = ldx<FULL, NT>(Rm + (int64_t)idx[q0 + i] * ldm + c0, nin);
                if constexpr (LO != kLoNone) xl[i] = ld_lo<FULL, LO, NT>(Rlo, (int64_t)idx[q0 + i] * ldm + c0, nin);
            }
        }
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            if (q0 + i < nu) {
                const double br = b[q0 + i].x, bi = b[q0 + i].y;
                const wire4 v = wire_value<LO>(x[i], xl[LO != kLoNone ? i : 0]);
                cmac(br, bi, v.x, v.y, are0, aim0);
                cmac(br, bi, v.z, v.w, are1, aim1);
            }
        }
    }
    if (realout) {  // unpacked wire: the sum is the real part, one float per complex entry
        const int64_t c = c0 / 2;
        if (FULL || 2 * c < d) u[c] = (float)are0;
        if (FULL || 2 * c + 2 < d) u[c + 1] = (float)are1;
    } else {
        stx<FULL>(u + c0, make_float4((float)are0, (float)aim0, (float)are1, (float)aim1), nout);
    }
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
    if (block_is_full<kSpreadRecombine>(d, d)) cyc_recombine_body<true, LO, UN, NT>(Rm, Rlo, ldm, b, idx, nu, u, realout != 0, d);
    else cyc_recombine_body<false, LO, UN, NT>(Rm, Rlo, ldm, b, idx, nu, u, realout != 0, d);
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

// float4 per lane and row (K) of the projection, by the length of a row alone: 8 where that still
// gives two workgroups per CU, else 2, else 1 (and then groups of rows as well).  Measured with 45
// rows of the 5-byte wire, in us: 25.6 M floats 863, 890 and 937 with K = 8, 2 and 1 (speculating 958, 1028
// and -); 1.2 M 71, 57 and 55; 30 000 with K = 1 in one group 18, in groups of 8 rows 9.
static int project_width(int64_t d) {
    const int64_t nvec = ((d + 1) / 2 + 1) / 2;
    return nvec >= 480 * kBlock * 8 ? 8 : nvec >= 480 * kBlock * 2 ? 2 : 1;
}
int64_t project_tiles(int64_t d) {
    const int64_t nvec = ((d + 1) / 2 + 1) / 2;
    const int64_t per = (int64_t)kBlock * project_width(d);
    return (nvec + per - 1) / per;
}
// Nodes per workgroup: all of them, or groups of 8 where the tiles alone leave CUs idle.
static int project_rows(int64_t d, int P) {
    return project_width(d) == 1 && project_tiles(d) < 256 ? std::min(P, 8) : P;
}
bool project_speculates(int64_t d, int P) { return project_rows(d, P) == P; }

template <class F>
static void with_format(const float* Rlo, int lo, F&& fn) {
    if (Rlo == nullptr) fn(std::integral_constant<int, kLoNone>{});
    else if (lo == kLoBf16) fn(std::integral_constant<int, kLoBf16>{});
    else if (lo == kLoI8) fn(std::integral_constant<int, kLoI8>{});
    else fn(std::integral_constant<int, kLoF32>{});
}
static int word_bytes(const float* Rlo, int lo) {
    return Rlo == nullptr ? 4 : lo == kLoI8 ? 5 : lo == kLoBf16 ? 6 : 8;
}

hipError_t launch_cyc_project(const float* R, const float* Rlo, int lo, int64_t ldm, const float* f, uint64_t f_seed,
                              double2* partial, const double2* b0, float* u, bool realout, const CycSpec& spec, int P,
                              int64_t d, hipStream_t stream) {
    const int K = project_width(d), rows = project_rows(d, P);
    const dim3 grid((unsigned)project_tiles(d), (unsigned)((P + rows - 1) / rows));
    // the second pass finds messages of this size in the memory-side cache (kernels.hpp)
    const bool stay = P * d * word_bytes(Rlo, lo) <= kSmallMessages;
    with_format(Rlo, lo, [&](auto fmt) {
        constexpr int LO = decltype(fmt)::value;
        auto go = [&](auto k, auto rb, auto nt) {
            hipLaunchKernelGGL((cyc_project_kernel<LO, decltype(k)::value, decltype(rb)::value, decltype(nt)::value>), grid,
                               dim3(kBlock), 0, stream, R, Rlo, ldm, f, f_seed, partial, b0, u, realout ? 1 : 0, spec, P,
                               rows, d);
        };
        auto shape = [&](auto nt) {
            if (K == 8) go(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{}, nt);
            else if (K == 2) go(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{}, nt);
            else go(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{}, nt);
        };
        if (stay) shape(std::false_type{});
        else shape(std::true_type{});
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

hipError_t launch_cyc_reduce(const double2* partial, double2* gamma, int P, int64_t tiles, hipStream_t stream) {
    hipLaunchKernelGGL(cyc_project_reduce_kernel, dim3((unsigned)P), dim3(kBlock), 0, stream, partial, gamma, P, tiles);
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
    // rows too short to fill the chip: 16 rows in flight per lane, workgroups unlimited ((P, s, d) =
    // (45, 3, 30 000): 11 us against 22 with two)
    const bool few = grid.x < 512;
    const bool stay = P * d * word_bytes(Rlo, lo) <= kSmallMessages;   // see launch_cyc_project
    with_format(Rlo, lo, [&](auto fmt) {
        constexpr int LO = decltype(fmt)::value;
        // Rows in flight and workgroups per CU at (45, 3, 25.6 M): with an 8-bit second word 0.81 of the
        // HBM peak with 4 workgroups x 2 rows (also 2 x 6 and 6 x 1); a 16-bit one wants more wavefronts
        // for its 8-byte loads (four workgroups 0.82, two 0.69-0.76).
        constexpr int UN = LO == kLoNone ? 6 : LO == kLoI8 ? 2 : 3;
        const size_t lds = throttle_lds(LO == kLoBf16 || LO == kLoI8 ? 4 : 2, 0, 0);
        auto go = [&](auto un, auto nt, size_t bytes) {
            constexpr int N = decltype(un)::value;
            constexpr bool NT = decltype(nt)::value;
            allow_large_lds<cyc_recombine_kernel<LO, N, NT>>();
            hipLaunchKernelGGL((cyc_recombine_kernel<LO, N, NT>), grid, block, bytes, stream, R, Rlo, ldm, b, idx, nu, state,
                               u, realout ? 1 : 0, d);
        };
        if (few) go(std::integral_constant<int, 16>{}, std::false_type{}, 0);
        else if (stay) go(std::integral_constant<int, UN>{}, std::false_type{}, lds);
        else go(std::integral_constant<int, UN>{}, std::true_type{}, lds);
    });
    return hipGetLastError();
}


}  // namespace draco
