// Kernel templates of the cyclic encoder E^Cyc (Sec. 3, "Cyclic Code"), shared by the
// per-window-width translation units (one per s, so they compile in parallel).
#pragma once

#include <type_traits>

#include "device_util.hpp"

namespace draco {

// E^Cyc for all nodes: z_n = sum_{t=0}^{2s} W[(n+t) mod P][n] * g_{(n+t) mod P} on packed
// complex coordinates in fp64, W in the factored form described at tap_sum below.  A lane
// keeps the window g_n .. g_{n+2s} of its two complex coordinates in registers
// and slides it down the P rows, so every gradient row is read from HBM once;
// rows 0..2s-1, needed again by the last 2s nodes, are parked in LDS (each lane
// reads back only what it wrote: no barrier).
// W factors as W[k][j] = A_j * rho_t * B_k for k = j + t (t = 0..2s), with REAL taps rho_t: the
// nodes that do not hold gradient k are consecutive on the circle, so every factor
// w^j - w^m of W's closed form is a unit phase times a sine.  A message is therefore
//   z_j = A_j * sum_t rho_t * (B_{j+t} g_{j+t}),
// one complex rotation per gradient row as it enters the window, 2 real multiply-adds per tap and
// complex coordinate (instead of 4), one rotation per output.  B is indexed by the UNWRAPPED row
// j + t < P + 2s (its half-angle phase is not P-periodic).  Every packed encoder below forms
// these products in this order, so their messages agree bit for bit.
// Window entry of unwrapped gradient row kappa for a lane's two complex coordinates.
__device__ __forceinline__ void rotate_in(const CycTaps& tab, int kappa, double x, double y, double z, double w,
                                          double (&re)[2], double (&im)[2]) {
    const double2 B = table_entry(tab.rotB, kappa);
    cmul(B.x, B.y, x, y, re[0], im[0]);
    cmul(B.x, B.y, z, w, re[1], im[1]);
}
// Node n's two message entries from the window: taps on slots (first + t) mod R, then A_n.
template <int R>
__device__ __forceinline__ void tap_sum(const CycTaps& tab, int n, const double (&wre)[R][2], const double (&wim)[R][2],
                                        int first, double& are0, double& aim0, double& are1, double& aim1) {
    double sr0 = 0.0, si0 = 0.0, sr1 = 0.0, si1 = 0.0;
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const int slot = (first + t) % R;
        const double r = table_entry(tab.rho, t);
        sr0 = fma(r, wre[slot][0], sr0);
        si0 = fma(r, wim[slot][0], si0);
        sr1 = fma(r, wre[slot][1], sr1);
        si1 = fma(r, wim[slot][1], si1);
    }
    const double2 A = table_entry(tab.rotA, n);
    cmul(A.x, A.y, sr0, si0, are0, aim0);
    cmul(A.x, A.y, sr1, si1, are1, aim1);
}

// Stores a message entry of node n at column c0: the first word and, on the two-word wire, what
// that rounding lost.
template <bool FULL, int LO>
__device__ __forceinline__ void store_message(float* __restrict__ Z, float* __restrict__ Zlo, int64_t off, double are0,
                                              double aim0, double are1, double aim1, int nout) {
    const float4 hi = make_float4((float)are0, (float)aim0, (float)are1, (float)aim1);
    stx<FULL>(Z + off, hi, nout);
    if constexpr (LO != kLoNone) {
        const float4 lo = make_float4((float)(are0 - (double)hi.x), (float)(aim0 - (double)hi.y),
                                      (float)(are1 - (double)hi.z), (float)(aim1 - (double)hi.w));
        st_lo<FULL, LO>(Zlo, off, hi, lo, nout);
    }
}

// Rows in rounds of R, NB - 1 of them ahead of the arithmetic (a ring of NB register buffers).  Loads and stores alternate
// R at a time; a store and a load in turn (encode_cyc_body) is slower on the line grid, see launch_all_nodes.
template <int S, int NB, bool FULL, int LO>
__device__ __forceinline__ void encode_cyc_rounds_body(const float* __restrict__ G, int64_t ldg, float* __restrict__ Z,
                                                       float* __restrict__ Zlo, int64_t ldm,
                                                       const CycTaps tab, int P, int64_t d, int64_t c0,
                                                       float4* head /* LDS [2S][kBlock] */) {
    constexpr int R = 2 * S + 1;
    const int64_t mlen = 2 * ((d + 1) / 2);
    if (!FULL && c0 >= mlen) return;
    const int nin = FULL ? 4 : clamp4(d - c0);      // gradient floats that exist (the pad of an odd d reads as 0)
    const int nout = FULL ? 4 : clamp4(mlen - c0);  // message floats to write

    double wre[R][2], wim[R][2];  // window slot = row index mod R
    auto put = [&](int slot, const float4& raw, int kappa) {
        rotate_in(tab, kappa, (double)raw.x, (double)raw.y, (double)raw.z, (double)raw.w, wre[slot], wim[slot]);
    };
    // fetch the rows that nodes n0 .. n0+R-1 bring into the window
    auto issue = [&](int n0, float4 (&buf)[R]) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int kk = n0 + uu + 2 * S;
            if (n0 + uu < P) {
                if (kk < P) buf[uu] = ldx<FULL>(G + (int64_t)kk * ldg + c0, nin);
                else buf[uu] = head[(kk - P) * kBlock + threadIdx.x];
            }
        }
    };
    auto consume = [&](int n0, const float4 (&buf)[R]) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int n = n0 + uu;
            if (n < P) {
                put((uu + 2 * S) % R, buf[uu], n + 2 * S);
                double are0, aim0, are1, aim1;
                tap_sum<R>(tab, n, wre, wim, uu % R, are0, aim0, are1, aim1);
                store_message<FULL, LO>(Z, Zlo, (int64_t)n * ldm + c0, are0, aim0, are1, aim1, nout);
            }
        }
    };
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) {
        const float4 raw = ldx<FULL>(G + (int64_t)k * ldg + c0, nin);
        head[k * kBlock + threadIdx.x] = raw;
        put(k, raw, k);
    }
    float4 buf[NB][R];
#pragma unroll
    for (int b = 0; b < NB - 1; ++b)
        if (b * R < P) issue(b * R, buf[b]);
    for (int n0 = 0; n0 < P; n0 += NB * R) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int cur = n0 + b * R;
            if (cur < P) {
                const int nxt = cur + (NB - 1) * R;
                if (nxt < P) issue(nxt, buf[(b + NB - 1) % NB]);
                consume(cur, buf[b]);
            }
        }
    }
}

// D rows are in flight: a row's registers are loaded again as soon as it has entered the window.
template <int S, int D, bool FULL, int LO>
__device__ __forceinline__ void encode_cyc_body(const float* __restrict__ G, int64_t ldg, float* __restrict__ Z,
                                                float* __restrict__ Zlo, int64_t ldm,
                                                const CycTaps tab, int P, int64_t d, int64_t c0,
                                                float4* head /* LDS [2S][kBlock] */) {
    constexpr int R = 2 * S + 1;
    constexpr int U = R * ((D + R - 1) / R);   // nodes per round and slots of the ring: a multiple of R that holds D rows
    const int64_t mlen = 2 * ((d + 1) / 2);
    if (!FULL && c0 >= mlen) return;
    const int nin = FULL ? 4 : clamp4(d - c0);      // gradient floats that exist (the pad of an odd d reads as 0)
    const int nout = FULL ? 4 : clamp4(mlen - c0);  // message floats to write

    double wre[R][2], wim[R][2];  // window slot = row index mod R
    float4 ring[U];               // row n + 2S in slot n mod U
    auto put = [&](int slot, const float4& raw, int kappa) {
        rotate_in(tab, kappa, (double)raw.x, (double)raw.y, (double)raw.z, (double)raw.w, wre[slot], wim[slot]);
    };
    const float* src = G + c0;    // the next row to fetch
    auto fetch = [&]() -> float4 {
        const float4 v = ldx<FULL>(src, nin);
        src += ldg;
        return v;
    };
    auto node = [&](int uu, int n) {   // uu = n mod U: node n, its last row in the window
        double are0, aim0, are1, aim1;
        tap_sum<R>(tab, n, wre, wim, uu % R, are0, aim0, are1, aim1);
        store_message<FULL, LO>(Z, Zlo, (int64_t)n * ldm + c0, are0, aim0, are1, aim1, nout);
    };

    if constexpr (S > 0) {
        float4 raw[2 * S > 0 ? 2 * S : 1];
#pragma unroll
        for (int k = 0; k < 2 * S; ++k) raw[k] = fetch();
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (i + 2 * S < P) ring[i] = fetch();
#pragma unroll
        for (int k = 0; k < 2 * S; ++k) {
            head[k * kBlock + threadIdx.x] = raw[k];
            put(k, raw[k], k);
        }
    } else {
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (i < P) ring[i] = fetch();
    }
    // Nodes 0 .. last-1 fetch a row below P.  No load is under a condition: behind one the compiler cannot
    // count the loads in flight and waits for all of them, and for the stores before them.  The first round is
    // a copy of its own, so that the waits in the loop need not hold for the ring as it was filled, without
    // stores in between.
    const int last = P - 2 * S - D;
    int n0 = 0;
    auto step = [&](int uu) {
        put((uu + 2 * S) % R, ring[uu], n0 + uu + 2 * S);
        ring[(uu + D) % U] = fetch();
        node(uu, n0 + uu);
        if constexpr (S == 6 || S == 7) __builtin_amdgcn_sched_barrier(0);   // (rows loaded any earlier do not fit the registers)
    };
    if (last >= U) {
#pragma unroll
        for (int uu = 0; uu < U; ++uu) step(uu);
        for (n0 = U; n0 + U <= last; n0 += U) {
#pragma unroll
            for (int uu = 0; uu < U; ++uu) step(uu);
        }
    }
#pragma unroll
    for (int uu = 0; uu < U; ++uu) {
        if (n0 + uu >= last) goto rest;
        step(uu);
    }
rest:   // the other nodes: rows that are in flight, then those parked in LDS
    for (; n0 < P; n0 += U) {
#pragma unroll
        for (int uu = 0; uu < U; ++uu) {
            const int n = n0 + uu;
            if (n >= last && n < P) {
                const int kk = n + 2 * S;
                if (kk < P) put((uu + 2 * S) % R, ring[uu], kk);
                else put((uu + 2 * S) % R, head[(kk - P) * kBlock + threadIdx.x], kk);
                node(uu, n);
            }
        }
    }
}

// The kernels are compiled for the workgroups per CU that they are launched with (four wavefronts, one per SIMD, each): left
// alone the compiler gives windows of 11 rows and more over 256 registers, with which a second workgroup does not fit.
// LINES: workgroups own 4 KiB contiguously (device_util.hpp, "rows off the line grid"); else the spread footprint.
template <int S, int D, int LO, bool LINES, int PER_CU>
__global__ __launch_bounds__(kBlock, PER_CU) void encode_cyc_kernel(const float* __restrict__ G, int64_t ldg,
                                                                    float* __restrict__ Z, float* __restrict__ Zlo,
                                                                    int64_t ldm, const CycTaps tab, int P,
                                                                    int64_t d) {
    extern __shared__ float4 head[];  // [2S][kBlock]
    const int64_t mlen = 2 * ((d + 1) / 2);
    constexpr bool SPREAD = kSpreadEncodeCyc && !LINES;
    const int64_t c0 = lane_column<SPREAD>(mlen);
    if (block_is_full<SPREAD>(mlen, d)) encode_cyc_body<S, D, true, LO>(G, ldg, Z, Zlo, ldm, tab, P, d, c0, head);
    else encode_cyc_body<S, D, false, LO>(G, ldg, Z, Zlo, ldm, tab, P, d, c0, head);
}
template <int S, int NB, int LO, int PER_CU>
__global__ __launch_bounds__(kBlock, PER_CU) void encode_cyc_rounds_kernel(const float* __restrict__ G, int64_t ldg,
                                                                           float* __restrict__ Z, float* __restrict__ Zlo,
                                                                           int64_t ldm, const CycTaps tab, int P,
                                                                           int64_t d) {
    extern __shared__ float4 head[];  // [2S][kBlock]
    const int64_t mlen = 2 * ((d + 1) / 2);
    const int64_t c0 = lane_column<kSpreadEncodeCyc>(mlen);
    if (block_is_full<kSpreadEncodeCyc>(mlen, d)) encode_cyc_rounds_body<S, NB, true, LO>(G, ldg, Z, Zlo, ldm, tab, P, d, c0, head);
    else encode_cyc_rounds_body<S, NB, false, LO>(G, ldg, Z, Zlo, ldm, tab, P, d, c0, head);
}

// The same encoder for short rows (node_segment says which).  There the walk down P rows is
// latency: a workgroup (4 KiB contiguous, neighbours on one die) takes only `seg`
// nodes, blockIdx.y the segment, and the rows that neighbouring segments share (2s of them) come
// from the die's L2; no LDS, so the registers alone bound the workgroups per CU.  The tiles of a segment run before the next
// segment's: the chip streams few rows at a time.  The window's rows
// and the first round are in flight together.  Same taps in the same order: identical bits.
// Streaming stores: plain ones end the kernel sooner but leave the messages for the next kernel to
// wait for (whole step unsplit, split with plain stores, split: (45, 3, 500 001) on the 5-byte wire 116,
// 117 and 104 us, (30, 7, 1 000 001) on two fp32 words 155, 186 and 154).
template <int S, bool FULL, int LO, bool MULTI>
__device__ __forceinline__ void encode_cyc_small_body(const float* __restrict__ G, int64_t ldg, int m, float* __restrict__ Z,
                                                      float* __restrict__ Zlo, int64_t ldm, const CycTaps tab, int P,
                                                      int64_t d, int64_t c0, int first, int last) {
    constexpr int R = 2 * S + 1;
    const int64_t mlen = 2 * ((d + 1) / 2);
    if (!FULL && c0 >= mlen) return;
    const int nin = FULL ? 4 : clamp4(d - c0);
    const int nout = FULL ? 4 : clamp4(mlen - c0);
    double wre[R][2], wim[R][2];  // window slot = (row - first) mod R
    using unit_t = typename std::conditional<MULTI, double4, float4>::type;
    auto fetch = [&](int kappa) -> unit_t {   // unit gradient of unwrapped index kappa < P + 2S
        const int k = kappa < P ? kappa : kappa - P;
        if constexpr (MULTI) {   // the sum of its m sample rows, ascending, in fp64
            constexpr int UN = 4;
            double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
            const float* src = G + (int64_t)k * m * ldg + c0;
            for (int i0 = 0; i0 < m; i0 += UN) {
                float4 x[UN];
#pragma unroll
                for (int i = 0; i < UN; ++i)
                    if (i0 + i < m) x[i] = ldx<FULL, false>(src + (int64_t)(i0 + i) * ldg, nin);
#pragma unroll
                for (int i = 0; i < UN; ++i) {
                    if (i0 + i < m) {
                        acc.x += (double)x[i].x;
                        acc.y += (double)x[i].y;
                        acc.z += (double)x[i].z;
                        acc.w += (double)x[i].w;
                    }
                }
            }
            return acc;
        } else {
            return ldx<FULL, false>(G + (int64_t)k * ldg + c0, nin);
        }
    };
    auto put = [&](int slot, const unit_t& v, int kappa) {
        rotate_in(tab, kappa, (double)v.x, (double)v.y, (double)v.z, (double)v.w, wre[slot], wim[slot]);
    };
    unit_t head[2 * S > 0 ? 2 * S : 1], buf[R];
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) head[k] = fetch(first + k);
    auto issue = [&](int n0) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu)
            if (n0 + uu < last) buf[uu] = fetch(n0 + uu + 2 * S);
    };
    issue(first);
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) put(k, head[k], first + k);
    for (int n0 = first; n0 < last; n0 += R) {
        if (n0 != first) issue(n0);
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int n = n0 + uu;
            if (n < last) {
                put((uu + 2 * S) % R, buf[uu], n + 2 * S);
                double are0, aim0, are1, aim1;
                tap_sum<R>(tab, n, wre, wim, uu % R, are0, aim0, are1, aim1);
                store_message<FULL, LO>(Z, Zlo, (int64_t)n * ldm + c0, are0, aim0, are1, aim1, nout);
            }
        }
    }
}

// MULTI: a unit gradient is the sum of m sample rows (B > P).
template <int S, int LO, bool MULTI>
__global__ __launch_bounds__(kBlock) void encode_cyc_small_kernel(const float* __restrict__ G, int64_t ldg, int m,
                                                                  float* __restrict__ Z, float* __restrict__ Zlo,
                                                                  int64_t ldm, const CycTaps tab, int P, int seg,
                                                                  int64_t d) {
    // A segment of the launch has a whole number of workgroups per die (gridDim.x, a multiple of 8), so that all segments of a
    // tile run on one die and find in its L2 the rows that they share; a die has tiles/8 neighbouring tiles, or one more.
    const unsigned tiles = (unsigned)((2 * ((d + 1) / 2) + kBlock * 4 - 1) / (kBlock * 4));
    const unsigned die = blockIdx.x % 8, at = blockIdx.x / 8, more = tiles % 8;
    if (at >= tiles / 8 + (die < more ? 1 : 0)) return;
    const int64_t tile = die * (tiles / 8) + min(die, more) + at;
    const int64_t c0 = (tile * kBlock + threadIdx.x) * 4;
    const int first = (int)blockIdx.y * seg, last = min(P, first + seg);
    if ((tile + 1) * (kBlock * 4) <= d)
        encode_cyc_small_body<S, true, LO, MULTI>(G, ldg, m, Z, Zlo, ldm, tab, P, d, c0, first, last);
    else
        encode_cyc_small_body<S, false, LO, MULTI>(G, ldg, m, Z, Zlo, ldm, tab, P, d, c0, first, last);
}

// The same encoder with a wider lane: a lane owns C float4 of every row (its wavefront's C
// pieces of 1 KiB) and a workgroup's 4C pieces are spread evenly over the 128 KiB footprint
// window -- wavefront v, piece q at (v + 4q) * (32 KiB / C) -- so a compute unit has more
// distinct channels in flight at a time.  One row of loads is issued per finished row, D
// rows ahead (a ring of raw rows whose slot is the row index mod the unroll length).  Same
// taps in the same order as encode_cyc_body: identical bits.  Registers hold the window of
// C lanes' worth (R*C*8 doubles), so this form is for narrow windows.
// Measured at (P, s, d) = (45, 3, 25.6 M), one word per float: C = 4, D = 2 runs at 6.1 TB/s
// against 5.9 for encode_cyc_body on the same footprint window (and 5.65 contiguous); with an
// 8-bit second word 1750 us against 1770; with a 16- or 32-bit second word it gains nothing.
template <int S, int C, int D, int LO>
__device__ __forceinline__ void encode_cyc_strip_body(const float* __restrict__ G, int64_t ldg,
                                                      float* __restrict__ Z, float* __restrict__ Zlo, int64_t ldm,
                                                      const CycTaps tab, int P, int64_t d,
                                                      float4* head /* LDS [2S][C][kBlock] */,
                                                      const int64_t (&cq)[C]) {
    constexpr int R = 2 * S + 1;
    constexpr int U = R * ((D + R - 1) / R);  // unroll length and ring size: a multiple of R that holds D rows
    double wre[C][R][2], wim[C][R][2];  // [piece][window slot = row index mod R]
    auto put = [&](int slot, const float4 (&raw)[C], int kappa) {
#pragma unroll
        for (int q = 0; q < C; ++q)
            rotate_in(tab, kappa, (double)raw[q].x, (double)raw[q].y, (double)raw[q].z, (double)raw[q].w,
                      wre[q][slot], wim[q][slot]);
    };
    auto fetch = [&](int k, float4 (&dst)[C]) {  // row k; k >= P wraps to the rows parked in LDS
        if (k < P) {
#pragma unroll
            for (int q = 0; q < C; ++q)
                dst[q] = ld4(G + (int64_t)k * ldg + cq[q]);
        } else {
#pragma unroll
            for (int q = 0; q < C; ++q) dst[q] = head[((k - P) * C + q) * kBlock + threadIdx.x];
        }
    };
    float4 ring[U][C];
    {
        float4 row[C];
#pragma unroll
        for (int k = 0; k < 2 * S; ++k) {
            fetch(k, row);
#pragma unroll
            for (int q = 0; q < C; ++q) head[(k * C + q) * kBlock + threadIdx.x] = row[q];
            put(k, row, k);
        }
    }
#pragma unroll
    for (int i = 0; i < D; ++i)
        if (i < P) fetch(i + 2 * S, ring[i]);
    for (int n0 = 0; n0 < P; n0 += U) {
#pragma unroll
        for (int uu = 0; uu < U; ++uu) {
            const int n = n0 + uu;
            if (n < P) {
                put((uu + 2 * S) % R, ring[uu], n + 2 * S);
                if (n + D < P) fetch(n + D + 2 * S, ring[(uu + D) % U]);
#pragma unroll
                for (int q = 0; q < C; ++q) {
                    double are0, aim0, are1, aim1;
                    tap_sum<R>(tab, n, wre[q], wim[q], uu % R, are0, aim0, are1, aim1);
                    store_message<true, LO>(Z, Zlo, (int64_t)n * ldm + cq[q], are0, aim0, are1, aim1, 4);
                }
            }
        }
    }
}

template <int S, int C, int D, int REST, int LO>
__global__ __launch_bounds__(kBlock) void encode_cyc_strip_kernel(const float* __restrict__ G, int64_t ldg,
                                                                  float* __restrict__ Z, float* __restrict__ Zlo,
                                                                  int64_t ldm,
                                                                  const CycTaps tab, int P,
                                                                  int64_t d) {
    extern __shared__ float4 head[];  // [2S][C][kBlock]
    constexpr int64_t u = kWindow / (4 * C);   // floats between neighbouring pieces of the workgroup
    constexpr int64_t per = u / 256;           // workgroups per window
    const int64_t windows = d / kWindow;       // whole ones; the rest of the row in contiguous 4 KiB, first
    const int64_t tile = (int64_t)blockIdx.x - ((int64_t)gridDim.x - windows * per);
    if (tile < 0) {
        const int64_t base = windows * kWindow + (int64_t)blockIdx.x * (kBlock * 4);
        const int64_t c0 = base + threadIdx.x * 4;
        if (base + kBlock * 4 <= d) encode_cyc_body<S, REST, true, LO>(G, ldg, Z, Zlo, ldm, tab, P, d, c0, head);
        else encode_cyc_body<S, REST, false, LO>(G, ldg, Z, Zlo, ldm, tab, P, d, c0, head);
        return;
    }
    const int64_t base = (tile / per) * kWindow + (tile % per) * 256;
    int64_t cq[C];
#pragma unroll
    for (int q = 0; q < C; ++q) cq[q] = base + ((threadIdx.x >> 6) + 4 * q) * u + (threadIdx.x & 63) * 4;
    encode_cyc_strip_body<S, C, D, LO>(G, ldg, Z, Zlo, ldm, tab, P, d, head, cq);
}
// Workgroups of encode_cyc_strip_kernel<S, C, D> for gradients of d floats.
template <int C>
inline unsigned strip_grid(int64_t d) {
    const int64_t windows = d / kWindow, rest = 2 * ((d + 1) / 2) - windows * kWindow;
    return (unsigned)(windows * (kWindow / (4 * C) / 256)) + grid_for((rest + 3) / 4);
}

// E^Cyc on the real gradients as Sec. 3 states it, without the packing remark that closes
// the section: z_n = sum_t coef[n][t] * g_{(n+t) mod P} with real g, so a message has d
// complex entries (2d floats, re/im interleaved).  Same sliding window and ring of rows in flight
// as above, on four reals per lane instead of two complex numbers (two FMAs per tap and
// coordinate).  A message row is twice as long as a gradient row, so a lane owns two PAIRS
// of real coordinates half a wavefront span apart (8-byte loads): their complex outputs
// are 16 bytes each and every store instruction of a wavefront writes 1 KiB contiguously.
template <int S, int D, bool FULL>
__device__ __forceinline__ void encode_cyc_real_body(const float* __restrict__ G, int64_t ldg,
                                                     float* __restrict__ Z, int64_t ldm,
                                                     const double2* __restrict__ coef, int P, int64_t d, int64_t c0,
                                                     float4* head /* LDS [2S][kBlock] */) {
    constexpr int R = 2 * S + 1;
    constexpr int U = R * ((D + R - 1) / R);
    // the wavefront covers 256 consecutive real coordinates; mine are cA, cA+1, cA+128, cA+129
    const int64_t cA = c0 - (threadIdx.x & 63) * 2;
    const int64_t cB = cA + 128;
    if (!FULL && cA >= d) return;
    const int nA = FULL ? 2 : (d - cA >= 2 ? 2 : (int)(d - cA));
    const int nB = FULL ? 2 : (d - cB >= 2 ? 2 : (d - cB <= 0 ? 0 : (int)(d - cB)));

    const float* src = G + cA;   // the next row to fetch
    auto fetch = [&]() -> float4 {
        float2 a, b;
        if constexpr (FULL) {
            a = ld2(src);
            b = ld2(src + 128);
        } else {
            a = ld2_partial(src, nA);
            b = ld2_partial(src + 128, nB);
        }
        src += ldg;
        return make_float4(a.x, a.y, b.x, b.y);
    };

    double w[R][4];   // window slot = row index mod R
    float4 ring[U];   // row n + 2S in slot n mod U
    auto put = [&](int slot, const float4& raw) {
        w[slot][0] = (double)raw.x;
        w[slot][1] = (double)raw.y;
        w[slot][2] = (double)raw.z;
        w[slot][3] = (double)raw.w;
    };
    auto node = [&](int uu, int n) {
        const double2* cn = coef + (int64_t)n * R;
        double re[4] = {0.0, 0.0, 0.0, 0.0}, im[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const int slot = (uu + t) % R;
            const double2 c_nt = table_entry(cn, t);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                re[c] = fma(c_nt.x, w[slot][c], re[c]);
                im[c] = fma(c_nt.y, w[slot][c], im[c]);
            }
        }
        float* dst = Z + (int64_t)n * ldm;
        stx<FULL>(dst + 2 * cA, make_float4((float)re[0], (float)im[0], (float)re[1], (float)im[1]), 2 * nA);
        stx<FULL>(dst + 2 * cB, make_float4((float)re[2], (float)im[2], (float)re[3], (float)im[3]), 2 * nB);
    };

    float4 raw[2 * S > 0 ? 2 * S : 1];
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) raw[k] = fetch();
#pragma unroll
    for (int i = 0; i < D; ++i)
        if (i + 2 * S < P) ring[i] = fetch();
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) {
        head[k * kBlock + threadIdx.x] = raw[k];
        put(k, raw[k]);
    }
    // rounds without a load under a condition, then what is in flight, then what is parked: see encode_cyc_body
    const int last = P - 2 * S - D;
    int n0 = 0;
    auto step = [&](int uu) {
        put((uu + 2 * S) % R, ring[uu]);
        ring[(uu + D) % U] = fetch();
        node(uu, n0 + uu);
        if constexpr (S == 10) __builtin_amdgcn_sched_barrier(0);   // (rows loaded any earlier go to scratch memory)
    };
    if (last >= U) {
#pragma unroll
        for (int uu = 0; uu < U; ++uu) step(uu);
        for (n0 = U; n0 + U <= last; n0 += U) {
#pragma unroll
            for (int uu = 0; uu < U; ++uu) step(uu);
        }
    }
#pragma unroll
    for (int uu = 0; uu < U; ++uu) {
        if (n0 + uu >= last) goto rest;
        step(uu);
    }
rest:
    for (; n0 < P; n0 += U) {
#pragma unroll
        for (int uu = 0; uu < U; ++uu) {
            const int n = n0 + uu;
            if (n >= last && n < P) {
                const int kk = n + 2 * S;
                if (kk < P) put((uu + 2 * S) % R, ring[uu]);
                else put((uu + 2 * S) % R, head[(kk - P) * kBlock + threadIdx.x]);
                node(uu, n);
            }
        }
    }
}

template <int S, int D, bool LINES, int PER_CU>
__global__ __launch_bounds__(kBlock, PER_CU) void encode_cyc_real_kernel(const float* __restrict__ G, int64_t ldg,
                                                                         float* __restrict__ Z, int64_t ldm,
                                                                         const double2* __restrict__ coef, int P,
                                                                         int64_t d) {
    extern __shared__ float4 head[];  // [2S][kBlock]
    constexpr bool SPREAD = kSpreadEncodeCyc && !LINES;
    const int64_t c0 = lane_column<SPREAD>(d);
    if (block_is_full<SPREAD>(d, d)) encode_cyc_real_body<S, D, true>(G, ldg, Z, ldm, coef, P, d, c0, head);
    else encode_cyc_real_body<S, D, false>(G, ldg, Z, ldm, coef, P, d, c0, head);
}

// E^Cyc when every unit gradient is the sum of m = B/P per-sample gradients (rows k*m ..
// k*m+m-1 of the sample slab): the same sliding window, but a window entry is the fp64
// sum of m rows, formed as the rows arrive; the first 2s unit sums are parked in LDS in
// fp64 for the wrap-around.  Units are fetched one round ahead.
template <int S, int LO>
__device__ __forceinline__ void encode_cyc_multi_body(const float* __restrict__ G, int64_t ldg, int m,
                                                      float* __restrict__ Z, float* __restrict__ Zlo, int64_t ldm,
                                                      const CycTaps tab, int P,
                                                      int64_t c0, double4* head /* LDS [2S][kBlock] */) {
    constexpr int R = 2 * S + 1;
    constexpr int UN = 4;

    double wre[R][2], wim[R][2];
    auto put = [&](int slot, const double4& v, int kappa) {
        rotate_in(tab, kappa, v.x, v.y, v.z, v.w, wre[slot], wim[slot]);
    };
    auto unit_sum = [&](int k) -> double4 {  // g_k = sum of its m sample rows, ascending, in fp64
        double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
        const float* src = G + (int64_t)k * m * ldg + c0;
        for (int i0 = 0; i0 < m; i0 += UN) {
            float4 x[UN];
#pragma unroll
            for (int i = 0; i < UN; ++i)
                if (i0 + i < m) x[i] = ld4(src + (int64_t)(i0 + i) * ldg);
#pragma unroll
            for (int i = 0; i < UN; ++i) {
                if (i0 + i < m) {
                    acc.x += (double)x[i].x;
                    acc.y += (double)x[i].y;
                    acc.z += (double)x[i].z;
                    acc.w += (double)x[i].w;
                }
            }
        }
        return acc;
    };
    auto issue = [&](int n0, double4 (&buf)[R]) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int kk = n0 + uu + 2 * S;
            if (n0 + uu < P) {
                if (kk < P) buf[uu] = unit_sum(kk);
                else buf[uu] = head[(kk - P) * kBlock + threadIdx.x];
            }
        }
    };
    auto consume = [&](int n0, const double4 (&buf)[R]) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int n = n0 + uu;
            if (n < P) {
                put((uu + 2 * S) % R, buf[uu], n + 2 * S);
                double are0, aim0, are1, aim1;
                tap_sum<R>(tab, n, wre, wim, uu % R, are0, aim0, are1, aim1);
                store_message<true, LO>(Z, Zlo, (int64_t)n * ldm + c0, are0, aim0, are1, aim1, 4);
            }
        }
    };
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) {
        const double4 v = unit_sum(k);
        head[k * kBlock + threadIdx.x] = v;
        put(k, v, k);
    }
    double4 bufA[R], bufB[R];
    issue(0, bufA);
    for (int n0 = 0; n0 < P; n0 += 2 * R) {
        if (n0 + R < P) issue(n0 + R, bufB);
        consume(n0, bufA);
        if (n0 + R < P) {
            if (n0 + 2 * R < P) issue(n0 + 2 * R, bufA);
            consume(n0 + R, bufB);
        }
    }
}

// The same one unit at a time, the first UN rows of the next one in flight: 138 registers at s = 5 where
// two rounds of unit sums take 290 and leave one wavefront per SIMD ((45, 5, 2, 1 998 848): 450 us and 241; the
// narrower windows fit twice as they are, LDS holds the wider ones to one workgroup per CU).
template <int S, int LO>
__device__ __forceinline__ void encode_cyc_multi_ahead_body(const float* __restrict__ G, int64_t ldg, int m,
                                                            float* __restrict__ Z, float* __restrict__ Zlo,
                                                            int64_t ldm, const CycTaps tab, int P, int64_t c0,
                                                            double4* head /* LDS [2S][kBlock] */) {
    constexpr int R = 2 * S + 1;
    constexpr int UN = 4;

    double wre[R][2], wim[R][2];
    auto put = [&](int slot, const double4& v, int kappa) {
        rotate_in(tab, kappa, v.x, v.y, v.z, v.w, wre[slot], wim[slot]);
    };
    // the first UN rows of a unit are fetched while the one before it is encoded
    float4 ahead[UN];
    auto fetch = [&](int k) {
#pragma unroll
        for (int i = 0; i < UN; ++i)
            if (i < m) ahead[i] = ld4(G + ((int64_t)k * m + i) * ldg + c0);
    };
    auto unit_sum = [&](int k) -> double4 {  // g_k = sum of its m sample rows, ascending, in fp64
        double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
        auto add = [&](const float4& x) {
            acc.x += (double)x.x;
            acc.y += (double)x.y;
            acc.z += (double)x.z;
            acc.w += (double)x.w;
        };
#pragma unroll
        for (int i = 0; i < UN; ++i)
            if (i < m) add(ahead[i]);
        const float* src = G + (int64_t)k * m * ldg + c0;
        for (int i0 = UN; i0 < m; i0 += UN) {
            float4 x[UN];
#pragma unroll
            for (int i = 0; i < UN; ++i)
                if (i0 + i < m) x[i] = ld4(src + (int64_t)(i0 + i) * ldg);
#pragma unroll
            for (int i = 0; i < UN; ++i)
                if (i0 + i < m) add(x[i]);
        }
        if (k + 1 < P) fetch(k + 1);
        return acc;
    };
    fetch(0);
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) {
        const double4 v = unit_sum(k);
        head[k * kBlock + threadIdx.x] = v;
        put(k, v, k);
    }
    for (int n0 = 0; n0 < P; n0 += R) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int n = n0 + uu;
            if (n < P) {
                const int kk = n + 2 * S;
                const double4 v = kk < P ? unit_sum(kk) : head[(kk - P) * kBlock + threadIdx.x];
                put((uu + 2 * S) % R, v, kk);
                double are0, aim0, are1, aim1;
                tap_sum<R>(tab, n, wre, wim, uu % R, are0, aim0, are1, aim1);
                store_message<true, LO>(Z, Zlo, (int64_t)n * ldm + c0, are0, aim0, are1, aim1, 4);
            }
        }
    }
}

// The same when m is a multiple of D: the B = m P sample rows are consumed in one linear
// walk with the next D rows always in flight (a ring of D raw rows whose slot is the row
// index mod D, static because m is a multiple of D), so the loads of the next unit overlap
// the sums of this one.  Same additions in the same order as above: identical bits.
template <int S, int D, int LO>
__device__ __forceinline__ void encode_cyc_multi_ring_body(const float* __restrict__ G, int64_t ldg, int m,
                                                           float* __restrict__ Z, float* __restrict__ Zlo,
                                                           int64_t ldm, const CycTaps tab, int P, int64_t c0,
                                                           double4* head /* LDS [2S][kBlock] */) {
    constexpr int R = 2 * S + 1;
    const int64_t rows = (int64_t)P * m;

    float4 ring[D];
    int64_t next = 0;  // next sample row to fetch
    const float* src = G + c0;
#pragma unroll
    for (int t = 0; t < D; ++t) {
        ring[t] = ld4(src + next * ldg);
        ++next;
    }
    auto unit_sum = [&]() -> double4 {  // the next unit gradient: its m rows, ascending, in fp64
        double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
        for (int t0 = 0; t0 < m; t0 += D) {
#pragma unroll
            for (int t = 0; t < D; ++t) {
                const float4 x = ring[t];
                if (next < rows) ring[t] = ld4(src + next * ldg);
                ++next;
                acc.x += (double)x.x;
                acc.y += (double)x.y;
                acc.z += (double)x.z;
                acc.w += (double)x.w;
            }
        }
        return acc;
    };
    double wre[R][2], wim[R][2];
    auto put = [&](int slot, const double4& v, int kappa) {
        rotate_in(tab, kappa, v.x, v.y, v.z, v.w, wre[slot], wim[slot]);
    };
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) {
        const double4 v = unit_sum();
        head[k * kBlock + threadIdx.x] = v;
        put(k, v, k);
    }
    for (int n0 = 0; n0 < P; n0 += R) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int n = n0 + uu;
            if (n < P) {
                const int kk = n + 2 * S;
                const double4 v = kk < P ? unit_sum() : head[(kk - P) * kBlock + threadIdx.x];
                put((uu + 2 * S) % R, v, kk);
                double are0, aim0, are1, aim1;
                tap_sum<R>(tab, n, wre, wim, uu % R, are0, aim0, are1, aim1);
                store_message<true, LO>(Z, Zlo, (int64_t)n * ldm + c0, are0, aim0, are1, aim1, 4);
            }
        }
    }
}

// m = 4 (the paper's B = 180 on P = 45): one unit's four rows in flight, fetched again as soon as they are summed.
// Structure, and the reasons for it, as in encode_cyc_body: rounds of R units without a load under a
// condition, the first one a copy of its own, then the unit whose rows are in flight, then those parked in LDS.
// At (45, 5, B = 180, 25.6 M) on the 5-byte wire with one workgroup per CU 4247 us; two or three units in flight 4292 and
// 4399, two workgroups per CU 4445, two units behind conditions (as the ring above) on two workgroups 4309.  (Those two are
// still the shorter ones where a launch has two workgroups per CU at most: (45, 5, B = 180, 500 001) 84 us, now 91.)
template <int S, int LO>
__device__ __forceinline__ void encode_cyc_multi_four_body(const float* __restrict__ G, int64_t ldg,
                                                           float* __restrict__ Z, float* __restrict__ Zlo,
                                                           int64_t ldm, const CycTaps tab, int P, int64_t c0,
                                                           double4* head /* LDS [2S][kBlock] */) {
    constexpr int R = 2 * S + 1;
    float4 rows[4];
    const float* src = G + c0;   // next sample row to fetch
    auto fetch = [&]() {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            rows[t] = ld4(src);
            src += ldg;
        }
    };
    auto unit_sum = [&]() -> double4 {  // a unit gradient: its 4 rows, ascending, in fp64
        double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc.x += (double)rows[t].x;
            acc.y += (double)rows[t].y;
            acc.z += (double)rows[t].z;
            acc.w += (double)rows[t].w;
        }
        return acc;
    };
    double wre[R][2], wim[R][2];
    auto put = [&](int slot, const double4& v, int kappa) {
        rotate_in(tab, kappa, v.x, v.y, v.z, v.w, wre[slot], wim[slot]);
    };
    auto node = [&](int uu, int n) {
        double are0, aim0, are1, aim1;
        tap_sum<R>(tab, n, wre, wim, uu, are0, aim0, are1, aim1);
        store_message<true, LO>(Z, Zlo, (int64_t)n * ldm + c0, are0, aim0, are1, aim1, 4);
    };
    fetch();
#pragma unroll
    for (int k = 0; k < 2 * S; ++k) {
        const double4 v = unit_sum();
        fetch();   // unit k + 1 <= 2S < P
        head[k * kBlock + threadIdx.x] = v;
        put(k, v, k);
    }
    const int last = P - 2 * S - 1;   // nodes below it fetch a unit below P
    int n0 = 0;
    auto step = [&](int uu) {
        const double4 v = unit_sum();
        fetch();
        put((uu + 2 * S) % R, v, n0 + uu + 2 * S);
        node(uu, n0 + uu);
    };
    if (last >= R) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) step(uu);
        for (n0 = R; n0 + R <= last; n0 += R) {
#pragma unroll
            for (int uu = 0; uu < R; ++uu) step(uu);
        }
    }
#pragma unroll
    for (int uu = 0; uu < R; ++uu) {
        if (n0 + uu >= last) goto rest;
        step(uu);
    }
rest:
    for (; n0 < P; n0 += R) {
#pragma unroll
        for (int uu = 0; uu < R; ++uu) {
            const int n = n0 + uu;
            if (n >= last && n < P) {
                const int kk = n + 2 * S;
                if (kk < P) put((uu + 2 * S) % R, unit_sum(), kk);
                else put((uu + 2 * S) % R, head[(kk - P) * kBlock + threadIdx.x], kk);
                node(uu, n);
            }
        }
    }
}

// The last d mod 4 floats of every row, which no whole vector covers: a workgroup of their own (the
// last of the launch, only if there are any), a lane per unit gradient, then a lane per node.  As
// lanes of a row's last workgroup they made that one walk all rows behind guarded loads, one memory
// latency after the other, longer than the rest of the launch ((45, 2, B = 180, 400 001): 80 us against
// 67 for 393 216).
template <int S, int LO>
__device__ __forceinline__ void encode_cyc_multi_tail(const float* __restrict__ G, int64_t ldg, int m,
                                                      float* __restrict__ Z, float* __restrict__ Zlo, int64_t ldm,
                                                      const CycTaps tab, int P, int64_t d,
                                                      double4* units /* LDS [P] */) {
    constexpr int R = 2 * S + 1;
    constexpr int UN = 8;
    const int64_t c0 = d / 4 * 4;
    const int nin = (int)(d - c0), k = threadIdx.x;   // 1 .. 3 floats (the pad of an odd d reads as 0)
    if (k < P) {
        double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
        const float* src = G + (int64_t)k * m * ldg + c0;
        for (int i0 = 0; i0 < m; i0 += UN) {
            float x[UN], y[UN], z[UN];
#pragma unroll
            for (int i = 0; i < UN; ++i) {
                const float* row = src + (int64_t)min(i0 + i, m - 1) * ldg;
                x[i] = row[0];
                y[i] = nin > 1 ? row[1] : 0.f;
                z[i] = nin > 2 ? row[2] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < UN; ++i) {
                if (i0 + i < m) {
                    acc.x += (double)x[i];
                    acc.y += (double)y[i];
                    acc.z += (double)z[i];
                }
            }
        }
        units[k] = acc;
    }
    __syncthreads();
    if (k < P) {
        double wre[R][2], wim[R][2], are0, aim0, are1, aim1;
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const double4 v = units[k + t < P ? k + t : k + t - P];
            rotate_in(tab, k + t, v.x, v.y, v.z, v.w, wre[t], wim[t]);
        }
        tap_sum<R>(tab, k, wre, wim, 0, are0, aim0, are1, aim1);
        store_message<false, LO>(Z, Zlo, (int64_t)k * ldm + c0, are0, aim0, are1, aim1, (nin + 1) / 2 * 2);
    }
}

// Workgroups that share the whole vectors of a row, and this lane's column among them (device_util.hpp, "rows off the line
// grid").  lines: 0 the spread footprint, on the line grid; off it contiguous 4 KiB (1), with neighbours on one die (2) where
// two workgroups per CU walk rows that are always in flight, but for long rows on few nodes.  Encoder in us, contiguous /
// spread / contiguous with neighbours on one die: one workgroup per CU, (45, 3, B = 4P, 3.7 M + 1) 732 / 793 / 902, (45, 5,
// B = 4P, 3 M + 1) 569 / 616 / 577; two, (45, 3, B = 8P, 1 M + 1) 331 / 344 / 319, (45, 3, B = 4P, 800 001) 155 / 163 / 147, (10, 3,
// B = 8P, 4 M + 1) 272 / - / 286; rows not always in flight, (45, 5, B = 2P, 3.7 M + 1) on two fp32 words 618 / 635 / 776.
__device__ __forceinline__ unsigned multi_blocks(int64_t d) { return gridDim.x - (d % 4 != 0 ? 1u : 0u); }
__device__ __forceinline__ int64_t multi_column(int lines, int64_t d) {
    if (lines == 2) return (xcd_tile(multi_blocks(d)) * kBlock + threadIdx.x) * 4;
    if (lines == 1) return ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
    return lane_column<kSpreadEncodeCyc>(d / 4 * 4, multi_blocks(d));
}

template <int S, int LO>
__global__ __launch_bounds__(kBlock) void encode_cyc_multi_four_kernel(const float* __restrict__ G, int64_t ldg,
                                                                       float* __restrict__ Z, float* __restrict__ Zlo,
                                                                       int64_t ldm, const CycTaps tab,
                                                                       int P, int lines, int64_t d) {
    extern __shared__ double4 head_sums[];  // [2S][kBlock], or a row of units
    if (blockIdx.x == multi_blocks(d)) {
        encode_cyc_multi_tail<S, LO>(G, ldg, 4, Z, Zlo, ldm, tab, P, d, head_sums);
        return;
    }
    const int64_t c0 = multi_column(lines, d);
    if (c0 + 4 > d) return;
    encode_cyc_multi_four_body<S, LO>(G, ldg, Z, Zlo, ldm, tab, P, c0, head_sums);
}

template <int S, int D, int LO>
__global__ __launch_bounds__(kBlock) void encode_cyc_multi_ring_kernel(const float* __restrict__ G, int64_t ldg, int m,
                                                                       float* __restrict__ Z, float* __restrict__ Zlo,
                                                                       int64_t ldm, const CycTaps tab,
                                                                       int P, int lines, int64_t d) {
    extern __shared__ double4 head_sums[];  // [2S][kBlock], or a row of units
    if (blockIdx.x == multi_blocks(d)) {
        encode_cyc_multi_tail<S, LO>(G, ldg, m, Z, Zlo, ldm, tab, P, d, head_sums);
        return;
    }
    const int64_t c0 = multi_column(lines, d);
    if (c0 + 4 > d) return;
    encode_cyc_multi_ring_body<S, D, LO>(G, ldg, m, Z, Zlo, ldm, tab, P, c0, head_sums);
}

template <int S, int LO>
__global__ __launch_bounds__(kBlock) void encode_cyc_multi_kernel(const float* __restrict__ G, int64_t ldg, int m,
                                                                       float* __restrict__ Z, float* __restrict__ Zlo,
                                                                       int64_t ldm, const CycTaps tab,
                                                                       int P, int lines, int64_t d) {
    extern __shared__ double4 head_sums[];  // [2S][kBlock], or a row of units
    if (blockIdx.x == multi_blocks(d)) {
        encode_cyc_multi_tail<S, LO>(G, ldg, m, Z, Zlo, ldm, tab, P, d, head_sums);
        return;
    }
    const int64_t c0 = multi_column(lines, d);
    if (c0 + 4 > d) return;
    if constexpr (S == 5) encode_cyc_multi_ahead_body<S, LO>(G, ldg, m, Z, Zlo, ldm, tab, P, c0, head_sums);
    else encode_cyc_multi_body<S, LO>(G, ldg, m, Z, Zlo, ldm, tab, P, c0, head_sums);
}


// Launch of the all-node encoder for one s (defined in the translation unit of that s).
// lo: format of the second word when Zlo is not null.
template <int S>
hipError_t launch_encode_cyc_s(hipStream_t stream, const float* G, int64_t ldg, float* Z,
                               float* Zlo, int lo, int64_t ldm, const CycTaps& tab, int P, int64_t d);
// Same for the unpacked wire (real gradients in, d complex entries out).
template <int S>
hipError_t launch_encode_cyc_real_s(hipStream_t stream, const float* G, int64_t ldg, float* Z,
                                    int64_t ldm, const double2* coef, int P, int64_t d);
// Same for the B > P form (m per-sample rows per unit gradient).
template <int S>
hipError_t launch_encode_cyc_multi_s(hipStream_t stream, const float* G, int64_t ldg, int m, float* Z,
                                     float* Zlo, int lo, int64_t ldm, const CycTaps& tab, int P, int64_t d);

}  // namespace draco
