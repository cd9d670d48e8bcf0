// Device-side phi and recombination vector of the cyclic code (Sec. 3, phi; Algorithm 1,
// lines 1-3): the same steps as host_math.cpp, run by ONE wavefront in fp64 so that a cyclic
// decode needs no host round trip.
//
//   gamma[P] (projections f R)  ->  mask words, status, and the honest nodes'
//   indices and coefficients b (compacted, ascending) for the recombination.
//
// The work is a chain of small dependent steps, so its time is latency, not throughput: a
// dependent LDS access costs over 100 cycles here, a dependent fp64 instruction about 8, an
// integer division or an IEEE fp64 division about 150.  What keeps the chain short:
//   * a lane owns node j (j = lane, lane+64, ...) and keeps its projection and its root of unity; up to 64 nodes
//     the median compares lanes with lanes (v_readlane), and eight syndromes are summed over the wavefront together;
//   * the usual case of s <= 7 takes neither the recurrence nor the transform nor the ranking (locate_exact), and one
//     orthonormal basis serves its check and b; the general form below remains for what that cannot settle;
//   * t = C h is evaluated by Horner's rule (even and odd powers: two chains) from the lane's own
//     root of unity, so nothing is gathered from the table of roots;
//   * the recurrence scatters each new value into the S pending ones instead of gathering S old
//     values, so one multiply-add is on its critical path;
//   * beta comes from a pivoted QR factorisation, a lane group per column; only where that leaves
//     the rank open do Jacobi sweeps run, and those rotate column pairs that share no column at the
//     same time (a round-robin tournament), A in one half of a lane group and V in the other;
//   * orthonormal columns are kept in registers, spread over the lane groups, and a new column is
//     made orthogonal to all of them at once (classical Gram-Schmidt, twice);
//   * sums over lanes are DPP row operations and v_permlane swaps, never LDS.
// Measured with the code in the instruction cache (the first call of a kernel takes 1 200 to 6 000 cycles more), one call in cycles at
// 2.3 GHz: (P, s, liars) = (45, 3, 0) 3 700, (45, 3, 1) 7 600, (45, 3, 3) 13 900, (45, 7, 4) 17 500, (15, 2, 2) 9 100, (32, 4, 1) 7 400,
// (40, 8, 3) 29 900, (45, 10, 5) 250 000.  Of the 13 900 the median takes 1 800 and locate_exact 9 200, b's coefficients included, for
// which the general form takes 22 800 (QR 5 800); of the 250 000 the Jacobi sweeps 222 000 and the recurrence 5 400.
// Limits: P <= 256, s <= kLocateMaxS.
#pragma once

#include <cfloat>
#include <type_traits>
#include <utility>

#include "host_math.hpp"
#include "kernels.hpp"
#include "wave_reduce.hpp"

namespace draco {
namespace {

constexpr int kW = 64;  // one wavefront

// Orders this wavefront's LDS accesses (the hardware executes them in order): what other lanes
// stored before is visible after.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// The same sizes, lane and node as far as the compiler can tell others: what a block derives from them it then computes
// itself.  (Out of the loop over the passes it moves everything that does not change, the rare branches' shares too,
// some 3000 cycles before the first sum.)
__device__ __forceinline__ void only_here(int& P, int& s, int& lane) {
    P = __builtin_amdgcn_readfirstlane(P);
    s = __builtin_amdgcn_readfirstlane(s);
    asm volatile("" : "+s"(P), "+s"(s), "+v"(lane));
}
__device__ __forceinline__ bool lane0_says(bool b) { return __builtin_amdgcn_readfirstlane(b ? 1 : 0) != 0; }

// Several kernels locate, and b has to be the same from each: products and sums are fused here where they are written so and
// nowhere else.
#pragma clang fp contract(off)

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(fma(-a.y, b.y, a.x * b.x), fma(a.y, b.x, a.x * b.y));
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double cnorm2(double2 a) { return fma(a.y, a.y, a.x * a.x); }
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
template <int N>
__device__ __forceinline__ double2 group_sum_c(double2 a) {
    double v[2] = {a.x, a.y};
    group_sums<N>(v);
    return make_double2(v[0], v[1]);
}
// acc + a * b with fused multiply-adds (two deep per component)
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 acc) {
    return make_double2(fma(-a.y, b.y, fma(a.x, b.x, acc.x)), fma(a.y, b.x, fma(a.x, b.y, acc.y)));
}
// 1/sqrt(x) for positive, finite, normal x: the hardware's estimate refined by two Newton steps
// (the library form costs three to four times the latency)
__device__ __forceinline__ double rsqrt_pos(double x) {
    double r = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x;
    r = r * fma(-hx * r, r, 1.5);
    r = r * fma(-hx * r, r, 1.5);
    return r;
}
// 1/x likewise
__device__ __forceinline__ double rcp_pos(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}
// (a + b) mod P for 0 <= a, b < P
__device__ __forceinline__ int addmod(int a, int b, int P) {
    const int c = a + b;
    return c >= P ? c - P : c;
}
// a * b mod P for 0 <= a, b < P <= 256: the product is below 2^16, so the fp32 quotient is off by
// at most one
__device__ __forceinline__ int mulmod(int a, int b, int P) {
    const int x = a * b;
    int r = x - (int)((float)x * __builtin_amdgcn_rcpf((float)P)) * P;
    r = r < 0 ? r + P : r;
    return r >= P ? r - P : r;
}

struct LocateSmem {
    double2 root[kMaxNodes];  // exp(2 pi i k / P)
    double2 gam[kMaxNodes];
    double2 h[kMaxNodes];
    alignas(16) double sq[kMaxNodes];          // |gamma_j|^2, padded to a multiple of 8 (more than 64 nodes)
    double2 A[kLocateMaxS * kLocateMaxS];      // column-major s x s
    double2 V[kLocateMaxS * kLocateMaxS];
    double2 hk[2 * kLocateMaxS];
    double2 beta[kLocateMaxS];
    double2 coef[kLocateMaxS];
    double inv[kLocateMaxS];
    int order[kLocateMaxS];
};

// A set of nodes, the same in every lane: bit j of word j / 64.
template <int CH>
struct NodeSet {
    uint64_t word[CH];
    __device__ __forceinline__ bool has(int c, int lane) const { return ((word[c] >> lane) & 1ull) != 0; }
    __device__ __forceinline__ void add(int j) {
#pragma unroll
        for (int c = 0; c < CH; ++c) word[c] |= j / kW == c ? 1ull << (j % kW) : 0ull;
    }
    __device__ __forceinline__ int count() const {
        int n = 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) n += __popcll(word[c]);
        return n;
    }
    __device__ __forceinline__ int take_first() {   // the lowest node, taken out; -1 if there is none
        int v = -1;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (v < 0 && word[c] != 0) {
                v = c * kW + __builtin_ctzll(word[c]);
                word[c] &= word[c] - 1;
            }
        }
        return v;
    }
};


template <class F, int... K>
__device__ __forceinline__ void unroll_slots(F& f, int l, std::integer_sequence<int, K...>) {
    (f(std::integral_constant<int, K>(), l + K), ...);
}
// phi step 3: h_l = sum_u beta_u h_{l+u-s} for l = 0 .. n-1 (indices mod P).  Serial by nature;
// every lane runs it redundantly.  next[m mod S] collects the terms of
// h_m as they become known (oldest first), so a new value costs one multiply-add on the critical
// path.
template <int S>
__device__ __forceinline__ void recurrence(LocateSmem& sm, int n, int P, int lane) {
    double2 beta[S], next[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        beta[u] = sm.beta[u];
        next[u] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int w = 0; w < S; ++w) {   // the known values h_{-S} .. h_{-1}: h_{w-S} enters h_m with beta_{w-m}
        const double2 v = sm.h[P - S + w];
#pragma unroll
        for (int m = 0; m <= w; ++m) next[m] = cfma(beta[w - m], v, next[m]);
    }
    auto step = [&](auto slot, int l) {   // h_l, l = slot (mod S); every lane stores the same value
        constexpr int k = decltype(slot)::value;
        const double2 v = next[k];
        sm.h[l] = v;
#pragma unroll
        for (int u = S - 1; u >= 1; --u) next[(k + S - u) % S] = cfma(beta[u], v, next[(k + S - u) % S]);
        next[k] = cfma(beta[0], v, make_double2(0.0, 0.0));
    };
    int l = 0;
    for (; l + S <= n; l += S) unroll_slots(step, l, std::make_integer_sequence<int, S>());
    const int left = n - l;
    auto rest = [&](auto slot, int at) {
        if (decltype(slot)::value < left) step(slot, at);
    };
    unroll_slots(rest, l, std::make_integer_sequence<int, S>());
}
// The same for windows too long to unroll (s <= 16): lane i of each row of 16 holds what is known of h_{l+i}.  A new value
// is lane 0's; the others move down a lane and each takes its term.  (One lane that gathers s values out of LDS for
// each new one, 160 cycles a term: decodes of 7 000 floats with one liar, (256, 16) 401 us, 143 so, (200, 9) 211 and 93.)
__device__ __forceinline__ void recurrence_lanes(LocateSmem& sm, int n, int P, int s, int lane) {
    const int i = lane % 16;
    const double2 beta = i < s ? sm.beta[s - 1 - i] : make_double2(0.0, 0.0);
    const double2 known = sm.h[P - s + min(i, s - 1)];   // h_{-s} .. h_{-1}
    double2 next = make_double2(0.0, 0.0);
    auto enter = [&](double2 v) {
        next = cfma(beta, v, make_double2(dpp_move<kDppShl1>(next.x), dpp_move<kDppShl1>(next.y)));
    };
    for (int w = 0; w < s; ++w) enter(make_double2(lane_value(known.x, w), lane_value(known.y, w)));
    for (int l = 0; l < n; ++l) {
        const double2 v = make_double2(lane_value(next.x, 0), lane_value(next.y, 0));
        sm.h[l] = v;   // (every lane the same)
        enter(v);
    }
}

// What the locator finds, in registers: the set and the status are the same in every lane, a lane holds the coefficients of
// its nodes (the honest ones').
template <int CH>
struct Located {
    NodeSet<CH> flagged;
    int status;
    double2 b[CH];
    __device__ __forceinline__ bool clean() const { return flagged.count() == 0 && status == 0; }
};

// Orthonormal columns of length <= ROWS, at most kLocateMaxS (or 8 with ROWS = 16) of them: row r of
// column i in lane r of lane group i % kGroups, register i / kGroups.
template <int ROWS>
struct Basis {
    static constexpr int kGroups = kW / ROWS;
    static constexpr int kCols = ROWS / 2 / kGroups;   // a system of 2s rows has at most s columns
    double2 q[kCols];

    // Sum over the lane groups of a per-lane vector.
    static __device__ __forceinline__ double2 over_groups(double2 v) {
        double w[2] = {v.x, v.y}, o[2];
        auto step = [&](auto width) {   // both components in step, as in group_sums
#pragma unroll
            for (int i = 0; i < 2; ++i) o[i] = w[i];
#pragma unroll
            for (int i = 0; i < 2; ++i) lane_swap<decltype(width)::value>(w[i], o[i]);
#pragma unroll
            for (int i = 0; i < 2; ++i) w[i] += o[i];
        };
        if constexpr (ROWS <= 16) step(std::integral_constant<int, 16>());
        step(std::integral_constant<int, 32>());
        return make_double2(w[0], w[1]);
    }
    // Appends column c (every lane group holds the same `col`, 0 beyond its rows; len2: its squared
    // length): made orthogonal to columns 0 .. c-1 and normalised.  Classical Gram-Schmidt, with a
    // second pass unless the first took less than three quarters of the squared length away.
    // Returns the new column; inv: 1 / the length of the part orthogonal to the others.  R, if not null,
    // receives what it had of columns 0 .. c-1 (R[i * kLocateMaxS]).
    __device__ __forceinline__ double2 append(double2 col, double len2, int c, int lane, double& inv, double2* R = nullptr) {
        const int g = lane / ROWS;
        double n2 = len2;
        double2 had[kCols];
#pragma unroll
        for (int k = 0; k < kCols; ++k) had[k] = make_double2(0.0, 0.0);
        if (c > 0) {
#pragma unroll 1
            for (int pass = 0; pass < 2; ++pass) {
                double2 sum = make_double2(0.0, 0.0);
#pragma unroll
                for (int k = 0; k < kCols; ++k) {
                    if (k * kGroups < c) {
                        const double2 qi = k * kGroups + g < c ? q[k] : make_double2(0.0, 0.0);
                        const double2 prod = cmul(cconj(qi), col);
                        const double2 dot = group_sum_c<ROWS>(prod);
                        sum = cfma(dot, qi, sum);
                        had[k] = cadd(had[k], dot);
                    }
                }
                col = csub(col, over_groups(sum));
                n2 = group_sum<ROWS>(cnorm2(col));
                if (lane0_says(n2 >= 0.25 * len2)) break;
            }
            if (R != nullptr && lane % ROWS == 0) {
#pragma unroll
                for (int k = 0; k < kCols; ++k)
                    if (k * kGroups + g < c) R[(k * kGroups + g) * kLocateMaxS] = had[k];
            }
        }
        inv = rsqrt_pos(n2);
        col = cscale(col, inv);
#pragma unroll
        for (int k = 0; k < kCols; ++k)
            if (k == c / kGroups && g == c % kGroups) q[k] = col;
        return col;
    }
    // One more equation col^H x = want for the minimum-norm x that already meets c of them.
    __device__ __forceinline__ double2 meet(double2 col, double len2, double2 want, double2 x, int c, int lane) {
        const double2 prod = cmul(cconj(col), x);
        const double2 have = group_sum_c<ROWS>(prod);
        double inv;
        const double2 q = append(col, len2, c, lane, inv);
        return cfma(cscale(csub(want, have), inv), q, x);
    }
};

// beta: least squares on the s x s system h_{P-s-(i+1)+k} beta_k = h_{P-(i+1)}, i = 0 .. s-1, with
// singular values <= sqrt(zero2) dropped (one-sided Jacobi: A V has orthogonal columns).  GL lanes
// work on a pair of columns: row i of A in lane i, row i of V in lane GL/2 + i.
template <int GL>
__device__ __forceinline__ void solve_beta(LocateSmem& sm, int P, int s, double zero2, int lane) {
    constexpr int kGroups = kW / GL, kHalf = GL / 2;
    const int g = lane / GL, row = lane % kHalf;
    const bool isV = (lane % GL) >= kHalf;
    const bool live = row < s;
    double2* const M = (isV ? sm.V : sm.A) + row;
    for (int k = g; k < s; k += kGroups) {
        if (live) {
            M[k * kLocateMaxS] = isV ? make_double2(row == k ? 1.0 : 0.0, 0.0)
                                     : sm.h[P - s - (row + 1) + k];
        }
    }
    wave_sync();
    const int ne = s + (s & 1);   // columns, one of them a dummy if s is odd
    for (int sweep = 0; sweep < 60 && s > 1; ++sweep) {
        bool rotated = false;
        for (int r = 0; r < ne - 1; ++r) {   // round r of the tournament: ne / 2 pairs without a common column
            for (int i0 = 0; i0 < ne / 2; i0 += kGroups) {
                const int i = i0 + g;
                int p = r + i, q = r - i;
                if (p >= ne - 1) p -= ne - 1;
                if (q < 0) q += ne - 1;
                if (i == 0) q = ne - 1;
                if (p > q) {
                    const int t = p;
                    p = q;
                    q = t;
                }
                const bool pair = i < ne / 2 && q < s;
                double2 ap = make_double2(0.0, 0.0), aq = ap;   // this lane's row of the two columns (of A or of V)
                if (pair && live) {
                    ap = M[p * kLocateMaxS];
                    aq = M[q * kLocateMaxS];
                }
                const double2 gp = cmul(cconj(ap), aq);
                double sums[4] = {isV ? 0.0 : cnorm2(ap), isV ? 0.0 : cnorm2(aq), isV ? 0.0 : gp.x, isV ? 0.0 : gp.y};
                group_sums<GL>(sums);
                const double alpha = sums[0], bet = sums[1];
                const double2 gd = make_double2(sums[2], sums[3]);
                const double ag2 = cnorm2(gd);
                // columns that both end below the cutoff are dropped from the solution: no need
                // to make them orthogonal to each other
                const bool skip = !pair || ag2 == 0.0 || ag2 <= 1e-20 * (alpha * bet) || (alpha <= zero2 && bet <= zero2);
                if (!skip) {
                    // rotation that makes the two columns orthogonal: with zeta = (bet - alpha) / (2 |g|),
                    // t = sign(zeta) / (|zeta| + sqrt(1 + zeta^2)), c = 1 / sqrt(1 + t^2), sn = c t.  All of it to
                    // fp64: the last sweep then leaves columns orthogonal to rounding, not to the 1e-10 that ends
                    // the sweeps.
                    const double inv_ag = rsqrt_pos(ag2);
                    const double2 ph = make_double2(gd.x * inv_ag, -gd.y * inv_ag);
                    const double zeta = (bet - alpha) * (0.5 * inv_ag);
                    const double w2 = fma(zeta, zeta, 1.0);
                    const double t = (zeta >= 0.0 ? 1.0 : -1.0) * rcp_pos(fabs(zeta) + w2 * rsqrt_pos(w2));
                    const double c = rsqrt_pos(fma(t, t, 1.0)), sn = c * t;
                    const double2 aqr = cmul(aq, ph);
                    if (live) {
                        M[p * kLocateMaxS] = make_double2(fma(ap.x, c, -(aqr.x * sn)), fma(ap.y, c, -(aqr.y * sn)));
                        M[q * kLocateMaxS] = make_double2(fma(aqr.x, c, ap.x * sn), fma(aqr.y, c, ap.y * sn));
                    }
                }
                rotated |= __ballot(!skip) != 0ull;
                wave_sync();
            }
        }
        if (!rotated) break;
    }
    // beta_k = sum_i V[k][i] (a_i^H rhs) / |a_i|^2 over columns with |a_i| > zero
    const double2 rhs = (live && !isV) ? sm.h[P - (row + 1)] : make_double2(0.0, 0.0);
    for (int i0 = 0; i0 < s; i0 += kGroups) {
        const int i = i0 + g;
        double2 ai = make_double2(0.0, 0.0);
        if (i < s && live && !isV) ai = M[i * kLocateMaxS];
        const double s2 = group_sum<GL>(cnorm2(ai));
        const double2 dp = cmul(cconj(ai), rhs);
        const double2 dot = group_sum_c<GL>(dp);
        if (i < s && lane % GL == 0) sm.coef[i] = s2 > zero2 ? cscale(dot, 1.0 / s2) : make_double2(0.0, 0.0);
    }
    wave_sync();
    if (lane < s) {
        double2 bk = make_double2(0.0, 0.0);
        for (int i = 0; i < s; ++i) bk = cadd(bk, cmul(sm.coef[i], sm.V[i * kLocateMaxS + lane]));
        sm.beta[lane] = bk;
    }
    wave_sync();
}

// The same system for s <= 8 by a QR factorisation with column pivoting, where that settles which
// singular values are dropped: a column group of 8 lanes per column (row i in lane i), the pivot is
// the column with the longest remainder.  With remainder m at step k the k-th singular value is at
// least m / (85 sqrt 8) and those beyond are at most m sqrt(s - k), so a step counts as kept if
// m > 1024 zero and the rest as dropped if m sqrt(s - k) <= zero; in between (nearly dependent
// columns) it returns false and the Jacobi form decides.  The minimum-norm solution of the kept rows
// is the truncated one up to the size of what was dropped.
// Cycles against the tournament's: (P, s, liars) = (45, 7, 4) 8 100 and 46 700, (45, 3, 3) 5 800 and 14 100, (40, 8, 3) 6 100 and
// 51 800.
__device__ __forceinline__ bool solve_beta_qr(LocateSmem& sm, int P, int s, double zero2, int lane) {
    const int g = lane >> 3, row = lane & 7;
    double2 col = make_double2(0.0, 0.0), rhs = col;
    if (row < s) {
        if (g < s) col = sm.h[P - s - (row + 1) + g];
        rhs = sm.h[P - (row + 1)];
    }
    bool used = g >= s;
    int rank = 0;
    for (; rank < s; ++rank) {
        double n2 = group_sum<8>(cnorm2(col));
        if (used) n2 = -1.0;
        double m2 = fmax(n2, dpp_move<kDppRor8>(n2));
        {
            double o = m2;
            lane_swap<16>(m2, o);
            m2 = fmax(m2, o);
            o = m2;
            lane_swap<32>(m2, o);
            m2 = fmax(m2, o);
        }
        if (lane0_says(m2 * (double)(s - rank) <= zero2)) break;
        if (lane0_says(!(m2 > 1048576.0 * zero2))) return false;
        const unsigned long long at = __ballot(n2 == m2);   // groups with the longest remainder: take the first
        const int pivot = __builtin_ctzll(at) >> 3;
        const int from = pivot * 8 + row;
        double2 q = cscale(make_double2(__shfl(col.x, from), __shfl(col.y, from)), rsqrt_pos(m2));
        used |= g == pivot;
        const double2 pc = cmul(cconj(q), col), pr = cmul(cconj(q), rhs);
        const double2 rc = group_sum_c<8>(pc);
        const double2 rr = group_sum_c<8>(pr);
        col = csub(col, cmul(rc, q));
        rhs = csub(rhs, cmul(rr, q));
        if (row == 0) sm.A[rank * kLocateMaxS + g] = rc;   // row `rank` of R over the columns
        if (lane == 0) sm.coef[rank] = rr;
    }
    wave_sync();
    // x = beta: R x = Q^H rhs over the kept rows, minimum norm
    Basis<16> basis;
    double2 x = make_double2(0.0, 0.0);
    const int k = lane & 15;
    for (int i = 0; i < rank; ++i) {
        const double2 c = k < s ? cconj(sm.A[i * kLocateMaxS + k]) : make_double2(0.0, 0.0);
        x = basis.meet(c, group_sum<16>(cnorm2(c)), sm.coef[i], x, i, lane);
    }
    if (lane < s) sm.beta[lane] = x;
    wave_sync();
    return true;
}

// Shortest leading part of the ranking whose errors account for the syndromes: the residual of the
// syndromes loses its component along each new orthonormal column.  0 if there is none.
template <int ROWS>
__device__ __forceinline__ int fit_syndromes(LocateSmem& sm, int P, int s, int n, double isq, double zero2, int lane) {
    const int row = lane % ROWS;
    const bool live = row < 2 * s;
    const double len2 = 2 * s * isq * isq;   // every entry has modulus isq
    Basis<ROWS> basis;
    double2 res = live ? sm.hk[row] : make_double2(0.0, 0.0);
    for (int a = 0; a < s; ++a) {
        const int v = sm.order[a];
        const double2 col = live ? cscale(cconj(sm.root[mulmod(n + row, v, P)]), isq) : make_double2(0.0, 0.0);
        double inv;
        const double2 qa = basis.append(col, len2, a, lane, inv);
        // qa is orthogonal to the earlier columns, so is res: one projection removes the new component
        const double2 prod = cmul(cconj(qa), res);
        const double2 dot = group_sum_c<ROWS>(prod);
        res = csub(res, cmul(dot, qa));
        // largest |residual| against the zero threshold, on squares
        if (lane0_says(group_max<ROWS>(live ? cnorm2(res) : 0.0) <= zero2)) return a + 1;
    }
    return 0;
}

// The 2s free coefficients Bv of b (see host_math.cpp), Bv_m in the lanes m (mod ROWS): smallest Bv with
// sum_m conj w^{(n+m) v} Bv_m = -conj w^{(n-1) v} for the nodes v of a set of at most s, taken in ascending
// order, so that b depends on the set alone.  Adding a multiple of a new orthonormal column leaves the equations of the
// earlier nodes as they are.
// The same columns, conjugated, are the syndromes of single errors, so one orthonormal basis serves both this and the
// question whether the set accounts for the syndromes: res (not null) is what is left of them and loses its component
// along each column, which sm.coef keeps, with the columns' R in sm.V and 1 / R_ii in sm.inv.
template <int ROWS, int CH>
__device__ __forceinline__ double2 solve_set(LocateSmem& sm, NodeSet<CH> set, int P, int s, int n, double isq, int lane,
                                             double2* res) {
    only_here(P, s, lane);
    const int row = lane % ROWS;
    const bool live = row < 2 * s;
    const double len2 = 2 * s * isq * isq;   // every entry has modulus isq
    Basis<ROWS> basis;
    double2 Bv = make_double2(0.0, 0.0);
    // the roots of the next node are read while this one's column is made orthogonal
    int v = set.take_first();
    double2 col_root = sm.root[mulmod(live ? n + row : 0, max(v, 0), P)], want_root = sm.root[mulmod(n - 1, max(v, 0), P)];
    for (int i = 0; i < s && v >= 0; ++i) {
        const double2 col = live ? cscale(cconj(col_root), isq) : make_double2(0.0, 0.0);
        const double2 want = cscale(cconj(want_root), -isq);
        v = set.take_first();
        col_root = sm.root[mulmod(live ? n + row : 0, max(v, 0), P)];
        want_root = sm.root[mulmod(n - 1, max(v, 0), P)];
        double inv;
        const double2 q = basis.append(col, len2, i, lane, inv, res != nullptr ? &sm.V[i] : nullptr);
        const double2 met = cmul(col, Bv), part = res != nullptr ? cmul(cconj(q), *res) : make_double2(0.0, 0.0);
        double sums[4] = {met.x, met.y, part.x, part.y};
        group_sums<ROWS>(sums);
        Bv = cfma(cscale(csub(want, make_double2(sums[0], sums[1])), inv), cconj(q), Bv);
        if (res != nullptr) {   // q is orthogonal to the earlier columns, so is res: one projection removes the new component
            const double2 dot = make_double2(sums[2], sums[3]);
            *res = csub(*res, cmul(dot, q));
            if (lane == 0) {
                sm.coef[i] = dot;
                sm.inv[i] = inv;
            }
        }
    }
    return Bv;
}

// Smallest key over the wavefront.
__device__ __forceinline__ unsigned wave_min(unsigned v) {
    v = min(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, kDppXor1, 0xF, 0xF, true));
    v = min(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, kDppXor2, 0xF, 0xF, true));
    v = min(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, kDppHalfMirror, 0xF, 0xF, true));
    v = min(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, kDppRor8, 0xF, 0xF, true));
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min((unsigned)a[0], (unsigned)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return min((unsigned)b[0], (unsigned)b[1]);
}

// |z^A - sum_k c_k z^k|^2 where column A of the syndromes' system is sum_k c_k column k (R in sm.A, 1 / R_kk in sm.inv).
template <int A>
__device__ __forceinline__ void solve_relation(const LocateSmem& sm, double2 (&c)[7]) {
#pragma unroll
    for (int k = A - 1; k >= 0; --k) {
        double2 t = sm.A[k * kLocateMaxS + A];
#pragma unroll
        for (int i = k + 1; i < A; ++i) t = csub(t, cmul(sm.A[k * kLocateMaxS + i], c[i]));
        c[k] = cscale(t, sm.inv[k]);
    }
}
template <int A>
__device__ __forceinline__ double relation_at(const double2 (&c)[7], double2 z) {
    double2 acc = make_double2(1.0, 0.0);
#pragma unroll
    for (int k = A - 1; k >= 0; --k) acc = cfma(acc, z, cscale(c[k], -1.0));
    return cnorm2(acc);
}
// Whether the syndromes cannot do without any of the A nodes of a set that accounts for them: lane v < A holds row v of
// R^-1, whose length is 1 / the distance of column v from the others' span, and the coefficient of column v.
template <int A>
__device__ __forceinline__ bool all_needed(const LocateSmem& sm, double least2, int lane) {
    double2 z[A], x = make_double2(0.0, 0.0);
    double len2 = 0.0;
#pragma unroll
    for (int k = 0; k < A; ++k) {
        double2 t = make_double2(lane == k ? 1.0 : 0.0, 0.0);
#pragma unroll
        for (int i = 0; i < k; ++i) t = csub(t, cmul(z[i], sm.V[i * kLocateMaxS + k]));
        z[k] = cscale(t, sm.inv[k]);
        len2 += cnorm2(z[k]);
        x = cfma(z[k], sm.coef[k], x);
    }
    return __ballot(lane < A && !(cnorm2(x) > least2 * len2)) == 0ull;
}
template <class F>
__device__ __forceinline__ void with_count(int a, F&& f) {
    switch (a) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 5: f(std::integral_constant<int, 5>()); break;
        case 6: f(std::integral_constant<int, 6>()); break;
        default: f(std::integral_constant<int, 7>());
    }
}

// The usual case of s <= 7 without the recurrence and the transform: a errors make the syndromes a sum of a powers, so
// column a of the Hankel system is the first one that depends on those before it, and the errors sit at the a nodes where
// the relation between them, a polynomial of degree a, vanishes.  Columns 0 .. s (the last is the right-hand side), one per
// lane group of 8, are made orthogonal in turn; one whose remainder is below 64 times the zero threshold counts as
// dependent.  Nothing here has to be right: the set is taken only if it accounts for the syndromes and none of its nodes can
// be left out; else false, and the general form decides.  For lies well above the threshold no other set of up to s nodes
// accounts for them (any 2s columns are independent), so that set is the ranking's shortest leading part; near it both forms
// may settle on different sets that account for the syndromes.
template <int CH>
__device__ __forceinline__ bool locate_exact(LocateSmem& sm, const double2 (&root)[CH], int P, int s, int n, double isq,
                                             double zero2, int lane, NodeSet<CH>& found, double2& Bv) {
    only_here(P, s, lane);
    const int g = lane >> 3, row = lane & 7;
    double2 col = make_double2(0.0, 0.0);
    if (row < s && g <= s) col = sm.hk[s - 1 - row + g];
    int a = 0;
    for (; a < s; ++a) {
        const double n2 = group_sum<8>(cnorm2(col));
        const double len2 = lane_value(n2, a * 8);
        if (lane0_says(!(len2 > 4096.0 * zero2))) break;
        const double inv = rsqrt_pos(len2);
        const int from = a * 8 + row;
        const double2 q = cscale(make_double2(__shfl(col.x, from), __shfl(col.y, from)), inv);
        const double2 prod = cmul(cconj(q), col);
        const double2 dot = group_sum_c<8>(prod);
        col = csub(col, cmul(dot, q));
        if (row == 0) sm.A[a * kLocateMaxS + g] = dot;
        if (lane == 0) sm.inv[a] = inv;
    }
    if (a == 0) return false;
    wave_sync();
    unsigned key[CH];
    with_count(a, [&](auto count) {
        constexpr int A = decltype(count)::value;
        double2 c[7];
        solve_relation<A>(sm, c);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            // the upper word orders well enough
            const double at = relation_at<A>(c, cconj(root[k]));
            key[k] = k * kW + lane < P ? (unsigned)__double2hiint(at) : ~0u;
        }
    });
#pragma unroll
    for (int c = 0; c < CH; ++c) found.word[c] = 0;
    for (int i = 0; i < a; ++i) {   // the a smallest
        unsigned least = key[0];
#pragma unroll
        for (int c = 1; c < CH; ++c) least = min(least, key[c]);
        least = wave_min(least);
        bool taken = false;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const unsigned long long bal = __ballot(key[c] == least);
            if (!taken && bal != 0ull) {
                const int at = __builtin_ctzll(bal);
                found.word[c] |= 1ull << at;
                if (at == lane) key[c] = ~0u;
                taken = true;
            }
        }
    }
    if (found.count() != a) return false;   // (keys that are not numbers)
    double2 res = (lane & 15) < 2 * s ? sm.hk[lane & 15] : make_double2(0.0, 0.0);
    Bv = solve_set<16, CH>(sm, found, P, s, n, isq, lane, &res);
    if (__ballot(!(cnorm2(res) <= zero2)) != 0ull) return false;
    wave_sync();
    bool needed = false;
    with_count(a, [&](auto count) { needed = all_needed<decltype(count)::value>(sm, 8.0 * s * zero2, lane); });
    return needed;
}

// |sum_m h_m x^m|^2 over m = 0 .. P-1: Horner's rule in x^2 for the even and the odd powers.
__device__ __forceinline__ double horner(const double2* h, double2 x, int P) {
    const double2 x2 = cmul(x, x);
    double2 ev = make_double2(0.0, 0.0), od = ev;
    int k = (P + 1) / 2 - 1;
    if (P & 1) {   // the top even power has no odd partner
        ev = h[2 * k];
        --k;
    }
    for (; k >= 3; k -= 4) {
        double2 he[4], ho[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            he[i] = h[2 * (k - i)];
            ho[i] = h[2 * (k - i) + 1];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ev = cfma(x2, ev, he[i]);
            od = cfma(x2, od, ho[i]);
        }
    }
    for (; k >= 0; --k) {
        ev = cfma(x2, ev, h[2 * k]);
        od = cfma(x2, od, h[2 * k + 1]);
    }
    return cnorm2(cfma(x, od, ev));
}

// phi steps 2 to 4 in general: beta, the recurrence, the transform, and the shortest leading part of the ranking that
// accounts for the syndromes sm.hk.  Returns false if there is none (found: the s largest).
template <int CH>
__device__ __forceinline__ bool locate_general(LocateSmem& sm, const double2 (&root)[CH], int P, int s, double isq, double zero2,
                               int lane, NodeSet<CH>& found) {
    only_here(P, s, lane);
    const int n = P - 2 * s;
    for (int j = lane; j < P; j += kW) sm.h[j] = j < n ? make_double2(0.0, 0.0) : sm.hk[j - n];
    wave_sync();
    if (s > 8) solve_beta<32>(sm, P, s, zero2, lane);
    else if (!solve_beta_qr(sm, P, s, zero2, lane)) solve_beta<16>(sm, P, s, zero2, lane);
    // ---- recurrence h_l = sum_u beta_u h_{l+u-s}, l = 0 .. n-1
    switch (s) {
        case 1: recurrence<1>(sm, n, P, lane); break;
        case 2: recurrence<2>(sm, n, P, lane); break;
        case 3: recurrence<3>(sm, n, P, lane); break;
        case 4: recurrence<4>(sm, n, P, lane); break;
        case 5: recurrence<5>(sm, n, P, lane); break;
        case 6: recurrence<6>(sm, n, P, lane); break;
        case 7: recurrence<7>(sm, n, P, lane); break;
        case 8: recurrence<8>(sm, n, P, lane); break;
        default: recurrence_lanes(sm, n, P, s, lane);
    }
    wave_sync();
    // ---- t = C h, ranking by |t_j| (descending, ties to the lower index)
    double size[CH];   // P |t_j|^2 of this lane's nodes: the ranking needs no more
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        size[c] = -1.0;
        const int j = c * kW + lane;
        if (c * kW < P && j < P) {
            const double t2 = horner(sm.h, root[c], P);
            size[c] = t2 <= DBL_MAX ? t2 : DBL_MAX;   // overflow ranks first, in node order
        }
    }
    for (int rank = 0; rank < s; ++rank) {
        double best = size[0];
#pragma unroll
        for (int c = 1; c < CH; ++c) best = fmax(best, size[c]);
        best = group_max<kW>(best);
        int at = 0;
        bool taken = false;
#pragma unroll
        for (int c = 0; c < CH; ++c) {   // the first node, in order, with that size
            const unsigned long long bal = __ballot(size[c] == best);
            if (!taken && bal != 0ull) {
                at = c * kW + __builtin_ctzll(bal);
                if (at == c * kW + lane) size[c] = -1.0;
                taken = true;
            }
        }
        if (lane == 0) sm.order[rank] = at;
    }
    wave_sync();
    const int leading = s <= 8 ? fit_syndromes<16>(sm, P, s, n, isq, zero2, lane)
                               : fit_syndromes<32>(sm, P, s, n, isq, zero2, lane);
    const int take = leading != 0 ? leading : s;   // a failed decode flags the s largest |t_j|
#pragma unroll
    for (int c = 0; c < CH; ++c) found.word[c] = 0;
    for (int i = 0; i < take; ++i) found.add(__builtin_amdgcn_readfirstlane(sm.order[i]));
    return leading != 0;
}

// The square of rho = median |gamma_j|: the k-th smallest value is the largest one with at most k smaller ones, k = (P-1)/2 and
// P/2.  On squares, which order the same way (non-negative doubles order like their bits).
template <int CH>
__device__ __forceinline__ double median_size2(LocateSmem& sm, const double (&sq)[CH], int P, int lane) {
    double lo = 0.0, hi = 0.0;
    if constexpr (CH == 1) {
        int below = 0;
#pragma unroll
        for (int i = 0; i < kW; i += 8) {   // (lanes from P on hold infinity, below nothing)
            if (i < P) {
#pragma unroll
                for (int k = 0; k < 8; ++k) below += lane_value(sq[0], i + k) < sq[0] ? 1 : 0;
            }
        }
        const unsigned long long l = __ballot(below == (P - 1) / 2), h = __ballot(below == P / 2);
        if (l != 0ull && h != 0ull) {   // (equal ones leave gaps)
            lo = lane_value(sq[0], __builtin_ctzll(l));
            hi = lane_value(sq[0], __builtin_ctzll(h));
            if (P % 2 != 0) return lo;
            const double rho = 0.5 * (sqrt(lo) + sqrt(hi));
            return rho * rho;
        }
        if (lane < P && below <= (P - 1) / 2) lo = sq[0];
        if (lane < P && below <= P / 2) hi = sq[0];
    } else {
        const int P8 = (P + 7) / 8 * 8;   // padded to this length (at most kMaxNodes)
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (c * kW + lane < P8) sm.sq[c * kW + lane] = sq[c];
        wave_sync();
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (c * kW >= P) break;
            const double mine = sq[c];
            const double2* m2 = reinterpret_cast<const double2*>(sm.sq);
            int n0 = 0, n1 = 0;
            for (int i = 0; i < P8 / 2; i += 4) {
                const double2 a = m2[i], b = m2[i + 1], d = m2[i + 2], e = m2[i + 3];
                n0 += (a.x < mine) + (b.x < mine) + (d.x < mine) + (e.x < mine);
                n1 += (a.y < mine) + (b.y < mine) + (d.y < mine) + (e.y < mine);
            }
            const bool live = c * kW + lane < P;
            if (live && n0 + n1 <= (P - 1) / 2) lo = fmax(lo, mine);
            if (live && n0 + n1 <= P / 2) hi = fmax(hi, mine);
        }
    }
    const double rho = 0.5 * (sqrt(group_max<kW>(lo)) + sqrt(group_max<kW>(hi)));
    return rho * rho;
}

// Run by one wavefront (lane = 0 .. 63, all active) with sm.gam[0..P) and sm.root[0..P) filled; P <= 64 CH, isq =
// 1 / sqrt(P).
template <int CH>
__device__ __forceinline__ Located<CH> locate_wave(LocateSmem& sm, int P, int s, double tau, double isq,
                                                  const double2* __restrict__ b0, int lane) {
    const int n = P - 2 * s;  // rows of C_L
    Located<CH> out;
    NodeSet<CH>& flagged = out.flagged;
    int status = 0;

    // A lane's nodes: j = lane, lane + 64, ...
    double2 gam[CH], root[CH], b_clean[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int j = c * kW + lane;
        gam[c] = j < P ? sm.gam[j] : make_double2(0.0, 0.0);
        root[c] = j < P ? sm.root[j] : make_double2(0.0, 0.0);
        b_clean[c] = b0[min(j, P - 1)];   // (under way while the rest runs)
    }
    // A message with NaN or Inf entries is no vector of R^d: its node is flagged outright and
    // its projection taken as 0, which leaves an ordinary error at a known node.
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const bool bad = !(isfinite(gam[c].x) && isfinite(gam[c].y));
        if (bad) gam[c] = make_double2(0.0, 0.0);
        flagged.word[c] = __ballot(bad);
    }
    const int broken = flagged.count();

    if (broken > s) status = 2;  // DRACO_LOCATE_FAILED: more broken messages than tolerated
    // Passes of phi.  A projection more than kEnormous * rho in size is "enormous": its fp64
    // rounding can reach the zero threshold or swallow a smaller lie whole (an adversary may send
    // 1e30).  After a pass the located nodes whose projection is enormous and large enough for its
    // rounding to pass for a syndrome (kLocatedEnormousOverTau) -- or, if it found no set, the top
    // layer of the enormous nodes (within a factor kEnormous of the largest) -- are set aside like
    // broken ones and phi runs again, provided the flagged nodes stay within s; the
    // first pass that sets nothing aside is the last.  Every other pass flags at least one more node, so there are at
    // most s + 1.  Every branch below is taken by all 64 lanes together.
    int aside = broken;  // nodes flagged outright so far
    double2 Bv = make_double2(0.0, 0.0);
    bool have_Bv = false;   // Bv belongs to the flagged set
    for (int pass = 0; pass <= s && s > 0 && broken <= s; ++pass) {
        double sq[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) sq[c] = c * kW + lane < P ? cnorm2(gam[c]) : __builtin_inf();
        const double rho2 = median_size2<CH>(sm, sq, P, lane);

        // syndromes h_m = (1/sqrt P) sum_j gamma_j w^{-m j}, m = n .. P-1; with m = P - e, e = 1 .. 2s, a lane
        // needs the powers w^{e j} of its nodes, and eight sums over the wavefront are made together
        {
            int at[CH], step[CH];   // (lanes from P on: 0 times the root 1)
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                at[c] = 0;
                step[c] = c * kW + lane < P ? c * kW + lane : 0;
            }
            for (int e0 = 0; e0 < 2 * s; e0 += 8) {
                double v[16];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    double2 acc = make_double2(0.0, 0.0);
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        at[c] = addmod(at[c], step[c], P);
                        const double2 term = cmul(gam[c], sm.root[at[c]]);
                        acc = CH == 1 ? term : cadd(acc, term);
                    }
                    v[2 * i] = acc.x;
                    v[2 * i + 1] = acc.y;
                }
                const double t = reduce_over_wave<16>(v);   // of value lane / 4
                const int e = e0 + lane / 8 + 1;
                if (lane % 4 == 0 && e <= 2 * s) reinterpret_cast<double*>(&sm.hk[2 * s - e])[(lane / 4) % 2] = t * isq;
            }
        }
        wave_sync();
        const double zero2 = tau * tau * rho2;   // (the zero threshold tau * rho, squared)
        const bool any = __ballot(lane < 2 * s && cnorm2(sm.hk[min(lane, 2 * s - 1)]) > zero2) != 0ull;

        NodeSet<CH> found;   // the leading part of the ranking that accounts for the syndromes
#pragma unroll
        for (int c = 0; c < CH; ++c) found.word[c] = 0;
        bool located = true;
        have_Bv = false;
        if (any) {
            if (s <= 7) have_Bv = locate_exact<CH>(sm, root, P, s, n, isq, zero2, lane, found, Bv);
            if (!have_Bv) {
                located = locate_general<CH>(sm, root, P, s, isq, zero2, lane, found);
            }
        }
        bool last = pass == s;   // (never reached with something left to set aside: aside <= s)
        if (!last) {
            const double least = fmax(kEnormous, kLocatedEnormousOverTau * tau);
            const double limit2 = kEnormous * kEnormous * rho2, located2 = least * least * rho2;
            double top = 0.0;   // the largest enormous projection not flagged yet, squared
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if (c * kW + lane < P && !flagged.has(c, lane) && sq[c] > limit2) top = fmax(top, sq[c]);
            }
            if (__ballot(top > 0.0) == 0ull) {
                last = true;   // nothing enormous: this pass stands
            } else {
                top = group_max<kW>(top);
                NodeSet<CH> go;   // enormous, not flagged yet; located, or else in the top layer
                int huge = 0;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const bool open = c * kW + lane < P && !flagged.has(c, lane) && sq[c] > limit2;
                    go.word[c] = __ballot(open && (located ? found.has(c, lane) && sq[c] > located2
                                                           : sq[c] * (kEnormous * kEnormous) > top));
                    huge += __popcll(go.word[c]);
                }
                if (huge == 0 || aside + huge > s) {
                    last = true;   // nothing to set aside, or too many: this pass stands
                } else {
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        if (go.has(c, lane)) gam[c] = make_double2(0.0, 0.0);
                        flagged.word[c] |= go.word[c];
                    }
                    aside += huge;
                }
            }
        }
        if (last) {
            if (!located) status = 2;
            if (aside != 0) have_Bv = false;
#pragma unroll
            for (int c = 0; c < CH; ++c) flagged.word[c] |= found.word[c];
            break;
        }
    }

    // ---- b: minimum-norm solution of C_L[:, U] b_U = e_last (see host_math.cpp).  More than s flagged nodes only
    // happen in a failed decode; its equations have room for s, so it takes the first s
    const int nv = flagged.count();
    if (nv > s) status = 2;
    if (nv > 0 && !have_Bv) {   // (no node flagged: b0; s = 0 with a broken node: no free coefficients)
        Bv = s <= 8 ? solve_set<16, CH>(sm, flagged, P, s, n, isq, lane, nullptr)
                    : solve_set<32, CH>(sm, flagged, P, s, n, isq, lane, nullptr);
    }
    // b_j = (1/sqrt P) (conj w^{(n-1) j} + sum_m conj w^{(n+m) j} Bv_m) on honest nodes
#pragma unroll
    for (int c = 0; c < CH; ++c) out.b[c] = nv == 0 ? b_clean[c] : make_double2(0.0, 0.0);   // (the table the speculative pass used)
    if (nv > 0) {
        for (int m = 2 * s - 1; m >= 0; --m) {
            const double2 free_m = make_double2(lane_value(Bv.x, m), lane_value(Bv.y, m));
#pragma unroll
            for (int c = 0; c < CH; ++c) out.b[c] = cfma(cconj(root[c]), out.b[c], free_m);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int j = c * kW + lane;
            out.b[c] = cfma(cconj(root[c]), out.b[c], make_double2(1.0, 0.0));
            if (j < P) out.b[c] = cscale(cmul(cconj(sm.root[mulmod(n - 1, j, P)]), out.b[c]), isq);
        }
    }
    out.status = status;
    return out;
}

}  // namespace
}  // namespace draco
