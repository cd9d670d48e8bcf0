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
//   * a lane owns node j (j = lane, lane+64, ...) in the O(P) and O(P^2) loops, and those read
//     their LDS operands several iterations at a time;
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
// Measured, one call in cycles at 2.3 GHz (before: gathers, serial Jacobi over all pairs, LDS-held
// columns): (P, s, liars) = (45, 3, 0) 16 000 -> 10 500, (45, 3, 3) 60 000 -> 34 000,
// (45, 5, 5) 115 000 -> 50 000, (45, 7, 4) 198 000 -> 49 000; running it twice in a row shows that
// cold instructions are about a tenth of that.
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
// Sum over aligned groups of n lanes, n a power of two <= 32 known only at run time
// (the same n in every lane).
__device__ __forceinline__ double group_sum_n(double v, int n) {
    if (n > 1) v += dpp_move<kDppXor1>(v);
    if (n > 2) v += dpp_move<kDppXor2>(v);
    if (n > 4) v += dpp_move<kDppHalfMirror>(v);
    if (n > 8) v += dpp_move<kDppRor8>(v);
    if (n > 16) v = swap_add<16>(v, v);
    return v;
}
__device__ __forceinline__ bool lane0_says(bool b) { return __builtin_amdgcn_readfirstlane(b ? 1 : 0) != 0; }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double cnorm2(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
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
    alignas(16) double mag[kMaxNodes];         // padded to a multiple of 8
    double2 A[kLocateMaxS * kLocateMaxS];      // column-major s x s
    double2 V[kLocateMaxS * kLocateMaxS];
    double2 hk[2 * kLocateMaxS];
    double2 beta[kLocateMaxS];
    double2 coef[kLocateMaxS];
    double2 Bv[2 * kLocateMaxS];
    int order[kLocateMaxS];
    int vlist[kLocateMaxS];
    unsigned char mask[kMaxNodes];
};

// Where a located set goes.
struct LocateOut {
    uint64_t* mask;      // ceil(P/64) words
    int32_t* status;
    double2* b;          // honest nodes' coefficients, one behind the other
    int32_t* idx;        // and their indices
    int32_t* nu;         // how many
    double2* dense;      // the coefficients by node (flagged ones untouched), or nullptr
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
// The same out of LDS, for windows too long to unroll.
__device__ __forceinline__ void recurrence_lds(LocateSmem& sm, int n, int P, int s, int lane) {
    if (lane == 0) {
        for (int l = 0; l < n; ++l) {
            double2 acc = make_double2(0.0, 0.0);
            int e = l - s;
            if (e < 0) e += P;
            for (int u = 0; u < s; ++u) {
                acc = cadd(acc, cmul(sm.beta[u], sm.h[e]));
                e = addmod(e, 1, P);
            }
            sm.h[l] = acc;
        }
    }
}

// Orthonormal columns of length <= ROWS, at most kLocateMaxS (or 8 with ROWS = 16) of them: row r of
// column i in lane r of lane group i % kGroups, register i / kGroups.
template <int ROWS>
struct Basis {
    static constexpr int kGroups = kW / ROWS;
    static constexpr int kCols = ROWS / 2 / kGroups;   // a system of 2s rows has at most s columns
    double2 q[kCols];

    // Sum over the lane groups of a per-lane vector.
    static __device__ __forceinline__ double2 over_groups(double2 v) {
        if constexpr (ROWS <= 16) v = make_double2(swap_add<16>(v.x, v.x), swap_add<16>(v.y, v.y));
        return make_double2(swap_add<32>(v.x, v.x), swap_add<32>(v.y, v.y));
    }
    // Appends column c (every lane group holds the same `col`, 0 beyond its rows; len2: its squared
    // length): made orthogonal to columns 0 .. c-1 and normalised.  Classical Gram-Schmidt, with a
    // second pass unless the first took less than three quarters of the squared length away.
    // Returns the new column; inv: 1 / the length of the part orthogonal to the others.
    __device__ __forceinline__ double2 append(double2 col, double len2, int c, int lane, double& inv) {
        const int g = lane / ROWS;
        double n2 = len2;
        if (c > 0) {
#pragma unroll 1
            for (int pass = 0; pass < 2; ++pass) {
                double2 sum = make_double2(0.0, 0.0);
#pragma unroll
                for (int k = 0; k < kCols; ++k) {
                    if (k * kGroups < c) {
                        const double2 qi = k * kGroups + g < c ? q[k] : make_double2(0.0, 0.0);
                        const double2 prod = cmul(cconj(qi), col);
                        const double2 dot = make_double2(group_sum<ROWS>(prod.x), group_sum<ROWS>(prod.y));
                        sum = cfma(dot, qi, sum);
                    }
                }
                col = csub(col, over_groups(sum));
                n2 = group_sum<ROWS>(cnorm2(col));
                if (lane0_says(n2 >= 0.25 * len2)) break;
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
        const double2 have = make_double2(group_sum<ROWS>(prod.x), group_sum<ROWS>(prod.y));
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
                const double alpha = group_sum<GL>(isV ? 0.0 : cnorm2(ap));
                const double bet = group_sum<GL>(isV ? 0.0 : cnorm2(aq));
                const double2 gd = make_double2(group_sum<GL>(isV ? 0.0 : gp.x), group_sum<GL>(isV ? 0.0 : gp.y));
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
                        M[p * kLocateMaxS] = csub(cscale(ap, c), cscale(aqr, sn));
                        M[q * kLocateMaxS] = cadd(cscale(ap, sn), cscale(aqr, c));
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
        const double2 dot = make_double2(group_sum<GL>(dp.x), group_sum<GL>(dp.y));
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
// (P, s, liars) = (45, 7, 4): 10 000 cycles against 55 000 for the tournament and 141 000 for Jacobi
// sweeps one pair at a time; (45, 3, 3): 7 000 against 18 000 and 17 000.
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
        const double2 rc = make_double2(group_sum<8>(pc.x), group_sum<8>(pc.y));
        const double2 rr = make_double2(group_sum<8>(pr.x), group_sum<8>(pr.y));
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
        const double2 dot = make_double2(group_sum<ROWS>(prod.x), group_sum<ROWS>(prod.y));
        res = csub(res, cmul(dot, qa));
        // largest |residual| against the zero threshold, on squares
        if (lane0_says(group_max<ROWS>(live ? cnorm2(res) : 0.0) <= zero2)) return a + 1;
    }
    return 0;
}

// The 2s free coefficients Bv of b (see host_math.cpp): smallest Bv with
// sum_m conj w^{(n+m) v} Bv_m = -conj w^{(n-1) v} for the flagged nodes v = vlist[0 .. a-1], taken in
// ascending order, so that b depends on the set of flagged nodes alone.  Adding a multiple of a new
// orthonormal column leaves the equations of the earlier nodes as they are.
template <int ROWS>
__device__ __forceinline__ void solve_bv(LocateSmem& sm, int P, int s, int n, double isq, int a, int lane) {
    const int row = lane % ROWS;
    const bool live = row < 2 * s;
    const double len2 = 2 * s * isq * isq;   // every entry has modulus isq
    Basis<ROWS> basis;
    double2 Bv = make_double2(0.0, 0.0);
    for (int i = 0; i < a; ++i) {
        const int v = sm.vlist[i];
        const double2 col = live ? cscale(sm.root[mulmod(n + row, v, P)], isq) : make_double2(0.0, 0.0);
        const double2 want = cscale(cconj(sm.root[mulmod(n - 1, v, P)]), -isq);
        Bv = basis.meet(col, len2, want, Bv, i, lane);
    }
    if (lane < 2 * s) sm.Bv[lane] = Bv;
    wave_sync();
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

// Run by one wavefront (lane = 0 .. 63, all active) with sm.gam[0..P) and sm.root[0..P) filled.
// Returns whether the decode was clean: nobody flagged, status OK.
__device__ __forceinline__ bool locate_wave(LocateSmem& sm, int P, int s, double tau, const double2* __restrict__ b0,
                                           const LocateOut& out, int lane) {
    const int n = P - 2 * s;  // rows of C_L
    const double isq = 1.0 / sqrt((double)P);
    int status = 0;

    // A message with NaN or Inf entries is no vector of R^d: its node is flagged outright and
    // its projection taken as 0, which leaves an ordinary error at a known node.
    int broken = 0;
    for (int c = 0; c < P; c += kW) {
        const int j = c + lane;
        bool bad = false;
        if (j < P) {
            const double2 g = sm.gam[j];
            bad = !(isfinite(g.x) && isfinite(g.y));
            if (bad) sm.gam[j] = make_double2(0.0, 0.0);
            sm.mask[j] = bad ? 1 : 0;
        }
        broken += __popcll(__ballot(bad));
    }
    wave_sync();

    if (broken > s) status = 2;  // DRACO_LOCATE_FAILED: more broken messages than tolerated
    // Passes of phi.  A projection more than kEnormous * rho in size is "enormous": its fp64
    // rounding can reach the zero threshold or swallow a smaller lie whole (an adversary may send
    // 1e30).  After a pass the located nodes whose projection is enormous and large enough for its
    // rounding to pass for a syndrome (kLocatedEnormousOverTau) -- or, if it found no set, the top
    // layer of the enormous nodes (within a factor kEnormous of the largest) -- are set aside like
    // broken ones and phi runs again, provided the flagged nodes stay within s; the
    // first pass that sets nothing aside is the last.  Every other pass flags at least one more node, so there are at
    // most s + 1.  Every branch below is taken by all 64 lanes together.
    const int P8 = (P + 7) / 8 * 8;   // mag is padded to this length (at most kMaxNodes)
    int aside = broken;  // nodes flagged outright so far
    for (int pass = 0; pass <= s && s > 0 && broken <= s; ++pass) {
        for (int j = lane; j < P8; j += kW)
            sm.mag[j] = j < P ? sqrt(cnorm2(sm.gam[j])) : __builtin_inf();
        for (int j = lane; j < P; j += kW) sm.h[j] = make_double2(0.0, 0.0);
        wave_sync();
        // rho = median |gamma_j|: the k-th smallest value is the largest one with at most k smaller
        // ones, k = (P-1)/2 and P/2
        double lo = 0.0, hi = 0.0;
        for (int j = lane; j < P; j += kW) {
            const double mj = sm.mag[j];
            const double2* m2 = reinterpret_cast<const double2*>(sm.mag);
            int n0 = 0, n1 = 0;
            for (int i = 0; i < P8 / 2; i += 4) {
                const double2 a = m2[i], b = m2[i + 1], c = m2[i + 2], e = m2[i + 3];
                n0 += (a.x < mj) + (b.x < mj) + (c.x < mj) + (e.x < mj);
                n1 += (a.y < mj) + (b.y < mj) + (c.y < mj) + (e.y < mj);
            }
            if (n0 + n1 <= (P - 1) / 2) lo = fmax(lo, mj);
            if (n0 + n1 <= P / 2) hi = fmax(hi, mj);
        }
        const double rho = 0.5 * (group_max<kW>(lo) + group_max<kW>(hi));

        // syndromes h_m = (1/sqrt P) sum_j gamma_j w^{-m j}, m = n .. P-1: `parts` lanes share a
        // syndrome, each summing the nodes j = part, part + parts, ...
        int parts = 1;
        while (2 * parts * 2 * s <= kW && parts < 32) parts *= 2;
        double mymax = 0.0;
        {
            const int mp = lane / parts, part = lane % parts;
            const bool on = mp < 2 * s;
            const int m = n + (on ? mp : 0);
            double2 acc = make_double2(0.0, 0.0);
            int e = mulmod(m, part < P ? part : 0, P);
            const int step = mulmod(m, parts < P ? parts : 0, P);
            for (int j = part; j < P; j += 4 * parts) {
                double2 g[4], w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = j + i * parts;
                    g[i] = k < P ? sm.gam[k] : make_double2(0.0, 0.0);
                    w[i] = sm.root[e];
                    e = addmod(e, step, P);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = cadd(acc, cmul(g[i], cconj(w[i])));
            }
            acc = make_double2(group_sum_n(acc.x, parts), group_sum_n(acc.y, parts));
            acc = cscale(acc, isq);
            if (on && part == 0) {
                sm.hk[mp] = acc;
                sm.h[m] = acc;
            }
            if (on) mymax = cnorm2(acc);
        }
        wave_sync();
        const double hmax2 = group_max<kW>(mymax);
        const double zero = tau * rho;
        const double zero2 = zero * zero;

        int found = 0;      // length of the leading part of the ranking that accounts for the syndromes
        bool located = true;
        if (hmax2 > zero2) {
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
                default: recurrence_lds(sm, n, P, s, lane);
            }
            wave_sync();
            // ---- t = C h, ranking by |t_j| (descending, ties to the lower index)
            double size[kMaxNodes / kW];   // P |t_j|^2 of this lane's nodes: the ranking needs no more
#pragma unroll
            for (int c = 0; c < kMaxNodes / kW; ++c) {
                size[c] = -1.0;
                const int j = c * kW + lane;
                if (c * kW < P && j < P) {
                    const double2 x = sm.root[j];
                    const double t2 = horner(sm.h, x, P);
                    size[c] = t2 <= DBL_MAX ? t2 : DBL_MAX;   // overflow ranks first, in node order
                }
            }
            for (int rank = 0; rank < s; ++rank) {
                double best = size[0];
#pragma unroll
                for (int c = 1; c < kMaxNodes / kW; ++c) best = fmax(best, size[c]);
                best = group_max<kW>(best);
                int at = 0;
                bool taken = false;
#pragma unroll
                for (int c = 0; c < kMaxNodes / kW; ++c) {   // the first node, in order, with that size
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
            found = s <= 8 ? fit_syndromes<16>(sm, P, s, n, isq, zero2, lane)
                           : fit_syndromes<32>(sm, P, s, n, isq, zero2, lane);
            located = found != 0;
        }
        bool last = pass == s;   // (never reached with something left to set aside: aside <= s)
        if (!last) {
            const double limit = kEnormous * rho;
            const double located_limit = fmax(limit, kLocatedEnormousOverTau * tau * rho);
            double top = 0.0;   // the largest enormous projection not flagged yet
            for (int j = lane; j < P; j += kW) {
                const double size = sqrt(cnorm2(sm.gam[j]));
                if (sm.mask[j] == 0 && size > limit) top = fmax(top, size);
            }
            top = group_max<kW>(top);
            if (top == 0.0) {
                last = true;   // nothing enormous: this pass stands
            } else {
                auto set_aside = [&](int j) {   // enormous, not flagged yet; located, or else in the top layer
                    const double size = sqrt(cnorm2(sm.gam[j]));
                    if (sm.mask[j] != 0 || !(size > limit)) return false;
                    if (!located) return size * kEnormous > top;
                    if (!(size > located_limit)) return false;
                    for (int i = 0; i < found; ++i)
                        if (sm.order[i] == j) return true;
                    return false;
                };
                bool go[kMaxNodes / kW];
                int huge = 0;
#pragma unroll
                for (int k = 0; k < kMaxNodes / kW; ++k) {
                    const int j = k * kW + lane;
                    go[k] = j < P && set_aside(j);
                    huge += __popcll(__ballot(go[k]));
                }
                if (huge == 0 || aside + huge > s) {
                    last = true;   // nothing to set aside, or too many: this pass stands
                } else {
#pragma unroll
                    for (int k = 0; k < kMaxNodes / kW; ++k) {
                        if (go[k]) {
                            sm.gam[k * kW + lane] = make_double2(0.0, 0.0);
                            sm.mask[k * kW + lane] = 1;
                        }
                    }
                    aside += huge;
                    wave_sync();
                }
            }
        }
        if (last) {
            const int take = located ? found : s;   // a failed decode flags the s largest |t_j|
            if (!located) status = 2;
            if (hmax2 > zero2 && lane < take) sm.mask[sm.order[lane]] = 1;
            wave_sync();
            break;
        }
    }

    // ---- b: minimum-norm solution of C_L[:, U] b_U = e_last (see host_math.cpp)
    // flagged nodes in ascending order.  More than s of them only happens in a failed decode; the
    // equations below have room for s, so it takes the first s
    int nv = 0;
    for (int c = 0; c < P; c += kW) {
        const int j = c + lane;
        const bool flagged = j < P && sm.mask[j] != 0;
        const unsigned long long bal = __ballot(flagged);
        const int pos = nv + __popcll(bal & ((1ull << lane) - 1ull));
        if (flagged && pos < s) sm.vlist[pos] = j;
        if (lane == 0) out.mask[c / kW] = bal;
        nv += __popcll(bal);
    }
    wave_sync();
    if (nv > s) status = 2;
    const int a = nv <= s ? nv : s;
    if (nv > 0) {   // (no node flagged: b0; s = 0 with a broken node: a = 0, no free coefficients)
        if (s <= 8) solve_bv<16>(sm, P, s, n, isq, a, lane);
        else solve_bv<32>(sm, P, s, n, isq, a, lane);
    }
    // b_j = (1/sqrt P) (conj w^{(n-1) j} + sum_m conj w^{(n+m) j} Bv_m) on honest nodes, written
    // one behind the other in ascending node order
    int nu = 0;
    for (int c = 0; c < P; c += kW) {
        const int j = c + lane;
        const bool honest = j < P && sm.mask[j] == 0;
        double2 acc = make_double2(0.0, 0.0);
        if (honest) {
            if (nv == 0) {
                acc = b0[j];  // the table the speculative pass used: identical results either way
            } else {
                const double2 y = cconj(sm.root[j]);
                for (int m = 2 * s - 1; m >= 0; --m) acc = cfma(y, acc, sm.Bv[m]);
                acc = cfma(y, acc, make_double2(1.0, 0.0));
                acc = cscale(cmul(cconj(sm.root[mulmod(n - 1, j, P)]), acc), isq);
            }
        }
        const unsigned long long bal = __ballot(honest);
        if (honest) {
            const int pos = nu + __popcll(bal & ((1ull << lane) - 1ull));
            out.idx[pos] = j;
            out.b[pos] = acc;
            if (out.dense != nullptr) out.dense[j] = acc;
        }
        nu += __popcll(bal);
    }
    if (lane == 0) {
        *out.nu = nu;
        *out.status = status;
    }
    return nu == P && status == 0;
}

}  // namespace
}  // namespace draco
