// Repetition code (Sec. 3, "Fractional Repetition Code"): encoder E^Rep and the
// majority-vote decoder D^Rep with the streaming vote of Algorithm 2.
#include "device_util.hpp"

#include <mutex>

namespace draco {

// ===========================================================================
// Repetition code
// ===========================================================================

// E^Rep for all nodes: one pass reads each gradient once, forms each group's
// sum in ascending gradient order and stores it r times.  A workgroup handles
// one column tile (blockIdx.x) of GU consecutive groups (blockIdx.y) and ends:
// with tiles varying fastest across the grid, the whole chip streams the same
// few rows at a time, which HBM serves measurably faster (6.3-6.6 TB/s for a
// copy of this shape) than workgroups that each walk down all P rows (5.9).
// The GU groups are loaded before the first is summed: GU*R 16-byte loads in
// flight per lane.
template <int R, int GU, bool FULL>
__device__ __forceinline__ void encode_rep_body(const float* __restrict__ G, int64_t ldg, float* __restrict__ Z,
                                                int64_t ldm, int groups, int64_t d, int64_t c0) {
    if (!FULL && c0 >= d) return;
    const int n = FULL ? 4 : clamp4(d - c0);
    {
        const int g0 = (int)blockIdx.y * GU;
        float4 x[GU][R];
#pragma unroll
        for (int a = 0; a < GU; ++a) {
            if (g0 + a < groups) {
                const float* src = G + (int64_t)(g0 + a) * R * ldg + c0;
#pragma unroll
                for (int i = 0; i < R; ++i) x[a][i] = ldx<FULL>(src + (int64_t)i * ldg, n);
            }
        }
#pragma unroll
        for (int a = 0; a < GU; ++a) {
            if (g0 + a < groups) {
                float4 acc = x[a][0];
#pragma unroll
                for (int i = 1; i < R; ++i) {
                    acc.x += x[a][i].x;
                    acc.y += x[a][i].y;
                    acc.z += x[a][i].z;
                    acc.w += x[a][i].w;
                }
                float* dst = Z + (int64_t)(g0 + a) * R * ldm + c0;
#pragma unroll
                for (int i = 0; i < R; ++i) stx<FULL>(dst + (int64_t)i * ldm, acc, n);
            }
        }
    }
}

// SPREAD: the spread footprint, where message rows are on the line grid; 4 KiB contiguously where they are not
// (device_util.hpp).  Encoder in us, spread / contiguous / contiguous with neighbours on one die: (18, 4, 3.7 M + 1)
// 107 / 98 / 150, (45, 7, 3.7 M + 1) 277 / 252 / 351, (45, 2, 3.7 M + 1) 265 / 240 / 284, (45, 2, 11.2 M + 1) 808 / 724 /
// 756, (45, 2, 1.47 M + 1) 106 / 96 / 99, (45, 2, B = 180, 1 663 371) 280 / 263 / 264; on the grid (45, 2, 11.2 M)
// 622 / 659 / 701.
template <int R, int GU, bool SPREAD>
__global__ __launch_bounds__(kBlock) void encode_rep_kernel(const float* __restrict__ G, int64_t ldg,
                                                            float* __restrict__ Z, int64_t ldm,
                                                            int groups, int64_t d) {
    const int64_t c0 = lane_column<SPREAD>(d);
    if (block_is_full<SPREAD>(d, d)) encode_rep_body<R, GU, true>(G, ldg, Z, ldm, groups, d, c0);
    else encode_rep_body<R, GU, false>(G, ldg, Z, ldm, groups, d, c0);
}

// Any number of rows per group (also the one-node form with groups = 1, copies = 1, and
// the B > P form where a group sums its r*(B/P) consecutive per-sample rows): rows are
// added in ascending order, UN at a time.  The first HEAD of them, 1 to UN, make the others whole rounds: their number is known
// where the loads are issued, since a load under a condition makes the compiler wait for everything before each sum (one
// node's message of 15 rows, 168 113 floats: 6.5 us so, 4.0 now; (30, 1, B = 60, 909 408) 59.4 and 51.8).
template <bool FULL, int UN, int HEAD>
__device__ __forceinline__ float4 sum_rows(const float* __restrict__ src, int64_t ldg, int rows, int n) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), head[HEAD], x[UN];
    auto fetch = [&](auto& row) {
#pragma unroll
        for (auto& v : row) {
            v = ldx<FULL>(src, n);
            src += ldg;
        }
    };
    auto add = [&](const float4& v) {
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
    };
    // a round is added and the next one fetched, row by row
    auto rounds = [&](auto& row, int left) {
        for (; left > UN; left -= UN) {
            // Four rows are waited for together, before the first sum ((15, 2, B = 240, 180 907) 37.1 us, 38.9 one by one; with the
            // wait behind the first sum 37.6, and (45, 1, B = 180, 400 001) 65.6 instead of 63.3).
            if constexpr (UN == 4)
                asm volatile("" : "+v"(row[0].x), "+v"(row[0].y), "+v"(row[0].z), "+v"(row[0].w), "+v"(row[1].x), "+v"(row[1].y),
                             "+v"(row[1].z), "+v"(row[1].w), "+v"(row[2].x), "+v"(row[2].y), "+v"(row[2].z), "+v"(row[2].w),
                             "+v"(row[3].x), "+v"(row[3].y), "+v"(row[3].z), "+v"(row[3].w));
#pragma unroll
            for (auto& v : row) {
                add(v);
                v = ldx<FULL>(src, n);
                src += ldg;
            }
        }
#pragma unroll
        for (auto& v : row) add(v);
    };
    fetch(head);
    if constexpr (UN == 4 && HEAD == UN) {   // whole rounds of four as they are: eight in flight at first cost 1 to 4 %
        rounds(head, rows);
    } else if (rows == HEAD) {
#pragma unroll
        for (auto& v : head) add(v);
    } else {
        fetch(x);
#pragma unroll
        for (auto& v : head) add(v);
        rounds(x, rows - HEAD);
    }
    return acc;
}
template <bool FULL, int UN, int HEAD>
__device__ __forceinline__ void encode_rep_generic_body(const float* __restrict__ G, int64_t ldg,
                                                        float* __restrict__ Z, int64_t ldm, int groups, int rows,
                                                        int copies, int64_t d, int64_t c0) {
    if (!FULL && c0 >= d) return;
    const int n = FULL ? 4 : clamp4(d - c0);
    const int g = (int)blockIdx.y;   // one group per workgroup (grid.y = groups)
    if (g >= groups) return;
    const float4 sum = sum_rows<FULL, UN, HEAD>(G + (int64_t)g * rows * ldg + c0, ldg, rows, n);
    float* dst = Z + (int64_t)g * copies * ldm + c0;
    for (int i = 0; i < copies; ++i) stx<FULL>(dst + (int64_t)i * ldm, sum, n);
}

// Four rows at a time; eight where a launch leaves CUs idle ((10, 2, B = 160, 50 001), 98 workgroups: 14.1 us, 18.2 with four), and
// where five to eight are added (all of them in flight).  Encoder in us, in bursts of eight at any length / so: (45, 2, B = 180, 1 663 371) 258 / 255, (45, 1,
// B = 180, 400 001) 63.3 / 62.5, (10, 2, B = 160, 200 000) 24.7 / 23.4; (10, 2, B = 160, 50 001) 15.1 / 14.1.  One workgroup
// per CU, which suits r rows in and r out (below), loses 4 to 60 % here.
template <bool SPREAD, int UN, int HEAD>
__global__ __launch_bounds__(kBlock) void encode_rep_generic_kernel(const float* __restrict__ G, int64_t ldg,
                                                                    float* __restrict__ Z, int64_t ldm,
                                                                    int groups, int rows, int copies, int64_t d) {
    const int64_t c0 = lane_column<SPREAD>(d);
    if (block_is_full<SPREAD>(d, d)) encode_rep_generic_body<true, UN, HEAD>(G, ldg, Z, ldm, groups, rows, copies, d, c0);
    else encode_rep_generic_body<false, UN, HEAD>(G, ldg, Z, ldm, groups, rows, copies, d, c0);
}

// Majority candidate among R bit patterns of one coordinate (the streaming vote of
// Algorithm 2): one candidate and its lead over everything else seen so far, updated with
// selects only.  A copy that agrees raises the lead, one that differs lowers it, and when
// the lead is used up the next copy takes over as candidate.  If some pattern is held by
// more than half of the copies it is the result.
__device__ __forceinline__ void vote_step(uint32_t copy, uint32_t& candidate, int& lead) {
    const bool vacant = lead == 0;
    const int delta = (copy == candidate) ? 1 : -1;
    candidate = vacant ? copy : candidate;
    lead = vacant ? 1 : lead + delta;
}
template <int R>
__device__ __forceinline__ uint32_t vote(const uint32_t (&v)[R]) {
    uint32_t candidate = v[0];
    int lead = 1;
#pragma unroll
    for (int i = 1; i < R; ++i) vote_step(v[i], candidate, lead);
    return candidate;
}

// Node flags of one wavefront (wavefront-uniform values, kept in scalar registers).
struct WaveFlags {
    uint64_t w[kMaskWords] = {0, 0, 0, 0};
    __device__ __forceinline__ void set(int node) {
        const uint64_t bit = 1ull << (node & 63);
        const int word = node >> 6;
        if (word == 0) w[0] |= bit;
        else if (word == 1) w[1] |= bit;
        else if (word == 2) w[2] |= bit;
        else w[3] |= bit;
    }
};
static_assert(kMaskWords == 4, "WaveFlags::set spells out four words");

// Where a vote's flags go.  flags: kMaskWords words of node flags (and, for votes that finish
// themselves, one that counts workgroups), all zero between calls.
struct VoteOut {
    uint64_t* flags;
    uint64_t* mask;     // ceil(P/64) words
    int32_t* status;
    int P, s;
};

// mask and status from the flag words, which are cleared for the next call (COUNTED: with the count).
// Run by one wavefront (a lane per group).
template <bool COUNTED>
__device__ __forceinline__ void finish_vote(const VoteOut& out) {
    unsigned long long word[kMaskWords];
    unsigned long long* flags = reinterpret_cast<unsigned long long*>(out.flags);
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) word[w] = __hip_atomic_load(flags + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int r = 2 * out.s + 1;
    bool bad = false;
    for (int g = threadIdx.x; g < out.P / r; g += 64) {
        int cnt = 0;
        for (int i = 0; i < r; ++i) {
            const int node = g * r + i, w = node >> 6;
            const unsigned long long bits = w == 0 ? word[0] : w == 1 ? word[1] : w == 2 ? word[2] : word[3];
            cnt += (int)((bits >> (node & 63)) & 1ull);
        }
        bad |= cnt > out.s;   // DRACO_NO_MAJORITY
    }
    const bool any = __ballot(bad) != 0ull;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kMaskWords; ++w) {
            if (w < (out.P + 63) / 64) out.mask[w] = word[w];
            __hip_atomic_store(flags + w, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if constexpr (COUNTED) __hip_atomic_store(flags + kMaskWords, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *out.status = any ? 1 : 0;
    }
}
__global__ __launch_bounds__(64) void decode_rep_finish_kernel(const VoteOut out) { finish_vote<false>(out); }

// ORs the wavefront-uniform flag words of the four wavefronts of a workgroup into the global flag
// words, touching global memory only for bits that are not set there yet.  FINISH (small launches):
// the last workgroup to do so finishes the vote; a kernel of its own for that costs 4 us, an eighth of
// the smallest step ((P, s, d) = (15, 1, 10 000): 32 us against 33).  A large launch cannot: the count
// is one address and takes about 40 ns a workgroup, so 11 000 of them would need 440 us.
//
// A liar is mostly seen by every workgroup, and those of the first turn end within a microsecond of each
// other: all saw the bit unset, and 500 to 1000 ORs of one address, 9 ns each, stood at its end.  So one
// workgroup in sixteen of each die sets its bits at once and the others look up to three more times, 0.4 us
// apart, before they do.  A bit that no other workgroup sets costs its own workgroup 3 us, and only that one.  One liar, before
// and after: (6, 1, 600 000) 14.8 -> 10.5 us, (10, 2, 1.1 M) 21.3 -> 15.0, (10, 2, 5 M) 46.2 -> 39.1, (45, 1, 600 000) 29.4
// -> 28.1, (45, 1, 11.2 M) 315 both; no liar the same.  One in eight, 0.2 us apart: 1.5 % behind; one in thirty-two, 0.6 us: the same.  A look
// at the start of the walk, to spare the one at its end, costs calls without a liar 2 to 7 %.
constexpr unsigned kVoteLeaders = 16;
constexpr int kVoteLooks = 3;
constexpr int kVoteNap = 16;      // s_sleep units of 64 clocks
template <bool FINISH>
__device__ __forceinline__ void publish_flags(const WaveFlags& wf, const VoteOut& out) {
    __shared__ unsigned long long sflags[kMaskWords];
    if (threadIdx.x < kMaskWords) sflags[threadIdx.x] = 0ull;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        if (wf.w[0]) atomicOr(&sflags[0], (unsigned long long)wf.w[0]);
        if (wf.w[1]) atomicOr(&sflags[1], (unsigned long long)wf.w[1]);
        if (wf.w[2]) atomicOr(&sflags[2], (unsigned long long)wf.w[2]);
        if (wf.w[3]) atomicOr(&sflags[3], (unsigned long long)wf.w[3]);
    }
    __syncthreads();
    unsigned long long* flags = reinterpret_cast<unsigned long long*>(out.flags);
    auto publish = [&](int w) {
        const unsigned long long mine = sflags[w];
        if (mine) {
            // (few workgroups: no look first, which would be a round trip of its own: (15, 1, 10 000) vote 7.6 us, 8.2 with)
            unsigned long long cur =
                FINISH ? 0ull : __hip_atomic_load(flags + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if constexpr (!FINISH) {
                const bool waits = (blockIdx.x >> 3) % kVoteLeaders != 0;   // (workgroup b runs on die b mod 8)
                for (int look = 0; waits && (mine & ~cur) && look < kVoteLooks; ++look) {
                    __builtin_amdgcn_s_sleep(kVoteNap);
                    cur = __hip_atomic_load(flags + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (mine & ~cur) (void)__hip_atomic_fetch_or(flags + w, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    if constexpr (!FINISH) {
        if (threadIdx.x < kMaskWords) publish(threadIdx.x);
    } else {
        __shared__ int last;
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 0; w < kMaskWords; ++w) publish(w);
            // Releases this workgroup's flags with its count and acquires those of the workgroups before
            // it, so the last one reads every flag.
            const unsigned long long before =
                __hip_atomic_fetch_add(flags + kMaskWords, 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            last = before + 1 == (unsigned long long)gridDim.x ? 1 : 0;
        }
        __syncthreads();
        if (last != 0 && threadIdx.x < 64) finish_vote<true>(out);
    }
}

// Vote of one group held in registers: returns the winner of each of the
// lane's four coordinates and ORs the flags of differing nodes (wavefront-
// uniform) into wflags.  Honest groups take the fast path: all copies equal,
// decided for the whole wavefront by one ballot.
template <int R>
__device__ __forceinline__ uint4 vote_group(const uint4 (&x)[R], int first_node, WaveFlags& wflags) {
    uint32_t differ = 0;
#pragma unroll
    for (int i = 1; i < R; ++i)
        differ |= (x[i].x ^ x[0].x) | (x[i].y ^ x[0].y) | (x[i].z ^ x[0].z) | (x[i].w ^ x[0].w);
    uint4 win = x[0];
    if (__ballot(differ != 0) != 0ull) {   // some lane of the wavefront saw a disagreement in this group
        uint32_t bad = 0;                  // bit i: copy i differs from the vote in one of my coordinates
        if (differ != 0) {
            uint32_t v[R];
#pragma unroll
            for (int i = 0; i < R; ++i) v[i] = x[i].x;
            win.x = vote<R>(v);
#pragma unroll
            for (int i = 0; i < R; ++i) bad |= (uint32_t)(v[i] != win.x) << i;
#pragma unroll
            for (int i = 0; i < R; ++i) v[i] = x[i].y;
            win.y = vote<R>(v);
#pragma unroll
            for (int i = 0; i < R; ++i) bad |= (uint32_t)(v[i] != win.y) << i;
#pragma unroll
            for (int i = 0; i < R; ++i) v[i] = x[i].z;
            win.z = vote<R>(v);
#pragma unroll
            for (int i = 0; i < R; ++i) bad |= (uint32_t)(v[i] != win.z) << i;
#pragma unroll
            for (int i = 0; i < R; ++i) v[i] = x[i].w;
            win.w = vote<R>(v);
#pragma unroll
            for (int i = 0; i < R; ++i) bad |= (uint32_t)(v[i] != win.w) << i;
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (__ballot((bad >> i) & 1u) != 0ull) wflags.set(first_node + i);
        }
    }
    return win;
}

// D^Rep: per coordinate and group, the vote over the r copies; winners are
// summed over groups in ascending order; a node is flagged when any of its
// coordinates differs from the winner.  GU groups are loaded before the first
// is voted on (GU*R 16-byte loads in flight per lane).
template <int R, int GU, bool FULL>
__device__ __forceinline__ void decode_rep_body(const float* __restrict__ Rm, int64_t ldm, float* __restrict__ u,
                                                WaveFlags& wflags, int groups, int64_t d) {
    const int64_t c0 = lane_column<kSpreadVote>(d);
    const bool active = FULL || c0 < d;
    const int n = FULL ? 4 : (active ? clamp4(d - c0) : 0);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int g0 = 0; g0 < groups; g0 += GU) {
        uint4 x[GU][R];
#pragma unroll
        for (int a = 0; a < GU; ++a) {
            if (g0 + a < groups) {
                const float* src = Rm + (int64_t)(g0 + a) * R * ldm + c0;
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);   // lanes past the end vote on zeros
                    if (active) t = ldx<FULL>(src + (int64_t)i * ldm, n);
                    x[a][i] = make_uint4(__float_as_uint(t.x), __float_as_uint(t.y), __float_as_uint(t.z),
                                         __float_as_uint(t.w));
                }
            }
        }
#pragma unroll
        for (int a = 0; a < GU; ++a) {
            if (g0 + a < groups) {
                const uint4 win = vote_group<R>(x[a], (g0 + a) * R, wflags);
                acc.x += __uint_as_float(win.x);
                acc.y += __uint_as_float(win.y);
                acc.z += __uint_as_float(win.z);
                acc.w += __uint_as_float(win.w);
            }
        }
    }
    if (active) stx<FULL>(u + c0, acc, n);
}

template <int R, int GU, bool FINISH>
__global__ __launch_bounds__(kBlock) void decode_rep_kernel(const float* __restrict__ Rm, int64_t ldm,
                                                            float* __restrict__ u, const VoteOut out,
                                                            int groups, int64_t d) {
    WaveFlags wflags;
    if (block_is_full<kSpreadVote>(d, d)) decode_rep_body<R, GU, true>(Rm, ldm, u, wflags, groups, d);
    else decode_rep_body<R, GU, false>(Rm, ldm, u, wflags, groups, d);
    publish_flags<FINISH>(wflags, out);
}

// Any r: the copies of a group stream through the vote's two words of state per
// coordinate (candidate, lead), eight rows in flight, so every message byte is read
// once.  Only where some lane of the wavefront saw a copy differ from the first one is the
// group read again, to flag the nodes that differ from the winner.
template <bool FULL>
__device__ __forceinline__ void decode_rep_stream_body(const float* __restrict__ Rm, int64_t ldm,
                                                       float* __restrict__ u, WaveFlags& wflags, int groups,
                                                       int r, int64_t d) {
    constexpr int UN = 8;
    const int64_t c0 = lane_column<kSpreadVote>(d);
    const bool active = FULL || c0 < d;
    const int n = FULL ? 4 : (active ? clamp4(d - c0) : 0);
    auto fetch = [&](const float* p) -> uint4 {
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);   // lanes past the end vote on zeros
        if (active) t = ldx<FULL>(p, n);
        return make_uint4(__float_as_uint(t.x), __float_as_uint(t.y), __float_as_uint(t.z), __float_as_uint(t.w));
    };
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int g = 0; g < groups; ++g) {
        const float* src = Rm + (int64_t)g * r * ldm + c0;
        uint4 ma = make_uint4(0u, 0u, 0u, 0u), first = ma;   // ma: the four coordinates' candidates
        int cx = 0, cy = 0, cz = 0, cw = 0;                   // their leads (0: no candidate yet)
        uint32_t differ = 0;
        for (int i0 = 0; i0 < r; i0 += UN) {
            uint4 x[UN];
#pragma unroll
            for (int i = 0; i < UN; ++i)
                if (i0 + i < r) x[i] = fetch(src + (int64_t)(i0 + i) * ldm);
#pragma unroll
            for (int i = 0; i < UN; ++i) {
                if (i0 + i < r) {
                    if (i0 + i == 0) first = x[i];
                    differ |= (x[i].x ^ first.x) | (x[i].y ^ first.y) | (x[i].z ^ first.z) | (x[i].w ^ first.w);
                    vote_step(x[i].x, ma.x, cx);
                    vote_step(x[i].y, ma.y, cy);
                    vote_step(x[i].z, ma.z, cz);
                    vote_step(x[i].w, ma.w, cw);
                }
            }
        }
        if (__ballot(differ != 0) != 0ull) {
            for (int i = 0; i < r; ++i) {
                const uint4 x = fetch(src + (int64_t)i * ldm);
                const bool bad = (x.x != ma.x) | (x.y != ma.y) | (x.z != ma.z) | (x.w != ma.w);
                if (__ballot(bad) != 0ull) wflags.set(g * r + i);
            }
        }
        acc.x += __uint_as_float(ma.x);
        acc.y += __uint_as_float(ma.y);
        acc.z += __uint_as_float(ma.z);
        acc.w += __uint_as_float(ma.w);
    }
    if (active) stx<FULL>(u + c0, acc, n);
}

template <bool FINISH>
__global__ __launch_bounds__(kBlock) void decode_rep_generic_kernel(const float* __restrict__ Rm, int64_t ldm,
                                                                    float* __restrict__ u, const VoteOut out,
                                                                    int groups, int r, int64_t d) {
    WaveFlags wflags;
    if (block_is_full<kSpreadVote>(d, d)) decode_rep_stream_body<true>(Rm, ldm, u, wflags, groups, r, d);
    else decode_rep_stream_body<false>(Rm, ldm, u, wflags, groups, r, d);
    publish_flags<FINISH>(wflags, out);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

// Groups fetched per round (GU0 .. GU3 for r = 1, 3, 5, 7, one group otherwise) and workgroups per CU
// (BPC1 .. BPC3 for r = 3, 5, 7, BPC otherwise; 0: unlimited): keeps r * groups 16-byte loads in flight
// per lane.
#define DRACO_REP_DISPATCH(KERNEL, GU0, GU1, BPC1, GU2, BPC2, GU3, BPC3, BPC)              \
    switch (s) {                                                                           \
        case 0: KERNEL(1, GU0, BPC); break;                                                \
        case 1: KERNEL(3, GU1, BPC1); break;                                               \
        case 2: KERNEL(5, GU2, BPC2); break;                                               \
        case 3: KERNEL(7, GU3, BPC3); break;                                               \
        case 4: KERNEL(9, 1, BPC); break;                                                  \
        case 5: KERNEL(11, 1, BPC); break;                                                 \
        case 6: KERNEL(13, 1, BPC); break;                                                 \
        case 7: KERNEL(15, 1, BPC); break;                                                 \
        default: generic = true;                                                           \
    }

namespace {

// Which footprint the encoders take: see encode_rep_kernel.
bool on_lines(int64_t ldm) { return ldm % 32 == 0; }

// With two workgroups per CU, 513 to 768 of them would be one full turn and one nearly empty: four per CU make it one.  Sums over more
// than r rows, two per CU / four: (15, 2, B = 240, 180 907) 42.8 / 36.1 us, (28, 3, B = 56, 135 681) 10.9 / 10.5, (20, 2, B = 80,
// 131 603) 13.2 / 11.7; near 768 the same; from 900 workgroups on four are 0 to 6 % behind.  Three copies: (6, 1, 786 048) 8.1 / 7.0
// us; five copies have no such step (four: 4 to 9 % behind).
bool spills_two_per_cu(int64_t workgroups) { return workgroups > 512 && workgroups <= 768; }

template <class F, int... K>
void one_to(F&& f, std::integer_sequence<int, K...>) {
    (f(std::integral_constant<int, K + 1>()), ...);
}

// Sums of `rows` rows per group, stored `copies` times (copies = 1: one row, its stride does not matter).
void launch_generic(const float* G, int64_t ldg, float* Z, int64_t ldm, int groups, int rows, int copies, int per_cu,
                    int64_t d, hipStream_t stream) {
    auto go = [&](auto spread, auto ahead, auto first) {
        constexpr bool SPREAD = decltype(spread)::value;
        constexpr int UN = decltype(ahead)::value, HEAD = decltype(first)::value;
        if (rows < HEAD || (rows - HEAD) % UN != 0) return;
        const dim3 grid(grid_cols<SPREAD>(d), (unsigned)groups);
        if (per_cu == 2 && spills_two_per_cu((int64_t)grid.x * grid.y)) per_cu = 4;
        allow_large_lds<encode_rep_generic_kernel<SPREAD, UN, HEAD>>();
        hipLaunchKernelGGL((encode_rep_generic_kernel<SPREAD, UN, HEAD>), grid, dim3(kBlock), throttle_lds(per_cu, 0, 0), stream,
                           G, ldg, Z, ldm, groups, rows, copies, d);
    };
    auto any_head = [&](auto spread, auto ahead) {   // (go launches one of them)
        one_to([&](auto first) { go(spread, ahead, first); }, std::make_integer_sequence<int, decltype(ahead)::value>());
    };
    auto depth = [&](auto spread) {
        const bool idle = (int64_t)grid_for((d + 3) / 4) * groups < 256;
        // (up to four rows are all in flight either way, and fewer registers let more workgroups onto a CU)
        if ((rows > 4 && rows <= 8) || idle) any_head(spread, std::integral_constant<int, 8>{});
        else any_head(spread, std::integral_constant<int, 4>{});
    };
    if (on_lines(ldm)) depth(std::true_type{});
    else depth(std::false_type{});
}

}  // namespace

namespace {

template <bool SPREAD>
void launch_groups(const float* G, int64_t ldg, float* Z, int64_t ldm, int P, int s, int64_t d, hipStream_t stream) {
    const int r = 2 * s + 1, groups = P / r;
    const unsigned tiles = grid_cols<SPREAD>(d);
    const dim3 block(kBlock);
    bool generic = false;
    // Three copies: two workgroups per CU on the line grid ((45, 1, 11.2 M) 612 us, 631 with one), one off it (5 M + 1: 312, 323 with
    // two).  Five copies: two, but for long launches off it ((45, 2, 1 663 371) 100 us, 103 with two; 500 001 32 and 31).
    // Seven copies and more: one; but seven and nine two in launches of a few turns, whose last one is a large part ((42, 3, 85 334)
    // 7.2 -> 6.3 us, (42, 3, 170 667) 12.6 -> 12.1, (45, 4, 161 793) 13.1 -> 12.4; in more workgroups the same or 1 to 4 %
    // behind, nine copies in less than two turns 2 %, eleven and more 1 to 4 % at any length).
    const int64_t all = (int64_t)tiles * groups;
    const int three = spills_two_per_cu((int64_t)tiles * ((groups + 1) / 2)) ? 4 : SPREAD ? 2 : 1;
    const int five = !SPREAD && all >= 12000 ? 1 : 2;
    const int seven = all > 256 && all <= 1280 ? 2 : 1, more = s == 4 && all > 512 && all <= 1536 ? 2 : 1;
#define DRACO_LAUNCH(R, GU, BPC)                                                                                \
    {                                                                                                           \
        allow_large_lds<encode_rep_kernel<R, GU, SPREAD>>();                                                    \
        hipLaunchKernelGGL((encode_rep_kernel<R, GU, SPREAD>), dim3(tiles, (unsigned)((groups + GU - 1) / GU)), \
                           block, throttle_lds(BPC, 0, 0), stream, G, ldg, Z, ldm, groups, d);                  \
    }
    DRACO_REP_DISPATCH(DRACO_LAUNCH, 8, 2, three, 1, five, 1, seven, more)
#undef DRACO_LAUNCH
    if (generic) launch_generic(G, ldg, Z, ldm, groups, r, r, 2, d, stream);
}

}  // namespace

hipError_t launch_encode_rep(const float* G, int64_t ldg, float* Z, int64_t ldm, int P, int s, int64_t d,
                             hipStream_t stream) {
    if (on_lines(ldm)) launch_groups<true>(G, ldg, Z, ldm, P, s, d, stream);
    else launch_groups<false>(G, ldg, Z, ldm, P, s, d, stream);
    return hipGetLastError();
}

hipError_t launch_encode_rep_samples(const float* G, int64_t ldg, int m, float* Z, int64_t ldm, int P, int s, int64_t d,
                                     hipStream_t stream) {
    const int r = 2 * s + 1;
    launch_generic(G, ldg, Z, ldm, P / r, r * m, r, 2, d, stream);
    return hipGetLastError();
}

hipError_t launch_encode_rep_node(const float* Gn, int64_t ldg, float* z, int s, int64_t d, hipStream_t stream) {
    launch_generic(Gn, ldg, z, 0, 1, 2 * s + 1, 1, 0, d, stream);
    return hipGetLastError();
}

namespace {

// The vote, with its finish in the same launch (FINISH) or in a kernel of its own.  FEW: rows too short
// to fill the chip take more groups at a time, workgroups unlimited.
template <bool FEW, bool FINISH>
void launch_vote(const float* R, int64_t ldm, float* u, const VoteOut& out, int64_t d, hipStream_t stream) {
    const int s = out.s, r = 2 * s + 1, groups = out.P / r;
    const dim3 grid(grid_cols<kSpreadVote>(d)), block(kBlock);
    constexpr size_t fixed = kMaskWords * sizeof(unsigned long long) + (FINISH ? 8 : 0);   // static LDS of publish_flags
    bool generic = false;
#define DRACO_LAUNCH(R_, GU, BPC)                                                                                  \
    {                                                                                                              \
        allow_large_lds<decode_rep_kernel<R_, GU, FINISH>>(fixed);                                                 \
        hipLaunchKernelGGL((decode_rep_kernel<R_, GU, FINISH>), grid, block, throttle_lds(BPC, fixed, 0), stream,  \
                           R, ldm, u, out, groups, d);                                                             \
    }
    if constexpr (FEW) {
        DRACO_REP_DISPATCH(DRACO_LAUNCH, 4, 5, 0, 3, 0, 2, 0, 2)
    } else {
        // Workgroups per CU.  Long launches: two, but four for r = 5 (6.4 against 6.25 TB/s) and for r = 3 over six groups or
        // fewer, whose walks are too short to keep two workgroups' loads in flight ((6, 1, 11.2 M) 55 -> 51 us, with a liar 66 ->
        // 54; (18, 1, 6 M) 75 -> 73; but (45, 1, 4 M) 109 -> 111).  Short ones: as many as put them into one turn, where a second one
        // would be nearly empty: four up to 1024 workgroups ((45, 1, 600 000) 26.9 -> 21.6), r >= 7, whose second turn costs
        // less, up to 768 ((45, 4, 700 001) 27.9 -> 26.0; at 950 000 32.4 and 33.4), and six up to 1280 where one turn of them is well
        // filled ((45, 1, 1.3 M) 42.4 -> 39.9, (45, 2, 1 200 001) 47.1 -> 41.8; at 1.5 M 48.0 and 50.8, 51.4 and 50.4);
        // (6, 1) with a liar loses 0.5 of 11 and 13 us at 1.0 and 1.3 M).
        const unsigned c = grid.x;
        const int three = c <= 1024 ? 4 : c <= 1280 ? 6 : groups <= 6 ? 4 : 2;
        const int five = c > 1024 && c <= 1280 ? 6 : 4, more = c <= 768 ? 4 : 2;
        DRACO_REP_DISPATCH(DRACO_LAUNCH, 4, 1, three, 1, five, 1, more, more)
    }
#undef DRACO_LAUNCH
    if (generic) {
        allow_large_lds<decode_rep_generic_kernel<FINISH>>(fixed);
        hipLaunchKernelGGL(decode_rep_generic_kernel<FINISH>, grid, block, throttle_lds(2, fixed, 0), stream, R, ldm, u,
                           out, groups, r, d);
    }
    if constexpr (!FINISH) hipLaunchKernelGGL(decode_rep_finish_kernel, dim3(1), dim3(64), 0, stream, out);
}

}  // namespace

hipError_t launch_decode_rep(const float* R, int64_t ldm, float* u, uint64_t* flags, uint64_t* mask_out,
                             int32_t* status_out, bool counted, int P, int s, int64_t d, hipStream_t stream) {
    const unsigned workgroups = grid_cols<kSpreadVote>(d);
    const VoteOut out{flags, mask_out, status_out, P, s};
    if (counted && workgroups < 64) launch_vote<true, true>(R, ldm, u, out, d, stream);
    else if (workgroups < 256) launch_vote<true, false>(R, ldm, u, out, d, stream);
    else launch_vote<false, false>(R, ldm, u, out, d, stream);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// D^Rep without any allocation: the node-flag words live in a device array that is part of
// the loaded code object, one copy per GPU, kept until the process ends.
// ---------------------------------------------------------------------------
namespace {

// Node flags of the allocation-free decoder: kMaskWords 64-bit words (one bit per node,
// kMaxNodes nodes at most).  In host code this name is only a handle for
// hipGetSymbolAddress; kernels receive the address that call returns.
static __device__ __align__(256) unsigned long long scratch[kMaskWords];

constexpr int kMaxDevices = 64;
uint64_t* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each GPU, resolved once
std::mutex g_scratch_mutex;

__global__ void clear_flags_kernel(uint64_t* __restrict__ flags) {
    if (blockIdx.x == 0 && threadIdx.x < kMaskWords) flags[threadIdx.x] = 0;
}

// Address of the current device's copy of `scratch` (resolved on the first call per device).
hipError_t static_flags(uint64_t** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<uint64_t*>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

hipError_t launch_decode_rep_static(const float* R, int64_t ldm, float* u, uint64_t* mask_out, int32_t* status_out,
                                    int P, int s, int64_t d, hipStream_t stream) {
    uint64_t* flags = nullptr;
    hipError_t e = static_flags(&flags);
    if (e != hipSuccess) return e;
    // the array keeps what the last call left (zero after a call that ran to its end); a fill
    // kernel, not a memset, so that the sequence can be captured in a HIP graph
    hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(64), 0, stream, flags);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // not counted: another call's workgroups would be counted too, and then neither call's mask and
    // status might be written
    return launch_decode_rep(R, ldm, u, flags, mask_out, status_out, false, P, s, d, stream);
}


}  // namespace draco
