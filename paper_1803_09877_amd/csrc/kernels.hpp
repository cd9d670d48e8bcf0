// Launchers of the gfx950 kernels behind the C ABI.  All pointers are device
// pointers; every launcher only enqueues work on `stream` and returns the HIP
// error of the launch.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace draco {

constexpr int kBlock = 256;           // threads per workgroup (4 wavefronts of 64)
constexpr int kMaxS = 7;              // repetition kernels are specialised for r = 2s+1 <= 15; larger r takes the generic path
constexpr int kMaxCycS = 10;          // cyclic encoder: two complex per lane up to r = 21, one per lane up to r = 33, an LDS ring beyond
constexpr int kMaxNodes = 256;        // DRACO_MAX_NODES
constexpr int kMaskWords = 4;         // 64-bit words of node flags (kMaxNodes / 64)
constexpr int kVoteWords = kMaskWords + 1;   // and the vote's count of workgroups
// Messages of a whole step (both words, bytes) up to which kernels count on the 256 MiB memory-side
// cache: measured wins at 216 and 270 MB, losses at 450 MB and beyond.
constexpr int64_t kSmallMessages = 320ll << 20;
// Messages up to which the joint pass leaves its rows there as well.  It is the only pass if the speculation holds, and larger
// messages that come from elsewhere stream faster: steps over states in turn / over the same messages again, plain loads 1:
// 120 to 145 MB 0.94 to 1.02 / 1.01 to 1.10, 160 to 270 MB 0.94 to 1.00 / 0.97 to 1.02 ((45, 3, 1 200 001), 5 bytes: 193 -> 182 us).
constexpr int64_t kCachedMessages = 144ll << 20;
constexpr int kLocateMaxS = 16;       // largest s the on-device locator handles

// Which kernel families spread a workgroup's wavefronts over a 128 KiB window of each row
// (device_util.hpp, "workgroup footprint"); chosen per family by measurement.  The repetition encoder goes by its rows'
// stride alone (rep.hip).
constexpr bool kSpreadEncodeCyc = true;
constexpr bool kSpreadVote = true;
constexpr bool kSpreadRecombine = true;
constexpr bool kSpreadUpdate = true;

// Complex numbers in device tables: (re, im) as double2.

// ---- repetition code ----
hipError_t launch_encode_rep(const float* G, int64_t ldg, float* Z, int64_t ldm, int P, int s,
                             int64_t d, hipStream_t stream);
hipError_t launch_encode_rep_node(const float* Gn, int64_t ldg, float* z, int s, int64_t d,
                                  hipStream_t stream);
// The vote; mask_out <- node flags; status_out <- NO_MAJORITY if a group has more than s of them.
// flags[kMaskWords] is scratch, zero on entry and left zero; counted: it holds one word more, which
// lets the last workgroup of a small launch write mask and status (flags no other call uses).
hipError_t launch_decode_rep(const float* R, int64_t ldm, float* u, uint64_t* flags, uint64_t* mask_out,
                             int32_t* status_out, bool counted, int P, int s, int64_t d, hipStream_t stream);
// The same on flag words held in a device array of the library itself (one per
// GPU, shared by every call on that GPU): no allocation anywhere.
hipError_t launch_decode_rep_static(const float* R, int64_t ldm, float* u, uint64_t* mask_out,
                                    int32_t* status_out, int P, int s, int64_t d, hipStream_t stream);

// B > P: the gradient slab holds m = B/P per-sample rows per unit gradient (rows k*m .. k*m+m-1).
hipError_t launch_encode_rep_samples(const float* G, int64_t ldg, int m, float* Z, int64_t ldm, int P,
                                     int s, int64_t d, hipStream_t stream);

// ---- cyclic code ----
// coef[n*(2s+1) + t] = W[(n+t) mod P][n]: the weight node n gives its t-th assigned gradient
// (used by the unpacked wire).  The packed encoders take W factored, W[(n+t) mod P][n] =
// rotA[n] * rho[t] * rotB[n+t] with real rho[2s+1], unit rotA[P] and unit rotB[P+2s] (indexed by
// the unwrapped row n + t): device pointers.
struct CycTaps {
    const double* rho;
    const double2* rotA;
    const double2* rotB;
};
// Zlo / zlo / Rlo below: second word of the two-word wire (message = hi + lo), or nullptr;
// lo names its format: kSecondWordF32 (a float slab), kSecondWordBf16 (a bfloat16 slab) or
// kSecondWordI8 (a slab of 8-bit residual codes), each with the same row stride counted in
// ELEMENTS.  Ignored when the pointer is null.
constexpr int kSecondWordF32 = 1, kSecondWordBf16 = 2, kSecondWordI8 = 3;
// B > P on the cyclic code (rows as for launch_encode_rep_samples).
hipError_t launch_encode_cyc_samples(const float* G, int64_t ldg, int m, float* Z, float* Zlo, int lo,
                                     int64_t ldm, const CycTaps& tab, int P, int s, int64_t d, hipStream_t stream);
hipError_t launch_encode_cyc(const float* G, int64_t ldg, float* Z, float* Zlo, int lo, int64_t ldm,
                             const CycTaps& tab, int P, int s, int64_t d, hipStream_t stream);
// Unpacked wire: real gradients [P][d] in, messages of d complex entries (2d floats) out.
hipError_t launch_encode_cyc_real(const float* G, int64_t ldg, float* Z, int64_t ldm, const double2* coef,
                                  int P, int s, int64_t d, hipStream_t stream);
// Gn holds only the node's 2s+1 gradients, in assignment order.
hipError_t launch_encode_cyc_real_node(const float* Gn, int64_t ldg, float* z, const double2* coef, int node,
                                       int P, int s, int64_t d, hipStream_t stream);
hipError_t launch_encode_cyc_node(const float* Gn, int64_t ldg, float* z, float* zlo, int lo,
                                  const CycTaps& tab, int node, int P, int s, int64_t d, hipStream_t stream);
// What a decode expects before it has located anybody (device memory of a plan).
//   state[kSpecClean]   clean decodes in a row, up to kCleanRun (a new plan starts with one)
//   state[kSpecNow]     what the projection pass of this call speculated on: 0, kSpecOnNobody, kSpecOnSample
//   state[kSpecDone]    1 if the locator found that set: the output holds the sum already
//   state[kSpecStatus]  of the locator on this call's sample
//   state[kSpecSkip]    decodes left that take no sample, state[kSpecMisses]: samples in a row that misled
//   mask, b             the set located on a sample of this call's messages (kMaskWords) and its
//                       recombination vector (P, dense); mask == nullptr where no sample is taken
// state == nullptr: never speculate.
enum : int { kSpecClean = 0, kSpecNow = 1, kSpecDone = 2, kSpecStatus = 3, kSpecSkip = 4, kSpecMisses = 5, kSpecWords = 6 };
enum : int { kSpecOnNobody = 1, kSpecOnSample = 2 };
struct CycSpec {
    int32_t* state;
    uint64_t* mask;
    double2* b;
};
constexpr int kSampleTiles = 64;      // of 1024 floats
constexpr int kShortTiles = 255;      // 4 KiB tiles of the longest rows that count as short,
constexpr int kFusedTiles = 64;       // and of those that are located and recombined by one kernel: a workgroup per CU has 1 KiB each
// Partial sums up to which the locator adds them itself; more of them take longer there than a launch (decodes with that
// launch / without, us: 98 tiles of 8 nodes 17.3 / 14.6, 20 17.3 / 15.1, 45 20.0 / 19.2, 100 33.9 / 35.4; 127 of 20 17.4 / 15.9,
// 45 21.0 / 20.9, 100 37.2 / 39.8).
inline int64_t inline_tiles(int P) { return P <= 64 ? 128 : 64; }
// Messages (both words, bytes) from which a decode may locate the adversaries on a sample first and
// then project and recombine in ONE pass.  The sample and its locator take 11 to 20 us and the
// joint pass 10 % more than a projection; the second pass they save runs at about 6.3 TB/s, so with
// adversaries it broke even near 250 MB when the sample and its locator took 15 to 30 (the line has not been measured again since).
constexpr int64_t kSampledMessages = 384ll << 20;
// A plan that saw kCleanRun clean decodes in a row expects nobody and takes no sample (15 to 20 us, 8 % of a
// clean step at (15, 2, 8 M)); until then, and after a decode that found somebody, it samples.  A
// lie that the sample does not hold (it need not touch every coordinate) costs the sample and the joint pass's
// surcharge on top of the two passes, 3 % of a step at (45, 3, 25.6 M); after the n-th such miss in a
// row the next 2^n - 1 decodes project only, so a persistent one costs that in 1 of 256 decodes.
constexpr int kCleanRun = 8;
constexpr int kMaxMisses = 8;
// Whether a call that has room for a sample (mask != nullptr) takes one.  All its kernels ask; the state
// changes in the last locator only.
__device__ __forceinline__ bool takes_sample(const CycSpec& spec) {
    return spec.state[kSpecClean] < kCleanRun && spec.state[kSpecSkip] == 0;
}

// Number of workgroups (= rows of `partial`) the projection uses for gradient length d and row stride ldm, the most it
// uses for any stride, and whether rows of d floats are short (the projection is split over the nodes and does not speculate).
int64_t project_tiles(int64_t d, int P, int64_t ldm);
int64_t project_tiles_at_most(int64_t d, int P);
bool short_rows(int64_t d, int P);
// partial[tile][P] <- per-tile sums of f_i * R[j][i].  b0[P]: recombination vector for "no
// adversary"; u: output written speculatively.
// f == nullptr: the entries of f are generated from f_seed (projection_rng.hpp).
// d is the number of floats a message carries (odd d: one more, zero); realout (unpacked
// wire, messages of d/2 complex entries): u receives only the real parts, d/2 floats.
hipError_t launch_cyc_project(const float* R, const float* Rlo, int lo, int64_t ldm, const float* f,
                              uint64_t f_seed, double2* partial, const double2* b0, float* u, bool realout,
                              const CycSpec& spec, int P, int64_t d, hipStream_t stream);
// The same sums for a sample of the columns, partial[kSampleTiles][P]: which ones is drawn from f (its
// first entries, or its seed), which the adversaries do not know.  Nothing if this call takes no sample.
hipError_t launch_cyc_sample(const float* R, const float* Rlo, int lo, int64_t ldm, const float* f, uint64_t f_seed,
                             double2* partial, const CycSpec& spec, int P, int64_t d, hipStream_t stream);
// sums[parts][P] <- the sums of partial[tiles][P] over `parts` runs of tiles.  Tables of more than one round of loads go in
// parts, which the locator adds (0.5 us); shorter ones take as long as an empty kernel in one (4.8 us of 4.5).
constexpr int kReduceParts = 8;
inline int reduce_parts(int64_t tiles) { return tiles > 8 * kBlock ? kReduceParts : 1; }
hipError_t launch_cyc_reduce(const double2* partial, double2* sums, int parts, int P, int64_t tiles, hipStream_t stream);
// phi steps 2-4 and the recombination vector on the device (one wavefront, fp64; s <= kLocateMaxS):
// gamma[P] (tiles == 0) or partial[tiles][P] -> mask words, status, and the
// honest nodes' (idx, b) compacted in ascending order with their count in *nu_out.
// roots[k] = exp(2 pi i k / P), k < P.  tau: relative zero threshold for syndromes.  With no located
// node the coefficients are copied from b0.  b is a function of the set of flagged nodes.
// spec.state: kSpecDone <- the set found is the one speculated on; kSpecClean, kSpecSkip and kSpecMisses
// for the next call.
hipError_t launch_cyc_locate(const double2* sums, int64_t tiles, const double2* roots, int P, int s, double tau,
                             const double2* b0, uint64_t* mask_out, int32_t* status_out, double2* b_out,
                             int32_t* idx_out, int32_t* nu_out, const CycSpec& spec, hipStream_t stream);
// The same on the sums of a sample: spec.mask and spec.b <- the set found and its coefficients
// (b_out, idx_out, nu_out are scratch).  Nothing if this call takes no sample.
hipError_t launch_cyc_locate_sample(const double2* partial, const double2* roots, int P, int s, double tau,
                                    const double2* b0, double2* b_out, int32_t* idx_out, int32_t* nu_out,
                                    const CycSpec& spec, hipStream_t stream);
// Where the locator's kernel recombines too: rows that are one KiB per CU, and of at most 64 nodes (a locator's registers)
// the rows that are not short (65 to 255 tiles: 17 us, 22 in one launch at (45, 3, 70 001), whose recombination
// needs more wavefronts; on 8 nodes or fewer it does not: 222 decodes of such rows take 0.63 to 0.93 of the time in two launches with
// the general locator, (8, 2, 117 459) with two liars 21.7 -> 17.0 us, (8, 1, 206 494) with none 14.5 -> 12.0), in messages that stay in the memory-side cache.  Beyond, two workgroups per CU recombine up to 3 % slower
// ((15, 2, 4 M) on the 6-byte wire: 119 and 121 us), and after a sample the locator alone finds its code in the instruction
// cache ((45, 7, 6 M) on two fp32 words: a step of 962 us, 966 in one launch).
inline bool one_chunk_per_cu(int64_t d) { return (d + 1) / 2 * 2 <= kFusedTiles * kBlock * 4; }
inline bool recombines_in_locator(int P, int64_t d, int64_t message_bytes) {
    return one_chunk_per_cu(d) || (P <= 64 && !short_rows(d, P) && message_bytes <= kSmallMessages);
}
// Brings the locators' code to the device, which their first launch would do otherwise: 0.3 to 1.7 ms of a process's first decode,
// in the record of the kernel that recombines too.
hipError_t load_locator();
// The locator on sums[tiles][P] and the recombination in one launch.
hipError_t launch_cyc_locate_recombine(const double2* sums, int64_t tiles, const double2* roots, int P, int s, double tau,
                                       const double2* b0, uint64_t* mask_out, int32_t* status_out, const CycSpec& spec,
                                       const float* R, const float* Rlo, int lo, int64_t ldm, float* u, bool realout, int64_t d,
                                       hipStream_t stream);
// u <- unpack( sum_{q < *nu} b[q] * R[idx[q]] ); nu is read from device memory.  Nothing if
// state[kSpecDone] is set (state may be nullptr).
hipError_t launch_cyc_recombine(const float* R, const float* Rlo, int lo, int64_t ldm, const double2* b,
                                const int32_t* idx, const int32_t* nu, const int32_t* state, int P,
                                float* u, bool realout, int64_t d, hipStream_t stream);

// params[i] <- params[i] - scale * sum[i], i < d (the model update of mini-batch SGD).
hipError_t launch_apply_update(float* params, const float* sum, float scale, int64_t d, hipStream_t stream);

// dst[j][0..row_len) <- src[j][0..row_len) for j < rows, row_len a multiple of 4 floats
// (bandwidth / counter calibration).
hipError_t launch_copy_probe(const float* src, float* dst, int rows, int64_t row_len, int64_t ld,
                             hipStream_t stream);

}  // namespace draco
