/*
 * draco_bench.h -- measuring instruments of the DRACO library: a calibration
 * copy kernel and per-kernel timing.  None of this is part of the method's
 * boundary (include/draco.h); the benchmark and the profiles use it.
 */
#ifndef DRACO_BENCH_H
#define DRACO_BENCH_H

#include "draco.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Plain device-to-device copy of a [rows][ld] fp32 slab (row_len floats used
 * per row; row_len and ld multiples of 4, pointers 16-byte aligned; rows <=
 * 65535) with 16-byte non-temporal accesses, one 4 KiB piece of one row per
 * workgroup, pieces of a row varying fastest: a calibration kernel, the fastest
 * slab copy found on this GPU.  Timing it gives the copy bandwidth the GPU
 * sustains (the ceiling of the encoders, which read and write equal amounts);
 * profiling it gives the scale of the hardware byte counters for a known
 * 2*4*rows*row_len bytes.  Asynchronous on `stream`. */
int draco_copy_probe(const float* src_dev, float* dst_dev, int rows, int64_t row_len, int64_t ld,
                     void* stream);

/* Kernel timing with HIP events recorded on the stream each kernel is launched
 * on.  draco_plan_set_timing(plan, n) gives every kernel kind n event pairs
 * (n = 0 switches timing off); from then on each launch of a kind uses the next
 * free pair (launches beyond n are not timed) and nothing waits.
 * draco_plan_kernel_time waits for the recorded kernels of one kind, returns
 * their summed duration in milliseconds and their number, and frees the pairs
 * for reuse.  draco_plan_kernel_times does the same but writes each launch's
 * duration, in launch order, to ms_host[0 .. min(*launches, capacity)).
 * kind: 0 encode, 1 repetition vote, 2 cyclic projection (with its small
 * reduction), 3 cyclic recombination (and the locator where one kernel does
 * both: rows of up to 65 536 floats, and messages of at most 320 MiB of at most
 * 64 nodes whose rows have 256 tiles of 1024 floats or more, 65 or more on up to
 * 8 nodes), 4 the cyclic locator (phi steps 2-4 and b, one wavefront) as a
 * kernel of its own. */
int draco_plan_set_timing(draco_plan* plan, int max_records);
int draco_plan_kernel_time(draco_plan* plan, int kind, double* total_ms, int* launches);
int draco_plan_kernel_times(draco_plan* plan, int kind, double* ms_host, int capacity,
                            int* launches);

/* What a cyclic plan that has been prepared expects of its next decode and what
 * became of the last one (waits for the device): words_host[0] clean decodes in
 * a row, up to the number from which no sample is taken; [1] what the last
 * decode's projection speculated on: 0 nothing, 1 nobody, 2 the set located on a
 * sample; [2] 1 if that was the set found, so that the second pass was left out;
 * [3] the status of the last sample's locator; [4] decodes left that take no
 * sample after samples that misled; [5] samples in a row that misled.
 * DRACO_EINVAL for other plans. */
int draco_plan_speculation_state(draco_plan* plan, int32_t* words_host);

#ifdef __cplusplus
}
#endif
#endif /* DRACO_BENCH_H */
