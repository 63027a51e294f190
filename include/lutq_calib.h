/*
 * Measurement helpers exported by liblutq.so next to the lutq_* entry points.  They are not part of
 * the method of the paper: they exist so that a benchmark can (a) quote the read bandwidth that a
 * plain streaming kernel reaches on the same device beside the nominal HBM peak, (b) calibrate
 * the profiler's HBM byte counters against a copy of known size, and (c) ask which kernel a call goes to.
 */
#ifndef LUTQ_CALIB_H
#define LUTQ_CALIB_H

#include <stddef.h>
#include <stdint.h>

#include "lutq.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Reads `bytes` (multiple of 16) from device memory `src` (16-byte aligned) with `grid` workgroups of
 * 256 threads and discards them. `sink4`: 4 writable device bytes. Asynchronous on `stream`.
 * Returns 0, 1 (bad argument) or 9 (launch failed). */
int lutq_calib_stream_read(const void* src, size_t bytes, int grid, void* sink4, void* stream);

/* Copies `bytes` (multiple of 16) from `src` to `dst` (device, 16-byte aligned, not overlapping).
 * Reads `bytes` and writes `bytes` of HBM traffic.  Same return codes. */
int lutq_calib_copy(const void* src, void* dst, size_t bytes, int grid, void* stream);

/* One launch of lutq_matmul_plan (same arguments, same result in Y; plan NULL = the library's choice;
 * dtype 0 = fp16, 1 = bf16; M <= 4) through a measurement build of the kernel that also records where
 * the time of a launch goes: every wavefront reads the device's constant 100 MHz clock at eight points,
 *   0 wave started, 1 kernel arguments arrived, 2 first loads issued, 3 table built (barrier passed),
 *   4 first tile multiplied, 5 K loop done, 6 waves reduced, 7 outputs stored,
 * and writes them to trace[workgroup][wave][8] with 16 wave slots per workgroup (uint64, device memory,
 * 8-byte aligned, trace_bytes >= workgroups * 1024; slots of waves that do not exist stay untouched).  *workgroups receives the number of workgroups launched.
 * Measurement builds exist for 4-bit weights, group 64 or 128, plans with one or two row blocks per
 * wave and two tiles in flight; anything else returns 10 (plan).  Other return values are those of
 * lutq_matmul_plan (0 = launched; 7 = trace buffer too small).  Asynchronous on `stream`. */
int lutq_calib_matmul_trace(const void* X, const void* packed, const void* scales, const void* lut,
                            int bits, int group_size, int64_t M, int64_t N, int64_t K, int dtype,
                            void* Y, void* workspace, size_t workspace_bytes, void* stream,
                            const lutq_plan* plan, void* trace, size_t trace_bytes, int* workgroups);

/* How lutq_matmul serves a call without a plan on a device with `compute_units` compute
 * units (1..4096) and a workspace of `workspace_bytes`; host logic only, no device is touched (the plan
 * table counts).  route[0] = 0: one launch for all rows, each workgroup on 32 route[1] activation rows by
 * 64 route[2] output channels, with K cut into route[3] slices and M into route[4] parts; else
 * route[0] = the rows per launch of the slices it is served in (32 or 64) and the others are 0.  Up to 32 rows the call is one launch in
 * either case, and route[0] = 0 says that it is panels (17..32 rows, route[1] = 1).
 * Return values: 0, or the status lutq_matmul would give the problem (7 also for less than 64 KiB of workspace up to 32 rows). */
int lutq_calib_route(int bits, int group_size, int64_t M, int64_t N, int64_t K, int dtype, int compute_units,
                     size_t workspace_bytes, int route[5]);

/* The launch of a call of 1..32 rows with `plan` (NULL: without one; the plan table counts then), or, row_tables != 0, of a call of
 * lutq_matmul_channel (plan NULL; the table does not count), on a device with `compute_units`
 * compute units and a workspace of `workspace_bytes` (at least 64 KiB): *runs = the decomposition that is launched, with every field
 * given; all zero where it is one that no plan names (panels of 32 rows).  Host logic only, no device is touched.
 * Return values: 0, or the status lutq_matmul_plan would give the problem and the plan (SHAPE also for M > 32). */
int lutq_calib_plan(int bits, int group_size, int64_t M, int64_t N, int64_t K, int dtype, int compute_units,
                    size_t workspace_bytes, const lutq_plan* plan, int row_tables, lutq_plan* runs);

#ifdef __cplusplus
}
#endif
#endif /* LUTQ_CALIB_H */
