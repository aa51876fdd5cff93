/*
 * hv_inspect.h -- inspection entry points for tests: the chunk scheduler's
 * leaf table, the leaf-kernel choice and the Merkle launch plan.
 *
 * hv_leaf_schedule runs the same device-side scheduling hv_hash_chunks runs
 * (Algorithm 1's chunking: ceil(|M| / C) chunks per message, the last one
 * shorter) and copies the resulting leaf table to the host, so a test can
 * check that every chunk appears exactly once, with the right source range
 * and output slot, in non-increasing order of SHA-256 block count.  It does
 * not hash.  Synchronous on `stream`.
 *
 *   msgs, n_msgs, chunk_bytes, workspace, workspace_bytes: as hv_hash_chunks.
 *   table: host, n_leaves * 3 uint64 values, written in schedule order as
 *          {source device address, byte length, leaf index} per leaf.
 * Errors: as hv_hash_chunks (HV_ERR_INVALID_ARG for a NULL table with
 * n_leaves > 0).
 */
#ifndef HV_INSPECT_H
#define HV_INSPECT_H

#include "hv.h"

#ifdef __cplusplus
extern "C" {
#endif

hv_status hv_leaf_schedule(const hv_msg* msgs, uint32_t n_msgs, uint64_t chunk_bytes, uint64_t* table,
                           void* workspace, size_t workspace_bytes, hipStream_t stream);

/* Leaf-kernel choice for tests and measurements, per calling thread:
 * 0 = automatic (calls with at most 128 leaves per compute unit of the current
 * device -- 32768 on MI355X -- use the kernels that shorten each chunk's chain
 * of blocks, named two-wave here: the message schedule is made by other waves
 * than the rounds, and a chunk has two lanes, except with SHA-384 above 64
 * leaves per compute unit; others use the one-wave kernel), 1 = always the
 * one-wave kernel, 2 = always the two-wave kernel, 3 = always the two-wave
 * kernel with twice the chunks, 128, per workgroup (the layout it takes above
 * 64 leaves per compute unit; two lanes per chunk with SHA-256, one with
 * SHA-384).  From 128 to
 * 192 leaves per compute unit the automatic choice runs SHA-256's three-group
 * kernel (one lane per chunk, the schedules on other waves) in the one-wave
 * kernel's place unless the chunk size is 512 bytes or less, and calls and prepared passes for which it pays split the
 * one-wave kernel's work evenly over the resident waves, chunks cut between
 * them (hv_leaf_launch_for says which; a forced choice runs the kernel it
 * names).  Monitor scans (hv_monitor.h) take the
 * one-wave kernel under the automatic choice.  The same choice applies to
 * SHA-384's two leaf kernels.  The digests do not depend on it.
 * Errors: HV_ERR_INVALID_ARG for another value. */
hv_status hv_set_leaf_kernel(int choice);

/* The leaf kernel a hash call over n_leaves leaves would run on the current
 * device under this thread's choice: *kernel = 1 (one-wave, or three-group as
 * above), 2 (two-wave, 64 chunks per workgroup) or 3 (two-wave, 128).  Monitor
 * scans take the one-wave kernel under the automatic choice.
 * Errors: HV_ERR_INVALID_ARG for a NULL kernel. */
hv_status hv_leaf_kernel_for(uint64_t n_leaves, int* kernel);

/* The leaf launch of a hash call or a prepared pass (hv_plan.h) over n_leaves
 * leaves of n_msgs messages under this thread's choice, on a device of `cus`
 * compute units, or on the current device when cus = 0, for tests and
 * measurements: *launch = 1 (one-wave), 2 (two-wave, 64 chunks per workgroup),
 * 3 (two-wave, 128), 4 (three-group) or 5 (one-wave, the work split evenly over
 * the resident waves; with a workspace of hv_hash_workspace_bytes).
 * Host only; with cus > 0 no device is needed.
 * Errors: HV_ERR_INVALID_ARG for an unknown algorithm or a NULL launch;
 * HV_ERR_HIP if cus = 0 and the current device cannot be queried. */
hv_status hv_leaf_launch_for(hv_alg alg, uint32_t n_msgs, uint64_t n_leaves, uint64_t chunk_bytes, uint32_t cus,
                             int* launch);

/* How often a wave looks for the chunk states of the wave it shares chunks with
 * before it hashes those chunks from their first block itself (launch 5 of
 * hv_leaf_launch_for), per calling thread: at least `polls` times (16384 is
 * the default), or never with 0.  For tests; the digests do not depend on it. */
hv_status hv_set_handover_polls(uint32_t polls);

/* The launches hv_merkle_reduce_alg makes for these segments on a device of
 * `cus` compute units, or on the current device when cus = 0 (RFC 6962
 * section 2.1's tree, built level by level; Algorithm 1's
 * "construct Merkle tree from leaf_hashes using GPU"), for tests and
 * measurements: *launches (at most 8), and per launch k < *launches
 * kind[k] = 1 for a group launch (8 entries of a segment reduced by three
 * levels in registers) or 2 for a tile launch (512 entries, nine levels),
 * units[k] = the groups or tiles it reduces, and one_lane[k] = the groups a
 * group launch gives one lane each; its remaining units[k] - one_lane[k]
 * groups, the launch's last ones, take four lanes each (0 for a tile
 * launch).  kind, units and one_lane: host arrays of at least 8 entries.
 * Host only; no kernel runs, and with cus > 0 no device is needed.
 * Errors: HV_ERR_INVALID_ARG as hv_merkle_reduce_alg's checks of alg and
 * seg_offsets, or for a NULL output; HV_ERR_HIP if cus = 0 and the current
 * device cannot be queried. */
hv_status hv_merkle_launches(hv_alg alg, const uint64_t* seg_offsets, uint32_t n_seg, uint32_t cus, int* launches,
                             int* kind, uint64_t* units, uint64_t* one_lane);

#ifdef __cplusplus
}
#endif

#endif /* HV_INSPECT_H */
