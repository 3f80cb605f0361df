/*
 * pqkm_tuning.h -- tuning and measurement hooks of libpqkm.so.
 *
 * Not part of the method and not needed to use it: the entry points of pqkm.h choose their kernels and launch
 * shapes themselves.  These hooks exist so that tests can force every compiled kernel and so that a benchmark can
 * time the scan kernel on the stream it runs on.
 *
 * The options are PROCESS-WIDE.  Every pqkm.h entry point reads them once, when it is called, and works from that
 * copy, so a change made while a call runs does not affect it; but two callers in one process cannot hold
 * different settings, and setting an option while another thread is between two calls that belong together
 * (say pqkm_assign then pqkm_update) changes the second.  None of the options changes pqkm_workspace_bytes.
 */
#ifndef PQKM_TUNING_H
#define PQKM_TUNING_H

#include "pqkm.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * pqkm_set_option: integer knobs, by name (host string).  Unknown
 * name or out-of-range value -> PQKM_ERR_SHAPE.  Names:
 *   "assign_kernel"      0 = choose automatically (default), 1 = force the scans
 *                        that need no tile images (one lane per center; one per code where neither M nor the
 *                        alignment has a tiled scan and the centers are few),
 *                        2 = force the LDS-tiled scan (M in {4, 8, 16, 32} only)
 *   "scan_variant"       0 = default scan of the LDS-tiled assignment (for M = 4: codes regrouped for
 *                        conflict-free LDS reads when K >= 128 and N exceeds one round of 2048-code
 *                        workgroups, else the subspace-skewed scan in a launch shape chosen by N),
 *                        1..99 = one specific compiled scan and launch shape (for tuning sweeps;
 *                        e.g. 34 = the skewed M = 4 scan without regrouping, 70 = the regrouped one;
 *                        60 = the scan through lower bounds, M = 4 and 8, 59 the same for M = 16 and 32,
 *                        65 = the best of the plain M = 4 scans, 20 = the scan on the matrix cores, M = 8, 16 and 32, in front of
 *                        the default ones, unless these regroup the codes or the images leave it no room: M = 8 with
 *                        fewer than 17 centers)
 *   "hist_kernel"        0 = choose automatically (default; inside pqkm_fit / pqkm_fit_until with M = 4 this
 *                        includes counting from records the scan files by cluster group), 1 = force one global atomic
 *                        per code and subspace, 2 = force the LDS-privatised histogram over cluster
 *                        groups (falls back when K needs more than 255 groups), 3 = force the
 *                        histogram over code indices sorted by cluster
 *   "launch_codes_log2"  the scan is issued in launches of 2^value codes (default 26)
 *   "scan_rounds_per_launch"  the large scans (two-lane M = 4 scan, regrouped M = 8 scan, sliding-window
 *                        scan) issue the workgroups of such a launch in kernel launches of `value`
 *                        rounds (one workgroup per compute unit) each, so that the workgroups start
 *                        in step and share the tile images through the L2 (default 1); 0 = one
 *                        kernel launch for all of them
 *   "profile"            bit 0 (value 1) = bracket every scan-kernel launch with a pair of HIP
 *                        events on the caller's stream; bit 1 (value 2) = bracket every whole
 *                        assignment step (tile images, regrouping of the codes where it is
 *                        due, scan launches) the same way; 3 = both; 0 = off (default).
 *                        Events are created on first use and reused; this is the one place
 *                        the library creates HIP objects.
 *
 * pqkm_profile_read / pqkm_profile_read_steps: wait for the recorded stop events, return the
 * summed elapsed time of the bracketed scan kernels / assignment steps in milliseconds and
 * their number, and reset that record.  A pair of events brackets the scan kernels of one
 * stretch of codes (one launch, or one per round of workgroups, back to back on the stream);
 * `launches` counts the kernels, so total_ms / launches is the average duration of a scan
 * kernel, the short gaps between consecutive launches included.  They block the host.
 *   total_ms, launches / steps   host pointers, out
 */
pqkm_status pqkm_set_option(const char *name, int32_t value);
pqkm_status pqkm_profile_read(double *total_ms, int64_t *launches);
pqkm_status pqkm_profile_read_steps(double *total_ms, int64_t *steps);

/*
 * pqkm_scan_plan: what the assignment step of iteration `iteration` (from 0) of pqkm_fit runs for N codes against K
 * centers under the options as they are, for aligned operands: host arithmetic, nothing is launched (without a GPU the
 * answer is that for 256 compute units).
 * Where the scan on the matrix cores is tried first the answer is what it leaves the codes to.
 *   out   host, int64[6]: 0 the scan: 0 = one lane per center, 1 = LDS-tiled, 2 = through lower bounds;
 *         1 its number ("scan_variant"); 2 codes per stretch; 3 lanes per slot that it regroups the codes for (0 = it does
 *         not); 4 whether it takes over the regrouped copy of the iteration before; 5 where a code's first bound comes
 *         from (0 = the first tile, 1 = the assignment before, 2 = the key before, 3 = centers that share a pair of subcodes;
 *         M = 4 and 8 only)
 */
pqkm_status pqkm_scan_plan(int64_t N, int32_t M, int32_t K, int32_t iteration, int64_t out[6]);

/*
 * pqkm_dot_scan: the scan on the matrix cores in front of an LDS-tiled scan or one through lower bounds, for aligned operands, a call that
 * asks for no distances, and the options as they are.  Where pqkm_scan_plan names one lane per center, pqkm_call_plan says whether that is
 * preceded by it.
 *   workspace   that of a pqkm_assign or pqkm_fit call for these N, M, K, or NULL; with it the call waits for the device
 *   out         host, int32[2]: 0 whether the scan is tried first; 1 with a workspace, and where it is tried: whether the last
 *               assignment step there was left to the scans behind it, which pqkm_scan_plan names (1) or not (0), else -1
 */
pqkm_status pqkm_dot_scan(int64_t N, int32_t M, int32_t K, const void *workspace, int32_t out[2]);

/*
 * pqkm_call_plan: what one pqkm_assign and one pqkm_update call by themselves run under the options as they are: host arithmetic, as
 * pqkm_scan_plan.
 *   flags  1: codes, 2: centers that are not 4-byte aligned; 4: distances are asked for
 *   out    host, int64[8]: 0 the scan as pqkm_scan_plan names it; 1 its number, or for one lane per center whether the table rows go
 *          through the caches (0) or LDS (1), or a lane takes a code (2); 2 dimensions up to which the scan on the matrix cores is tried first
 *          (0 = it is not); 3 codes per block and 4 parts of the centers (one lane per center); 5 how the update counts: 1 = per group
 *          of clusters, 2 = per group of subspaces, 3 = from indices sorted by cluster, 4 = global atomics, or in the vote, 5 = a workgroup
 *          per cluster, 6 = per sixteen clusters; 6 its slices of the codes; 7 whether the vote takes a workgroup per cluster
 */
pqkm_status pqkm_call_plan(int64_t N, int32_t M, int32_t K, int32_t flags, int64_t out[8]);

#ifdef __cplusplus
}
#endif
#endif /* PQKM_TUNING_H */
