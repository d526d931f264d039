/*
 * dbsp_diag.h -- diagnostics that ship with libdbsp but are not part of the method's boundary
 * (dbsp.h): measurement helpers for the benchmark.  Same conventions as dbsp.h.
 */
#ifndef DBSP_DIAG_H
#define DBSP_DIAG_H

#include <stdint.h>

#include "dbsp.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * dbsp_mfma_probe -- the chip's sustained dense bf16 MFMA rate, measured on the spot (the
 * roofline's published peak assumes 2.4 GHz, the sustained rate shows what clock the chip holds).
 * Runs a kernel of back-to-back v_mfma_f32_32x32x16_bf16 on pseudo-random operands (eight waves per
 * compute unit; the rate a chip sustains depends on how many bits flip) four times, about 10 ms each,
 * on `stream`, synchronises and reports the last run.  tflops (required): achieved TFLOP/s; clock_ghz (may be
 * NULL): shader clock during the run.  Allocates and frees a small device buffer.
 * Errors: DBSP_EINVAL, DBSP_EHIP.
 */
int dbsp_mfma_probe(double* tflops, double* clock_ghz, void* stream);

/*
 * dbsp_plan_run_order -- what the workgroups of a plan's launches run (also of a host-only plan's).  partition_of:
 * int32 [P] or NULL, the partition that workgroup b has (b, but where DBSP_MODE_BALANCED made the placement).  items: int32,
 * as many as DBSP_PART_ITEMS has, or NULL: the workgroups' items one workgroup behind the other, in the order in which
 * they run.  local: int32 or NULL, 1 if the launches' waits count on KV blocks being found in the L2 (at d = 128 with items of
 * 128 queries; else 0 or 1 without effect).  staged: int32 or NULL, 1 if one of the plan's launches has read it where it was staged, without a fetch, else 0.
 * Errors: DBSP_EINVAL, DBSP_ENOMEM.
 */
int dbsp_plan_run_order(const dbsp_plan* plan, int32_t* partition_of, int32_t* items, int32_t* local, int32_t* staged);

#ifdef __cplusplus
}
#endif
#endif /* DBSP_DIAG_H */
