/*
 * mtfm_hta_timing.h -- optional instrumentation of libmtfm_hta.so for benchmarks and profiling: HIP event pairs
 * recorded by the library around each kernel it enqueues.  Not part of the attention interface (mtfm_hta.h) and not
 * bound by its contract: mtfm_hta_timing_read() blocks on its events, and the state is process-wide.  Off unless
 * switched on; while off, the attention calls record nothing.
 */
#ifndef MTFM_HTA_TIMING_H
#define MTFM_HTA_TIMING_H

#include "mtfm_hta.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Per-kernel timing.  mtfm_hta_timing_enable(slots) creates `slots`
 * HIP event pairs per kernel kind (slots <= 0: destroy them and switch timing off, the default).  While
 * on, every call records an event pair on its stream around each kernel it enqueues, into a ring of
 * `slots` entries per kind.  mtfm_hta_timing_read() waits for the recorded events of one kind (this is
 * the only blocking call of the library), writes up to `capacity` durations in milliseconds to the HOST
 * array `ms`, oldest first, empties that ring and returns how many it wrote (or a negative status).
 * Process-wide state; not meant to be toggled while another thread is inside a call.
 */
enum { MTFM_HTA_KERNEL_FWD = 0,      /* forward attention kernel */
       MTFM_HTA_KERNEL_BWD_SELF = 1, /* dk/dv of the target tokens' own keys: no launch of its own any more (its blocks
                                        ride at the end of another grid), never recorded */
       MTFM_HTA_KERNEL_BWD_DQ = 2,   /* dq and the own keys (row-stationary pass; the whole backward of the fp32 path).  In a
                                        call of little work only the row statistics: such a call forms dq, dk and dv in one
                                        launch, which is the next kind */
       MTFM_HTA_KERNEL_BWD_DKDV = 3, /* dk, dv of the history and real-time keys (key-stationary pass, one launch or two); of
                                        a call of little work everything but the row statistics, of a call whose users have
                                        few query rows the whole backward pass where one kernel forms it */
       MTFM_HTA_N_KERNELS = 7        /* kinds 4..6 belong to mtfm_gln.h */ };
MTFM_HTA_API int mtfm_hta_timing_enable(int slots);
MTFM_HTA_API int mtfm_hta_timing_read(int kernel, float* ms, int capacity);

#ifdef __cplusplus
}
#endif
#endif /* MTFM_HTA_TIMING_H */
