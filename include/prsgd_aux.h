/*
 * prsgd_aux.h -- measurement and test aids exported by libprsgd beside the method's own calls
 * (prsgd.h).  Nothing here is a step of Parallel Restarted SGD.
 */
#ifndef PRSGD_AUX_H
#define PRSGD_AUX_H

#include <stddef.h>
#include <stdint.h>

#include "prsgd.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * A plain device-to-device copy kernel of `bytes` bytes (a multiple of 16; both pointers device,
 * 16-byte aligned) whose traffic is known exactly.  The benchmark uses it to calibrate the
 * fetch/write hardware counters that the restart-average (eq. 2) and local-update (eq. 3)
 * kernels are compared against.  PRSGD_EINVAL on a null or misaligned pointer.
 */
int prsgd_copy_bytes(void* dst_dev, const void* src_dev, size_t bytes, void* hip_stream);

/*
 * The output tile that a forward or backward-data product of n_workers minibatches of `rows` rows and
 * a layer of `cols` columns is cut into: out[0] tile rows, out[1] tile columns, out[2] bytes of LDS a
 * workgroup takes.  Host only; tests use it to see which kernels a shape reaches.  PRSGD_EINVAL on
 * a size below 1, an unknown gemm_dtype or a null `out`.
 */
int prsgd_product_tile(int32_t rows, int32_t cols, int32_t n_workers, int32_t gemm_dtype, int32_t* out);

/*
 * Which launches of a configuration mark their weight traffic (ROWS: the drawn rows) non-temporal: a sum of the constants
 * below.  Host only, for tests.  PRSGD_EINVAL on an invalid configuration.
 */
enum { PRSGD_STREAM_STEPS = 1, PRSGD_STREAM_STEP_MEAN = 2, PRSGD_STREAM_MEAN = 4, PRSGD_STREAM_AVERAGE = 8,
       PRSGD_STREAM_ROWS = 16 };
int prsgd_streamed_uses(const prsgd_config* cfg);

/*
 * What prsgd_init_static leaves a configuration of the scratch that is no part of the method: PRSGD_SCRATCH_RUNS all of
 * it, PRSGD_SCRATCH_EPOCHS without what keeps restarts inside a launch, PRSGD_SCRATCH_LAYERS without what the one-launch
 * epoch kernel exchanges.  Host only, for tests.  PRSGD_EINVAL on an invalid configuration and on one that does not fit.
 */
enum { PRSGD_SCRATCH_LAYERS = 0, PRSGD_SCRATCH_EPOCHS = 1, PRSGD_SCRATCH_RUNS = 2 };
int prsgd_static_scratch(const prsgd_config* cfg);

/*
 * Launches whose workgroups wait for each other, of contexts on n_streams streams of one device (n_workers[k] teams of
 * team[k] workgroups on stream k; least squares: teams of one): PRSGD_WAIT_ALONE for a single stream,
 * PRSGD_WAIT_TOGETHER if all of them fit the device at once, XCD by XCD, PRSGD_WAIT_CROWDED if not (then they
 * follow each other by stream events, and restarts are launches of their own).  Host only, for tests.  PRSGD_EINVAL on a
 * null array, no stream or fewer than eight compute units.
 */
enum { PRSGD_WAIT_ALONE = 0, PRSGD_WAIT_TOGETHER = 1, PRSGD_WAIT_CROWDED = 2 };
int prsgd_waiting_regime(const int32_t* n_workers, const int32_t* team, int32_t n_streams, int32_t compute_units);

/*
 * out[0]: launches of this context that had restarts inside; out[1]: how often its stream was made to wait for a launch
 * of another stream.  PRSGD_EINVAL on a null pointer.
 */
int prsgd_waiting_launches(const prsgd_ctx* ctx, int64_t* out);

/*
 * Number of polls after which a workgroup of the one-launch epoch kernel stops waiting for its
 * team (see prsgd_status in prsgd.h); the default is 2^22.  Tests set a tiny value to drive the
 * give-up path from the host while every kernel still runs to its end.
 */
int prsgd_set_epoch_wait_limit(prsgd_ctx* ctx, uint32_t polls);

/*
 * on = 1 (default): on MLPs with bf16 operands the backward kernel of the first layer also runs the
 * first forward product of the next local iteration on the weights it writes (the minibatch of
 * iteration t + 1 is drawn during iteration t), so W_1 crosses HBM once per iteration.  on = 0: two
 * separate launches.  Which layers are taken is a rule on their size.  The results of layers of whole tiles (32, 64 or 128
 * minibatch rows, d_0 a multiple of 128 from 256 on, d_1 one of 64, and of 128 where d_0 exceeds 512) are identical bit for bit;
 * those of the other layers (d_0 from 512 on, up to 128 rows, d_1 from 512 on or padded to a multiple of 64) up to the order in
 * which the bias gradients are summed in fp32.  Tests compare the two.
 */
int prsgd_set_first_layer_fusion(prsgd_ctx* ctx, int32_t on);

/*
 * on = 1 (default): prsgd_run takes the iteration that completes an epoch and the restart after it
 * as one pass (see prsgd_run in prsgd.h).  on = 0: local iteration, then the restart kernel; equal
 * up to fp32 rounding.  Tests compare the two.
 */
int prsgd_set_restart_fusion(prsgd_ctx* ctx, int32_t on);

#ifdef __cplusplus
}
#endif
#endif /* PRSGD_AUX_H */
