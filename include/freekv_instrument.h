/* freekv_instrument.h -- measurement and test hooks of libfreekv.so.
 *
 * Not part of the retrieval-decode interface (freekv.h): these entry points exist for the benchmark
 * (kernel timers on the launch stream, the cost of an empty launch) and for tests of what the blocks of a
 * launch exchange.  A serving loop needs none of them.
 * Same conventions as freekv.h: 0 or a negative FKV_E* code, nothing throws.
 */
#ifndef FREEKV_INSTRUMENT_H
#define FREEKV_INSTRUMENT_H

#include "freekv.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Time the split attention kernel (the dominant HBM reader of the step) with a
 * HIP event pair around each of the next max_launches launches, on the stream it
 * is launched on.  max_launches = 0 switches the timers off.  Blocking. */
int fkv_profile_enable(fkv_ctx* ctx, int32_t max_launches);
/* Sum of the recorded durations (ms) and their number; resets the timers.  Blocking. */
int fkv_profile_read(fkv_ctx* ctx, double* total_ms, int32_t* launches);

/* Launch the attention kernel `reps` times for every layer in turn (ACTIVE selection, the
 * state is not changed), back to back on `stream` between one HIP event pair, and return
 * the elapsed time and the number of launches.  q_dev: layer l's queries at
 * q_dev + l * q_layer_stride bytes.  out_dev: [batch, n_q, d] fp32 scratch output.  Blocking. */
int fkv_profile_attn(fkv_ctx* ctx, const void* q_dev, size_t q_layer_stride, float* out_dev, int32_t reps,
                     void* stream, double* total_ms, int32_t* launches);

/* The same for the page-weight scan and the selection (Sec. 3.2) as fkv_page_select launches them: `reps`
 * times for every layer in turn between one HIP event pair; `launches` receives the kernel launches made
 * (one per call when the selection rides in the scoring launch, more otherwise).  The layers' PENDING id
 * buffers are overwritten; no other state changes.  Blocking. */
int fkv_profile_select(fkv_ctx* ctx, const void* q_dev, size_t q_layer_stride, int32_t reps, void* stream,
                       double* total_ms, int32_t* launches);

/* The cost of a launch as such: `reps` launches, back to back on `stream` between one HIP event
 * pair, of a kernel with the grid, block size and dynamic LDS of `layer`'s last one-launch
 * layer-step whose blocks return at once.  FKV_ESTATE if that step took several launches.
 * grid / lds_bytes (may be NULL) receive the shape.  Blocking. */
int fkv_profile_launch_floor(fkv_ctx* ctx, int32_t layer, int32_t reps, void* stream, double* total_ms,
                             int32_t* grid, int32_t* lds_bytes);

/* Test hook for what fkv_health reports: while on, the attention waves of a corrected head wait for picked page ids
 * under a tag that no launch has had yet, and go on waiting for them after their block has made the selection itself.
 * Every kernel still ends; the head's output rows are NaN and fkv_health returns FKV_ETIMEOUT.  Host-side switch, no
 * GPU work. */
int fkv_test_lose_selection(fkv_ctx* ctx, int32_t on);

/* Test hook for what a block does when another block of its launch keeps it waiting too long: waits of these kinds
 * run out.  Nothing is lost by that -- the waiting block makes what it waits for itself -- so ids and
 * outputs stay what they are, bit for bit.  Host-side switch, no GPU work. */
#define FKV_WAIT_WEIGHTS  1  /* the selection's, for page weights from scoring blocks of the launch       */
#define FKV_WAIT_MAXIMA   2  /* a slice's, for the other slices' maxima                                   */
#define FKV_WAIT_SUMS     4  /*                ... softmax sums                                           */
#define FKV_WAIT_KEYS     8  /* the last slice's, for the other slices' keys                              */
#define FKV_WAIT_SPLITS  16  /* attention's, for the sums of a head's other blocks                        */
#define FKV_WAIT_IDS     32  /* attention's of a corrected head, for the page ids picked in the launch    */
#define FKV_WAIT_ALL     63
int fkv_test_impatience(fkv_ctx* ctx, int32_t kinds);

/* How often, since the last call, a block of the layer's launches made by itself what it else gets from other blocks of its launch:
 * a wait ran out (or was made to: above), or the weights of a head were not finite.  Counted per selecting block and per wave of
 * attention.  Results do not depend on it, but such a launch takes milliseconds; 0 in a program whose launches find room.
 * at_home (may be NULL): whether the layer's last one-launch layer-step had each head's blocks on one XCD.  Blocking. */
int fkv_test_by_itself(fkv_ctx* ctx, int32_t layer, int32_t* count, int32_t* at_home);

/* Test hook for the numbers that tell one launch's exchanged values from another's (31 bits, one per launch): the
 * context's next launch gets the number after `last`.  Host-side, no GPU work. */
int fkv_test_launch_number(fkv_ctx* ctx, int32_t last);

/* While on, kernels record 100 MHz phase timestamps of head 0 (read with FKV_DBG_TSTAMP).  Of the 64 words these are
 * written, by a block of the head each (by the last one to come there, where several do); the others keep what they held:
 *    0  the first scoring block begins               1  its weights are out
 *    2  a selecting block has its weights             5  the keys of all that may be chosen are there
 *    8  the page ids are out
 *   16  attention's first block begins               17  its first wave's pages are done
 *   18  its waves are combined                       21  the head's output is out, or left to be made alone */
int fkv_instrument_timestamps(fkv_ctx* ctx, int32_t on);

#ifdef __cplusplus
}
#endif
#endif /* FREEKV_INSTRUMENT_H */
