/*
 * spark_bench.h -- measurement aids that ship in the same library as the SparK hot path
 * (include/spark.h) but are no part of the method.  bench.py and the profiler runs use them;
 * nothing in the method's entry points calls them.
 */
#ifndef SPARK_BENCH_H
#define SPARK_BENCH_H

#include "spark.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Reads `bytes` (a multiple of 16) from the device buffer `src` once, with 16-byte non-temporal
 * loads from n_blocks blocks of 256 threads, and discards them.  Its time is the streaming-read
 * ceiling the decode kernel is compared with, and its known size calibrates the HBM byte counters
 * of a profiler run.  `sink` is 4 writable device bytes.  Enqueued on `hip_stream`; no
 * synchronisation.  SPARK_ERR_INVALID_ARG for NULL / misaligned pointers, bytes < 16 or n_blocks < 1.
 */
spark_status spark_probe_read(const void *src, size_t bytes, void *sink, int32_t n_blocks,
                              void *hip_stream);

/*
 * Per-block timeline of the decode kernel.  After this call every decode launch of the process whose grid
 * fits (64 bytes per block) lets thread 0 of each block file eight 64-bit words into `device_buffer`:
 *   0 wall clock (100 MHz) at entry          1 at the start of streaming      2 at its end (wavefront 0)
 *   3 when its partial state is stored       4 at exit (after the merge, if it merged)
 *   5 tiles it streamed                      6 XCC id << 32 | HW_ID           7 1 if it merged a pair
 * (in the balanced cut of a ragged batch the wavefronts of a block work on their own: the words are wavefront
 * 0's, and word 5 is 1 << 32 | its tiles).
 * The caller owns the buffer, clears it, reads it back after synchronising, and calls again with NULL to
 * switch the aid off (the buffer must stay valid until then).  Process-wide and not thread safe; the
 * method's results do not depend on it.  SPARK_ERR_INVALID_ARG for a misaligned buffer or bytes < 64.
 */
spark_status spark_decode_timeline(void *device_buffer, size_t bytes);

/*
 * Which of its forms a call with this description takes (for tests and timings of the forms; launches nothing):
 *   SPARK_CALL_PRUNE        spark_prune:  1: the window statistic in the pruning launch   2: in a launch of its own (which a
 *                           window that is only 2-byte aligned takes always)
 *   SPARK_CALL_PRUNE_TOPP   1: selection and writing in one launch   3: in three
 *   SPARK_CALL_DECODE       spark_decode_attn:  1: chunks, blocks of four wavefronts (of four tiles or more, or, in short calls
 *                           whose workspace has room, of one)   2: chunks, blocks of sixteen   3: the balanced cut
 *   SPARK_CALL_DECODE_TAIL  spark_decode_attn_tail, the same
 *   SPARK_CALL_DECODE_TILES, SPARK_CALL_DECODE_TAIL_TILES  of the same two calls with the whole workspace, the tiles of a block where
 *                           sequences are cut by their length (more where that would make too many blocks): 1 is a block per
 *                           tile, four or more the other two forms; 0 with a given number of splits and in the balanced cut
 * 0 for an invalid description, another call, or a call that launches nothing.
 */
#define SPARK_CALL_PRUNE 0
#define SPARK_CALL_PRUNE_TOPP 1
#define SPARK_CALL_DECODE 2
#define SPARK_CALL_DECODE_TAIL 3
#define SPARK_CALL_DECODE_TILES 4
#define SPARK_CALL_DECODE_TAIL_TILES 5
int32_t spark_call_form(const spark_desc *desc, int32_t call);

#ifdef __cplusplus
}
#endif
#endif /* SPARK_BENCH_H */
