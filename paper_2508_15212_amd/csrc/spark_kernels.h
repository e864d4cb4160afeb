// Internal: launch functions implemented next to their kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spark_layout.h"

namespace spark {

// Immediate of s_waitcnt on gfx9-family parts: vmcnt in bits [3:0] and [15:14] (vector memory loads AND stores
// of this wavefront still outstanding), expcnt in bits [6:4], lgkmcnt in bits [11:8] (LDS, scalar memory).  A
// field left at its maximum does not wait.  This one waits for vmcnt == 0 only: every global load has returned
// and every global store of the wavefront has been acknowledged by the memory system.
constexpr int kWaitVmcnt0 = (0 << 0) | (0 << 14) | (7 << 4) | (15 << 8);      // = 0x0F70

struct DecodeParams;

// Words between the arrival counters of two (batch, KV head) pairs.  Device-scope atomics on one 64-byte block are served one
// after the other, 11.5 ns each, so the counters are spread over 2 KB, at most 128 bytes apart.  Blocks that only count in, all at
// once, on eight counters side by side / 128 bytes apart (us; 2.4 without counting): 512 blocks 7.2 / 2.4, 1024 13.0 / 3.1; on 64 counters
// side by side / 32 bytes apart: 512 4.1 / 2.3, 1024 6.2 / 2.6.  Decode, T = 26, eight heads, G = 1 / 4: 8192 tokens 12.1 / 14.0 ->
// 10.1 / 12.0, 16384 17.9 / 19.5 -> 15.6 / 17.8, 4 x 4096 14.6 / 16.6 -> 13.1 / 15.2; 2 x 8000 with packed values 18.5 -> 16.4.
inline int counter_stride(int64_t pairs)
{
    int stride = 32;
    while (stride > 1 && pairs * stride > 512) stride /= 2;
    return stride;
}

constexpr int kNoPriority = 1 << 28;   // (more than four times the tiles of a cache: every block stays at the lowest level)
constexpr int kFineTailRows = 64;      // appended rows per block of DecodePlan::short_call = 2

// Whether the decode kernels have an instantiation for the key rows' length (rows that carry the all-channel statistics are longer)
inline bool row_length_instantiated(const SparkLayout &L)
{
    return !L.stats && (L.T == 26 || L.T == 38 || L.T == 64 || (L.T == 25 && !L.int8));
}

// How the decode grid cuts sequences into blocks (chosen on the host from the description alone).
struct DecodePlan {
    int fixed_splits;   // > 0: every sequence is cut into this many chunks
    int chunk_tiles;    // else: a sequence spanning ntile tiles gets max(1, ceil(ntile / chunk_tiles)) chunks
    int chunk_limit;    // > 0: chunks are made longer until the batch has at most this many (up to 64 sequences, and not fewer)
    int nchunk_max;     // upper bound on the number of chunks in the batch (grid = nchunk_max * Hkv + tail blocks)
    int tail_slots;     // partial slots reserved per (batch, q head) for appended rows (none in a block-per-tile plan without them)
    int warm_waves;     // > 0: the balanced mode may be used, with this many wavefronts per KV head; decode_form
                        // falls back to the chunked cut for the kernel variants that have no balanced form
    int counter_stride; // words between the arrival counters of two pairs
    int short_call;     // blocks of 1: sixteen 2: four wavefronts of spark_decode_short.h; 1 is chosen by decode_form, 2 is the
                        // plan of a call whose workspace has room for a partial per tile
    int chunk_ids;      // chunk ids the workspace has partial slots for: all of a cut by length, and of the balanced
                        // mode, warm_waves + 2 * batch - 1; the appended rows' slots follow at chunk_ids * Hq
};

// measurement aid: later decode launches of this process file eight 64-bit words per block into `device_words`
// (room for `blocks` blocks; launches with more blocks file nothing); NULL switches it off
void set_decode_timeline(unsigned long long *device_words, size_t blocks);

int prune_launches(const SparkLayout &L, int Hq, int W);     // how many launches launch_prune takes (with a 4-byte aligned window)
hipError_t launch_prune(const uint16_t *k, int64_t k_tok_stride, int64_t k_head_stride, const uint16_t *qwin,
                        const int32_t *cu, uint8_t *packed, const SparkLayout &L, int Hq, int W, hipStream_t st);

// value-cache channel pruning: per (token, KV head) the L.T channels of largest |v| (L from spark_make_values_layout)
hipError_t launch_prune_values(const uint16_t *v, int64_t v_tok_stride, int64_t v_head_stride, uint8_t *packed,
                               const SparkLayout &L, hipStream_t st);

hipError_t launch_unpack(const uint8_t *packed, const SparkLayout &L, uint32_t *mask_out, void *vals_out,
                         float *mu_out, float *scale_out, float *a_out, float *mu_all_out, float *sigma_out,
                         hipStream_t st);

// The form that a decode call takes: which kernel, and the chunks it is launched with.  plain: dense values, degenerate recovery,
// a fixed-count cache; ntail: blocks of appended rows per (batch, KV head).
DecodePlan decode_form(DecodePlan cut, const SparkLayout &L, int Hq, bool plain, int ntail);

// q [B,Hq,128] bf16; the caller splits the workspace into part_acc / part_ml / counters.
// Values are either dense (v, strides; packed_v = NULL) or a packed value cache (packed_v, Lv; v = NULL).
// Partial slots: cut.chunk_ids * Hq, then batch * Hq * cut.tail_slots; tail_k != NULL adds the appended rows
// [B, tail_cap, Hkv, 128].
hipError_t launch_decode_attn(const uint16_t *q, const uint8_t *packed, const uint16_t *v, int64_t v_tok_stride,
                              int64_t v_head_stride, const uint8_t *packed_v, const SparkLayout *Lv,
                              const int32_t *cu, float *part_acc, float *part_ml,
                              uint32_t *counters, int Hq, const DecodePlan &cut, float softmax_scale, const SparkLayout &L,
                              void *out, int out_f32, const uint16_t *tail_k, const uint16_t *tail_v,
                              const int32_t *tail_len, int tail_cap, int rec, uint64_t seed, hipStream_t st);

hipError_t launch_zero_counters(uint32_t *counters, int n_words, hipStream_t st);

// channel weights a, 1/a (and the key cache's header) alone; for a top-p cache also its directory, cleared
hipError_t launch_window_stat(const uint16_t *qwin, uint8_t *packed, const SparkLayout &L, int Hq, int W, hipStream_t st);

// top-p variant (L from spark_make_topp_layout; launch_window_stat must have run before, for every call anew)
hipError_t launch_prune_topp(const uint16_t *k, int64_t k_tok_stride, int64_t k_head_stride, const int32_t *cu,
                             uint8_t *packed, const SparkLayout &L, int p_bp, hipStream_t st);
int topp_prune_launches(const SparkLayout &L);     // how many launches launch_prune_topp takes
hipError_t launch_unpack_topp(const uint8_t *packed, const SparkLayout &L, uint32_t *mask_out, int32_t *count_out,
                              uint16_t *vals_out, float *mu_out, float *a_out, hipStream_t st);

}  // namespace spark
