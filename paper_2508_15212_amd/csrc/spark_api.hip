// C ABI of the library (see include/spark.h): argument checks on the host, buffer sizing,
// kernel launches on the caller's stream.  Nothing here allocates or synchronises.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "../../include/spark.h"
#include "../../include/spark_bench.h"
#include "spark_kernels.h"
#include "spark_layout.h"

namespace {

bool desc_ok(const spark_desc *d, spark_status *why)
{
    *why = SPARK_ERR_INVALID_ARG;
    if (!d) return false;
    if (d->batch < 1 || d->n_q_heads < 1 || d->n_kv_heads < 1) return false;
    // token and tile indices are 32-bit in the kernels (a tile's last row index must still fit), block counts too
    if (d->total_tokens < 0 || d->total_tokens > ((int64_t)1 << 31) - 256) return false;
    if (d->batch > (1 << 18)) return false;
    if (d->keep < 1 || d->keep > d->head_dim) return false;
    if (d->n_q_heads % d->n_kv_heads) return false;
    if (d->n_splits < -1 || d->n_splits > 4096) return false;
    if (d->max_seqlen < 0) return false;
    if (d->keep_v < 0 || d->keep_v > d->head_dim) return false;
    if (d->tail_capacity < 0 || d->tail_capacity > (1 << 20)) return false;
    if (d->stats != 0 && d->stats != 1) return false;
    *why = SPARK_ERR_UNSUPPORTED;
    if (d->head_dim != SPARK_D) return false;
    const int G = d->n_q_heads / d->n_kv_heads;
    if (!(G == 1 || G == 2 || G == 4 || G == 8 || G == 16)) return false;
    if (d->pack_dtype != SPARK_PACK_BF16 && d->pack_dtype != SPARK_PACK_INT8) return false;
    if (d->out_dtype != SPARK_OUT_BF16 && d->out_dtype != SPARK_OUT_F32) return false;
    *why = SPARK_OK;
    return true;
}

SparkLayout layout_of(const spark_desc *d)
{
    return spark_make_layout(d->keep, d->pack_dtype == SPARK_PACK_INT8, d->batch, d->n_kv_heads, d->total_tokens,
                             d->stats);
}

SparkLayout topp_layout_of(const spark_desc *d)
{
    return spark_make_topp_layout(d->batch, d->n_kv_heads, d->total_tokens);
}

SparkLayout values_layout_of(const spark_desc *d)
{
    return spark_make_values_layout(d->keep_v, d->n_kv_heads, d->total_tokens);
}

bool strides_ok(int64_t tok, int64_t head)
{
    return tok >= SPARK_D && head >= SPARK_D && tok % 8 == 0 && head % 8 == 0;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// How the decode grid cuts the batch into blocks.  The decode kernel keeps two 4-wave blocks resident per
// compute unit (256 CUs), so about 512 blocks stream the cache in a single round with no tail; a block should
// still see at least 4 tiles (one per wavefront).  Sequences are cut into chunks of chunk_tiles tiles, so long
// sequences of a ragged batch get more blocks than short ones; n_splits > 0 (or a batch too large for the
// in-kernel numbering of the chunks) asks for the same number of chunks for every sequence instead.
spark::DecodePlan plan_of(const spark_desc *d, bool allow_balanced = true)
{
    spark::DecodePlan p;
    p.tail_slots = d->tail_capacity > 0 ? (d->tail_capacity + 255) / 256 : 1;
    const int64_t tiles = (d->total_tokens + SPARK_TILE_TOKENS - 1) / SPARK_TILE_TOKENS;
    int64_t chunk = (tiles * d->n_kv_heads + 511) / 512;
    // With many (batch, KV head) pairs the blocks of an evenly cut batch would already exceed what is resident
    // at once, and every further round costs a block's fixed start-up and merge latency: then only sequences
    // well above the average length are cut.
    if ((int64_t)d->batch * d->n_kv_heads >= 256) chunk *= 2;
    if (chunk < 4) chunk = 4;     // one tile per wavefront: below that a block's start-up outweighs its work
    p.chunk_tiles = (int)chunk;
    p.fixed_splits = 0;
    if (d->n_splits > 0) {
        p.fixed_splits = d->n_splits;
    } else if (d->batch > 256) {
        const int64_t avg_tiles = (d->total_tokens / d->batch + SPARK_TILE_TOKENS - 1) / SPARK_TILE_TOKENS;
        int64_t n = (avg_tiles + chunk - 1) / chunk;
        p.fixed_splits = (int)(n < 1 ? 1 : (n > 4096 ? 4096 : n));
    }
    if (p.fixed_splits > 0)
        p.nchunk_max = d->batch * p.fixed_splits;
    else   // a sequence of len tokens spans at most len / 64 + 2 tiles, and rounding up costs at most one chunk
        p.nchunk_max = (int)((tiles + 2 * (int64_t)d->batch) / chunk + d->batch + 1);
    // Rounding up every sequence's share can put a few blocks more on the chip than it holds at once, and they start when
    // the others are done.  The kernel, which knows the lengths, then takes longer chunks.  (Few sequences only: their
    // table is one register a lane; 256 pairs and more are cut less finely, see above.)  Llama heads, T = 26, without / with
    // the limit (us): 8 sequences of 20000 to 45000 tokens 133 / 110, 16 of 2000 to 9000 56 / 48 (T = 64: 76 / 66), 28 of
    // 500 to 3000 33 / 29, 10 of 8000 49 / 40; 4 of 12001 to 18777 with packed values, which are bound by each block's own
    // work, 35.1 / 34.9.
    p.chunk_limit = 0;
    if (p.fixed_splits == 0 && d->batch <= 64 && (int64_t)d->batch * d->n_kv_heads < 256 &&
        (int64_t)p.nchunk_max * d->n_kv_heads > 512)
        p.chunk_limit = 512 / d->n_kv_heads;
    // Many sequences, each too short to be cut: one block per (sequence, KV head) would make the launch last as
    // long as its longest sequence.  Then (or on request, n_splits = -1) the (sequence, tile) items of a KV head
    // are dealt out evenly to as many wavefronts as are resident at once, 2048 over all heads.  The mode holds
    // the batch's sequence table in registers (at most 256 sequences) and numbers items in 32 bits.
    p.warm_waves = 0;
    p.short_call = 0;
    p.counter_stride = spark::counter_stride((int64_t)d->batch * d->n_kv_heads);
    // (neighbours share a tile at most, so sequences cut by length span tiles + batch - 1 of them, in no more than
    //  (tiles - 1) / chunk + batch chunks: one fewer than nchunk_max)
    p.chunk_ids = p.fixed_splits > 0 ? p.nchunk_max : p.nchunk_max - 1;
    const int64_t pairs = (int64_t)d->batch * d->n_kv_heads;
    // (a batch that its caller knows to be near-uniform is balanced with one block per sequence already)
    const bool even = d->max_seqlen > 0 && (int64_t)d->max_seqlen * d->batch * 8 <= d->total_tokens * 9;
    const bool wanted = d->n_splits == -1 || (d->n_splits == 0 && d->batch >= 32 && pairs >= 256 && !even);
    if (allow_balanced && wanted && d->batch <= 256 && d->n_q_heads / d->n_kv_heads <= 8) {
        const int per_head = 512 / d->n_kv_heads > 0 ? 512 / d->n_kv_heads : 1;     // blocks of four wavefronts
        const int64_t nw = 4 * (int64_t)per_head;
        // (unasked, only where a wavefront gets two tiles or more: with less the partials cost more than the
        //  balance gains - 32 sequences of 100 to 1000 tokens: 19.0 against 20.6 us)
        const bool enough = d->n_splits == -1 || tiles >= 2 * nw;
        if (enough && (tiles + 2 * (int64_t)d->batch + 1) * nw < ((int64_t)1 << 32)) {
            p.warm_waves = (int)nw;
            const int ids = (int)nw + 2 * d->batch - 1;
            if (p.chunk_ids < ids) p.chunk_ids = ids;
        }
    }
    return p;
}

// A block of four wavefronts for every tile, four lanes a row (plan.short_call = 2, spark_decode_short.h): short calls whose
// workspace has room for a partial per tile.  Four tiles in a block keep to a quarter of the compute units, each bound by the
// table gathers in its LDS; a tile a block spreads them, for four times the partials, which the last block of a pair merges.  So it
// gains where blocks of four wavefronts would take four tiles each, and
//   - until the merge of ONE sequence's partials is the longer: the more query heads, the fewer tiles.  The lengths are on the device:
//     the longest of several sequences is taken to have four fifths of the batch's tiles, or what max_seqlen says.
//     (5000 and three times 100 tokens, G = 4, T = 64: 1.42; one KV head, 40000 and 21 times 200 tokens: 58.9 instead of 22.2 us.  One of
//     several with more than four fifths, at the limit: up to 1.09.)
//   - from sequences of 200 or 240 tokens on average: up to four tiles are one block of the other form, and nothing is merged there (with
//     appended rows both merge).  Sequences of 128 / 192 / 256 tokens, G = 2, up to 512 blocks: T = 26 1.30 / 1.23 / 0.99, T = 64 1.11 / 1.06 / 0.91,
//     T = 28 1.02 / 0.99 / 0.83; long rows of any length gain there as well: T = 48 0.91 / 0.88 / 0.77;
//   - while the blocks are resident at once, 512 of them (rows of any length, which gain more, up to 704; eight query heads, which
//     need more LDS, 256).  T = 64, 256 to 512 / 512 to 640 blocks: G = 1 0.96 / 1.02, G = 2 0.96 / 1.05, G = 4 0.97 / 1.10.
// Rows of 25 (bf16), 26 and 38 kept channels are the same either way with one query head (int8 codes of 26 lose 6 %) and lose with eight
// (38: from 16 tiles, up to 8 % at 20); this form has the smaller error against 64 bits.  Eight query heads with rows of any length are taken by blocks of
// sixteen wavefronts.  Time against blocks of four tiles (graphs of 40 to 160 calls; the larger of the
// ratios with caches in the L2 and with ones that rotate through 400 MB), tiles of the batch, sequences (s: the first has 80 % of them):
//   KV heads     G = 1, T = 26 / 32 / 38 / 48 / 64    G = 2                              G = 4                              G = 8, T = 26 / 38 / 64
//   8   3 in 1   1.42 / 1.07 / 1.35 / 0.97 / 1.19   1.37 / 1.06 / 1.31 / 0.95 / 1.13   1.26 / 1.01 / 1.21 / 0.93 / 1.08   1.32 / 1.28 / 1.13
//   8   8 in 4   1.40 / 1.07 / 1.33 / 0.97 / 1.18   1.35 / 1.04 / 1.29 / 0.93 / 1.13   1.25 / 0.99 / 1.19 / 0.91 / 1.06   1.30 / 1.26 / 1.12
//   8   8 in 1   1.03 / 0.85 / 1.04 / 0.78 / 0.93   0.99 / 0.81 / 0.97 / 0.75 / 0.87   1.01 / 0.82 / 0.95 / 0.77 / 0.88   1.00 / 0.99 / 0.89
//   8  20 in 1   1.01 / 0.85 / 1.03 / 0.78 / 0.92   1.01 / 0.84 / 0.98 / 0.78 / 0.89   1.04 / 0.88 / 1.01 / 0.81 / 0.93   1.08 / 1.08 / 0.98
//   8  32 in 1   1.04 / 0.86 / 1.05 / 0.80 / 0.94   1.04 / 0.86 / 1.01 / 0.80 / 0.93   1.11 / 0.93 / 1.08 / 0.87 / 0.98   1.20 / 1.20 / 1.09
//   8  40 in 1   1.07 / 0.91 / 1.10 / 0.85 / 1.00   1.08 / 0.92 / 1.07 / 0.87 / 1.00   1.25 / 1.07 / 1.22 / 1.00 / 1.12   1.38 / 1.36 / 1.24
//   8  64 in 1   1.09 / 1.00 / 1.10 / 1.01 / 1.01   1.14 / 0.97 / 1.13 / 0.91 / 1.05   1.39 / 1.18 / 1.33 / 1.00 / 1.24   1.54 / 1.51 / 1.39
//   8  32 in 4   1.08 / 0.91 / 1.11 / 0.86 / 1.02   1.06 / 0.87 / 1.04 / 0.83 / 0.97   1.07 / 0.90 / 1.04 / 0.84 / 0.97   1.09 / 1.09 / 0.99
//   8  64 in 8   1.15 / 0.97 / 1.15 / 1.00 / 1.07   1.14 / 0.97 / 1.14 / 0.95 / 1.08   1.18 / 1.02 / 1.17 / 1.00 / 1.11   1.26 / 1.27 / 1.19
//   8  64 in 4s  1.09 / 0.92 / 1.11 / 1.00 / 1.03   1.11 / 0.94 / 1.10 / 0.93 / 1.07   1.29 / 1.10 / 1.24 / 1.00 / 1.20   1.42 / 1.40 / 1.31
//   16 32 in 4   1.13 / 0.96 / 1.14 / 1.00 / 1.04   1.10 / 0.94 / 1.09 / 0.90 / 1.07   1.16 / 0.99 / 1.12 / 1.00 / 1.09   1.22 / 1.20 / 1.14
//   2  32 in 1   1.02 / 0.85 / 1.05 / 0.80 / 0.95   1.02 / 0.83 / 1.00 / 0.79 / 0.91   1.08 / 0.89 / 1.05 / 0.83 / 0.97   1.15 / 1.12 / 1.02
//   2  64 in 1   1.00 / 0.82 / 0.99 / 0.79 / 0.93   1.03 / 0.84 / 1.00 / 0.80 / 0.94   1.23 / 1.03 / 1.20 / 0.96 / 1.10   1.37 / 1.35 / 1.25
//   2  90 in 1   1.01 / 0.84 / 1.01 / 0.79 / 0.95   1.15 / 0.95 / 1.13 / 0.90 / 1.06   1.38 / 1.16 / 1.33 / 1.08 / 1.24   1.58 / 1.55 / 1.43
//   2  64 in 8   0.97 / 0.81 / 0.99 / 0.76 / 0.91   0.95 / 0.77 / 0.92 / 0.73 / 0.86   0.95 / 0.80 / 0.93 / 0.74 / 0.86   0.97 / 0.97 / 0.88
// Of 3564 such measurements that the rule takes without max_seqlen (1, 2, 4, 8 and 16 KV heads, T = 20 to 64) the worst is 1.07 (G = 1, T = 38,
// from memory; 0.96 from the L2) and the mean 0.88, with max_seqlen the same; with 200 appended rows 0.91 and 1.07, int8 codes 0.90 and 1.05.
bool fine_plan(const spark_desc *d, spark::DecodePlan &p, bool with_tail)
{
    const int G = d->n_q_heads / d->n_kv_heads;
    const int64_t tiles = (d->total_tokens + SPARK_TILE_TOKENS - 1) / SPARK_TILE_TOKENS;
    if (tiles == 0 || d->batch > 64 || d->n_splits != 0 || p.warm_waves > 0 || G > 8) return false;
    const SparkLayout L = layout_of(d);
    const int64_t cache_blocks = (tiles + d->batch) * d->n_kv_heads;
    int longest, blocks, tokens;         // tiles of one sequence, blocks of the cache at most; tokens a sequence at least
    if (!spark::row_length_instantiated(L)) {
        longest = G == 1 ? 96 : (G == 2 ? 64 : (G == 4 ? 36 : 0));
        blocks = G <= 2 ? 704 : 512;
        tokens = cache_blocks > 256 ? 240 : (L.T < 40 ? 200 : 0);
    } else if (L.T == 64) {
        longest = G == 1 ? 96 : (G == 2 ? 64 : (G == 4 ? 32 : 24));
        blocks = G <= 4 ? 512 : 256;
        tokens = G == 1 ? 240 : 200;
    } else {
        longest = G == 1 ? (L.int8 && L.T == 26 ? 0 : 32) : (G == 2 ? (L.T == 38 ? 48 : 32) : (G == 4 ? 20 : (L.T == 38 ? 20 : 0)));
        blocks = 256;
        tokens = 240;
    }
    if (longest == 0 || (!with_tail && d->total_tokens < tokens * (int64_t)d->batch)) return false;
    const int tail_slots = !with_tail ? 0 : (d->tail_capacity > 0 ? (d->tail_capacity + spark::kFineTailRows - 1) / spark::kFineTailRows : 1);
    int64_t most = d->batch > 1 ? (4 * tiles + 4) / 5 : tiles;
    if (d->max_seqlen > 0) most = std::min(tiles, ((int64_t)d->max_seqlen + SPARK_TILE_TOKENS - 1) / SPARK_TILE_TOKENS + 1);      // (it can begin and end in a tile)
    if (most + tail_slots > longest || cache_blocks > blocks) return false;
    if ((tiles + d->batch * (1 + (int64_t)tail_slots)) * d->n_kv_heads > 848) return false;
    if (spark::decode_form(p, L, d->n_q_heads, true, with_tail ? p.tail_slots : 0).short_call != 0) return false;
    p.short_call = 2;
    p.chunk_tiles = 1;
    p.chunk_limit = 0;
    p.nchunk_max = p.chunk_ids = (int)(tiles + d->batch - 1);      // (see plan_of)
    p.tail_slots = tail_slots;
    return true;
}

// chunks an average-length sequence is cut into; 0 for the balanced cut (what spark_decode_splits reports)
int pick_splits(const spark_desc *d)
{
    spark::DecodePlan p = plan_of(d);
    fine_plan(d, p, false);
    p = spark::decode_form(p, layout_of(d), d->n_q_heads, true, 0);
    if (p.warm_waves > 0) return 0;
    if (p.fixed_splits > 0) return p.fixed_splits;
    // (as the kernel numbers them, for a batch of sequences of that length)
    const int64_t avg_tiles = (d->total_tokens / d->batch + SPARK_TILE_TOKENS - 1) / SPARK_TILE_TOKENS;
    for (int64_t chunk = p.chunk_tiles;; chunk += 1 + chunk / 16) {
        const int64_t n = avg_tiles > chunk ? (avg_tiles + chunk - 1) / chunk : 1;
        if (p.chunk_limit == 0 || n * d->batch <= p.chunk_limit) return (int)n;
    }
}

// partial slots in the workspace: one per (chunk, q head), then the appended rows' (per (batch, q head): one per 256 rows of
// capacity, at least one, so a workspace serves calls with and without appended rows; with a block per tile one per 64 rows, or none)
size_t partial_slots(const spark_desc *d, const spark::DecodePlan &p)
{
    return (size_t)p.chunk_ids * d->n_q_heads + (size_t)d->batch * d->n_q_heads * p.tail_slots;
}

// The arrival counters sit at the START of the workspace, so their position depends on batch and n_kv_heads
// only and not on how a call cuts its sequences into blocks; the partial states follow at a 256-byte boundary.
size_t counter_bytes(const spark_desc *d, int stride)
{
    return (((size_t)d->batch * d->n_kv_heads * stride * sizeof(uint32_t)) + 255) & ~(size_t)255;
}

size_t bytes_of(const spark_desc *d, const spark::DecodePlan &p)
{
    return partial_slots(d, p) * (SPARK_D + 2) * sizeof(float) + counter_bytes(d, p.counter_stride);
}

// What a call asks for: never less than it took with the counters side by side and slots for a chunk more.
size_t workspace_bytes_of(const spark_desc *d, const spark::DecodePlan &p)
{
    spark::DecodePlan dense = p;
    dense.counter_stride = 1;
    dense.chunk_ids += p.fixed_splits > 0 && p.warm_waves == 0 ? 0 : 1;
    return bytes_of(d, p) > bytes_of(d, dense) ? bytes_of(d, p) : bytes_of(d, dense);
}

// What a call gets by with: its counters side by side.  (A call that has no more clears the places of counters further apart behind
// itself, which its partial states lie on: the next call finds zeros there.)
size_t least_workspace_of(const spark_desc *d, spark::DecodePlan p)
{
    p.counter_stride = 1;
    return workspace_bytes_of(d, p);
}

}  // namespace

extern "C" {

const char *spark_status_string(spark_status s)
{
    switch (s) {
        case SPARK_OK: return "ok";
        case SPARK_ERR_INVALID_ARG: return "invalid argument";
        case SPARK_ERR_UNSUPPORTED: return "unsupported configuration";
        case SPARK_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case SPARK_ERR_HIP: return "HIP runtime error";
        case SPARK_ERR_MISMATCH: return "packed cache does not match the description";
    }
    return "unknown status";
}

size_t spark_packed_bytes(const spark_desc *desc)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return 0;
    return (size_t)layout_of(desc).total_bytes;
}

size_t spark_prune_workspace(const spark_desc *desc)
{
    (void)desc;
    return 0;
}

int32_t spark_decode_splits(const spark_desc *desc)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return 0;
    return pick_splits(desc);
}

size_t spark_decode_workspace(const spark_desc *desc)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return 0;
    // (what the calls need; short ones are faster with more)
    size_t bytes = workspace_bytes_of(desc, plan_of(desc));
    for (const bool with_tail : {false, true}) {
        spark::DecodePlan fine = plan_of(desc);
        if (fine_plan(desc, fine, with_tail) && workspace_bytes_of(desc, fine) > bytes) bytes = workspace_bytes_of(desc, fine);
    }
    return bytes;
}

spark_status spark_decode_workspace_init(const spark_desc *desc, void *workspace, size_t workspace_bytes,
                                         void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!workspace || !aligned(workspace, 16)) return SPARK_ERR_INVALID_ARG;
    if (workspace_bytes < least_workspace_of(desc, plan_of(desc))) return SPARK_ERR_WORKSPACE_TOO_SMALL;
    // (a workspace has two slots of 520 bytes a pair at least, counters take 128 bytes a pair at most)
    uint32_t *counters = static_cast<uint32_t *>(workspace);
    const hipError_t e = spark::launch_zero_counters(counters, (int)(counter_bytes(desc, plan_of(desc).counter_stride) / sizeof(uint32_t)),
                                                     static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

spark_status spark_prune(const spark_desc *desc, const void *k_bf16, const void *qwin_bf16,
                         const int32_t *cu_seqlens, void *packed_out, void *workspace, size_t workspace_bytes,
                         void *hip_stream)
{
    (void)workspace;
    (void)workspace_bytes;
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!k_bf16 || !qwin_bf16 || !cu_seqlens || !packed_out) return SPARK_ERR_INVALID_ARG;
    if (desc->window < 1) return SPARK_ERR_INVALID_ARG;
    if (!strides_ok(desc->k_token_stride, desc->k_head_stride)) return SPARK_ERR_INVALID_ARG;
    // the prune kernel addresses the 64 rows of a tile with 32-bit byte offsets from the tile's first row
    if (desc->k_token_stride > ((int64_t)1 << 24)) return SPARK_ERR_UNSUPPORTED;
    if (!aligned(k_bf16, 16) || !aligned(qwin_bf16, 2) || !aligned(packed_out, 256)) return SPARK_ERR_INVALID_ARG;
    const SparkLayout L = layout_of(desc);
    const hipError_t e = spark::launch_prune(static_cast<const uint16_t *>(k_bf16), desc->k_token_stride,
                                             desc->k_head_stride, static_cast<const uint16_t *>(qwin_bf16),
                                             cu_seqlens, static_cast<uint8_t *>(packed_out), L, desc->n_q_heads,
                                             desc->window, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

size_t spark_packed_values_bytes(const spark_desc *desc)
{
    spark_status why;
    if (!desc_ok(desc, &why) || desc->keep_v < 1) return 0;
    return (size_t)values_layout_of(desc).total_bytes;
}

spark_status spark_prune_values(const spark_desc *desc, const void *v_bf16, void *packed_v_out, void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (desc->keep_v < 1 || !v_bf16 || !packed_v_out) return SPARK_ERR_INVALID_ARG;
    if (!strides_ok(desc->v_token_stride, desc->v_head_stride)) return SPARK_ERR_INVALID_ARG;
    if (desc->v_token_stride > ((int64_t)1 << 24)) return SPARK_ERR_UNSUPPORTED;
    if (!aligned(v_bf16, 16) || !aligned(packed_v_out, 256)) return SPARK_ERR_INVALID_ARG;
    const hipError_t e = spark::launch_prune_values(static_cast<const uint16_t *>(v_bf16), desc->v_token_stride,
                                                    desc->v_head_stride, static_cast<uint8_t *>(packed_v_out),
                                                    values_layout_of(desc), static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

spark_status spark_unpack_values(const spark_desc *desc, const void *packed_v, uint32_t *mask_out, void *vals_out,
                                 void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (desc->keep_v < 1 || !packed_v) return SPARK_ERR_INVALID_ARG;
    const hipError_t e = spark::launch_unpack(static_cast<const uint8_t *>(packed_v), values_layout_of(desc), mask_out,
                                              vals_out, nullptr, nullptr, nullptr, nullptr, nullptr, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

namespace {

spark_status decode_common(const spark_desc *desc, const void *q_bf16, const void *packed, const void *v_bf16,
                           const void *packed_v, const int32_t *cu_seqlens, void *out, void *workspace,
                           size_t workspace_bytes, void *hip_stream, const void *tail_k = nullptr,
                           const void *tail_v = nullptr, const int32_t *tail_len = nullptr, int rec = 0,
                           uint64_t seed = 0, bool topp = false, const spark::DecodePlan *given = nullptr)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!q_bf16 || !packed || !cu_seqlens || !out || !workspace) return SPARK_ERR_INVALID_ARG;
    if (packed_v) {
        if (desc->keep_v < 1) return SPARK_ERR_INVALID_ARG;
        if (!aligned(packed_v, 256)) return SPARK_ERR_INVALID_ARG;
    } else {
        if (!v_bf16) return SPARK_ERR_INVALID_ARG;
        if (!strides_ok(desc->v_token_stride, desc->v_head_stride)) return SPARK_ERR_INVALID_ARG;
        if (!aligned(v_bf16, 16)) return SPARK_ERR_INVALID_ARG;
    }
    if (!aligned(packed, 256) || !aligned(workspace, 16) || !aligned(q_bf16, 2) || !aligned(out, 8))
        return SPARK_ERR_INVALID_ARG;
    if (tail_k) {
        if (!tail_v || !tail_len || desc->tail_capacity < 1) return SPARK_ERR_INVALID_ARG;
        if (!aligned(tail_k, 16) || !aligned(tail_v, 16) || !aligned(tail_len, 4)) return SPARK_ERR_INVALID_ARG;
    }
    spark::DecodePlan plan = given ? *given : plan_of(desc);
    size_t clear = 0;                    // bytes at the start to clear behind the call
    if (!given && workspace_bytes < workspace_bytes_of(desc, plan)) {
        clear = counter_bytes(desc, plan.counter_stride);
        plan.counter_stride = 1;
    }
    if (workspace_bytes < workspace_bytes_of(desc, plan)) return SPARK_ERR_WORKSPACE_TOO_SMALL;
    if (!packed_v && rec == 0 && !topp) {
        spark::DecodePlan fine = plan;
        if (fine_plan(desc, fine, tail_k != nullptr) && workspace_bytes >= workspace_bytes_of(desc, fine)) plan = fine;
    }
    const size_t slots = partial_slots(desc, plan);
    const SparkLayout L = topp ? topp_layout_of(desc) : layout_of(desc);
    SparkLayout Lv = L;
    if (packed_v) Lv = values_layout_of(desc);
    uint32_t *counters = static_cast<uint32_t *>(workspace);
    float *part_acc = reinterpret_cast<float *>(static_cast<uint8_t *>(workspace) + counter_bytes(desc, plan.counter_stride));
    float *part_ml = part_acc + slots * SPARK_D;
    const float scale = desc->softmax_scale != 0.0f ? desc->softmax_scale : 1.0f / sqrtf((float)SPARK_D);
    const hipError_t e = spark::launch_decode_attn(
        static_cast<const uint16_t *>(q_bf16), static_cast<const uint8_t *>(packed),
        static_cast<const uint16_t *>(v_bf16), desc->v_token_stride, desc->v_head_stride,
        static_cast<const uint8_t *>(packed_v), packed_v ? &Lv : nullptr, cu_seqlens, part_acc, part_ml, counters,
        desc->n_q_heads, plan, scale, L, out, desc->out_dtype == SPARK_OUT_F32,
        static_cast<const uint16_t *>(tail_k), static_cast<const uint16_t *>(tail_v), tail_len,
        desc->tail_capacity, rec, seed, static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return SPARK_ERR_HIP;
    if (clear > 0 && spark::launch_zero_counters(counters, (int)(clear / sizeof(uint32_t)), static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return SPARK_ERR_HIP;
    return SPARK_OK;
}

}  // namespace

spark_status spark_decode_attn(const spark_desc *desc, const void *q_bf16, const void *packed, const void *v_bf16,
                               const int32_t *cu_seqlens, void *out, void *workspace, size_t workspace_bytes,
                               void *hip_stream)
{
    if (!v_bf16) return SPARK_ERR_INVALID_ARG;
    return decode_common(desc, q_bf16, packed, v_bf16, nullptr, cu_seqlens, out, workspace, workspace_bytes,
                         hip_stream);
}

spark_status spark_decode_attn_sampled(const spark_desc *desc, const void *q_bf16, const void *packed,
                                       const void *v_bf16, const int32_t *cu_seqlens, void *out, void *workspace,
                                       size_t workspace_bytes, int32_t recovery, uint64_t seed, void *hip_stream)
{
    if (!v_bf16) return SPARK_ERR_INVALID_ARG;
    if (recovery != SPARK_RECOVER_GAUSSIAN && recovery != SPARK_RECOVER_EXPONENTIAL) return SPARK_ERR_INVALID_ARG;
    if (desc && !desc->stats) return SPARK_ERR_INVALID_ARG;     // the cache must carry the all-channel statistics
    return decode_common(desc, q_bf16, packed, v_bf16, nullptr, cu_seqlens, out, workspace, workspace_bytes,
                         hip_stream, nullptr, nullptr, nullptr, recovery, seed);
}

spark_status spark_unpack_stats(const spark_desc *desc, const void *packed, float *mu_all_out, float *sigma_out,
                                void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!packed || !desc->stats) return SPARK_ERR_INVALID_ARG;
    const hipError_t e = spark::launch_unpack(static_cast<const uint8_t *>(packed), layout_of(desc), nullptr, nullptr,
                                              nullptr, nullptr, nullptr, mu_all_out, sigma_out,
                                              static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

spark_status spark_decode_attn_tail(const spark_desc *desc, const void *q_bf16, const void *packed, const void *v_bf16,
                                    const int32_t *cu_seqlens, const void *tail_k_bf16, const void *tail_v_bf16,
                                    const int32_t *tail_len, void *out, void *workspace, size_t workspace_bytes,
                                    void *hip_stream)
{
    if (!v_bf16 || !tail_k_bf16) return SPARK_ERR_INVALID_ARG;
    return decode_common(desc, q_bf16, packed, v_bf16, nullptr, cu_seqlens, out, workspace, workspace_bytes,
                         hip_stream, tail_k_bf16, tail_v_bf16, tail_len);
}

spark_status spark_decode_attn_values(const spark_desc *desc, const void *q_bf16, const void *packed,
                                      const void *packed_v, const int32_t *cu_seqlens, void *out, void *workspace,
                                      size_t workspace_bytes, void *hip_stream)
{
    if (!packed_v) return SPARK_ERR_INVALID_ARG;
    return decode_common(desc, q_bf16, packed, nullptr, packed_v, cu_seqlens, out, workspace, workspace_bytes,
                         hip_stream);
}

spark_status spark_decode_attn_values_tail(const spark_desc *desc, const void *q_bf16, const void *packed,
                                           const void *packed_v, const int32_t *cu_seqlens,
                                           const void *tail_k_bf16, const void *tail_v_bf16,
                                           const int32_t *tail_len, void *out, void *workspace,
                                           size_t workspace_bytes, void *hip_stream)
{
    if (!packed_v || !tail_k_bf16) return SPARK_ERR_INVALID_ARG;
    return decode_common(desc, q_bf16, packed, nullptr, packed_v, cu_seqlens, out, workspace, workspace_bytes,
                         hip_stream, tail_k_bf16, tail_v_bf16, tail_len);
}

spark_status spark_unpack(const spark_desc *desc, const void *packed, uint32_t *mask_out, void *vals_out,
                          float *mu_out, float *scale_out, float *a_out, void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!packed) return SPARK_ERR_INVALID_ARG;
    const SparkLayout L = layout_of(desc);
    const hipError_t e = spark::launch_unpack(static_cast<const uint8_t *>(packed), L, mask_out, vals_out, mu_out,
                                              scale_out, a_out, nullptr, nullptr, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

spark_status spark_check_packed(const spark_desc *desc, const void *packed, int32_t is_value_cache, void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!packed || !aligned(packed, 256)) return SPARK_ERR_INVALID_ARG;
    if (is_value_cache && desc->keep_v < 1) return SPARK_ERR_INVALID_ARG;
    uint32_t hdr[16];
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (hipMemcpyAsync(hdr, packed, sizeof hdr, hipMemcpyDeviceToHost, st) != hipSuccess) return SPARK_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return SPARK_ERR_HIP;
    const SparkLayout L = is_value_cache ? values_layout_of(desc) : layout_of(desc);
    // header words: magic, T, int8, batch, Hkv, total_tokens, words per row, value-cache flag, statistics flag
    const uint32_t want[9] = {SPARK_MAGIC, (uint32_t)L.T, (uint32_t)L.int8, (uint32_t)L.batch, (uint32_t)L.n_kv_heads,
                              (uint32_t)L.total_tokens, (uint32_t)L.ndw, is_value_cache ? 1u : 0u, (uint32_t)L.stats};
    for (int i = 0; i < 9; ++i)
        if (hdr[i] != want[i]) return SPARK_ERR_MISMATCH;
    return SPARK_OK;
}

// ---------------------------------------------------------------- the top-p variant

size_t spark_packed_topp_bytes(const spark_desc *desc)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return 0;
    return (size_t)topp_layout_of(desc).total_bytes;
}

spark_status spark_prune_topp(const spark_desc *desc, const void *k_bf16, const void *qwin_bf16,
                              const int32_t *cu_seqlens, int32_t p_basis_points, void *packed_out, void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!k_bf16 || !qwin_bf16 || !cu_seqlens || !packed_out) return SPARK_ERR_INVALID_ARG;
    if (desc->window < 1 || p_basis_points < 1 || p_basis_points > 10000) return SPARK_ERR_INVALID_ARG;
    if (!strides_ok(desc->k_token_stride, desc->k_head_stride)) return SPARK_ERR_INVALID_ARG;
    if (desc->pack_dtype != SPARK_PACK_BF16 || desc->stats) return SPARK_ERR_UNSUPPORTED;
    if (!aligned(k_bf16, 16) || !aligned(qwin_bf16, 2) || !aligned(packed_out, 256)) return SPARK_ERR_INVALID_ARG;
    const SparkLayout L = topp_layout_of(desc);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipError_t e = spark::launch_window_stat(static_cast<const uint16_t *>(qwin_bf16), static_cast<uint8_t *>(packed_out), L,
                                             desc->n_q_heads, desc->window, st);
    if (e == hipSuccess)
        e = spark::launch_prune_topp(static_cast<const uint16_t *>(k_bf16), desc->k_token_stride, desc->k_head_stride,
                                     cu_seqlens, static_cast<uint8_t *>(packed_out), L, p_basis_points, st);
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

spark_status spark_decode_attn_topp(const spark_desc *desc, const void *q_bf16, const void *packed, const void *v_bf16,
                                    const int32_t *cu_seqlens, void *out, void *workspace, size_t workspace_bytes,
                                    void *hip_stream)
{
    if (!v_bf16) return SPARK_ERR_INVALID_ARG;
    if (desc && (desc->pack_dtype != SPARK_PACK_BF16 || desc->stats)) return SPARK_ERR_UNSUPPORTED;
    return decode_common(desc, q_bf16, packed, v_bf16, nullptr, cu_seqlens, out, workspace, workspace_bytes, hip_stream,
                         nullptr, nullptr, nullptr, 0, 0, true);
}

int32_t spark_call_form(const spark_desc *desc, int32_t call)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return 0;
    if (call == SPARK_CALL_PRUNE) return spark::prune_launches(layout_of(desc), desc->n_q_heads, desc->window);
    const bool tiles = call == SPARK_CALL_DECODE_TILES || call == SPARK_CALL_DECODE_TAIL_TILES;
    if (call == SPARK_CALL_DECODE || call == SPARK_CALL_DECODE_TAIL || tiles) {
        const bool with_tail = call == SPARK_CALL_DECODE_TAIL || call == SPARK_CALL_DECODE_TAIL_TILES;
        spark::DecodePlan cut = plan_of(desc);
        fine_plan(desc, cut, with_tail);
        const spark::DecodePlan p = spark::decode_form(cut, layout_of(desc), desc->n_q_heads, true, with_tail ? cut.tail_slots : 0);
        if (tiles) return p.warm_waves > 0 || p.fixed_splits > 0 ? 0 : p.chunk_tiles;
        return p.warm_waves > 0 ? 3 : (p.short_call == 1 ? 2 : 1);      // (a block per tile: blocks of four wavefronts)
    }
    if (call == SPARK_CALL_PRUNE_TOPP) return spark::topp_prune_launches(topp_layout_of(desc));
    return 0;
}

spark_status spark_unpack_topp(const spark_desc *desc, const void *packed, uint32_t *mask_out, int32_t *count_out,
                               void *vals_out, float *mu_out, float *a_out, void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!packed) return SPARK_ERR_INVALID_ARG;
    const hipError_t e = spark::launch_unpack_topp(static_cast<const uint8_t *>(packed), topp_layout_of(desc), mask_out,
                                                   count_out, static_cast<uint16_t *>(vals_out), mu_out, a_out,
                                                   static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SPARK_OK : SPARK_ERR_HIP;
}

// ---------------------------------------------------------------- decode without a caller-provided workspace

// Split partials and arrival counters of spark_decode_attn_static: one array per GPU, held until the process
// ends.  In host code this name is only a handle for hipGetSymbolAddress; kernels get the looked-up address.
static __device__ __align__(256) unsigned char scratch[SPARK_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];      // device address of `scratch` on each GPU, looked up on first use
std::mutex g_scratch_mutex;

// address of this GPU's copy of the array (the current device's), or nullptr after a runtime error
void *scratch_address()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

spark_status spark_decode_attn_static(const spark_desc *desc, const void *q_bf16, const void *packed,
                                      const void *v_bf16, const int32_t *cu_seqlens, void *out, void *hip_stream)
{
    spark_status why;
    if (!desc_ok(desc, &why)) return why;
    if (!v_bf16) return SPARK_ERR_INVALID_ARG;
    // the balanced cut of a ragged batch needs more partial slots than the chunked one: where only the chunked
    // one fits the array, that one is used
    spark::DecodePlan plan = plan_of(desc);
    if (workspace_bytes_of(desc, plan) > (size_t)SPARK_STATIC_WORKSPACE_BYTES) plan = plan_of(desc, false);
    if (workspace_bytes_of(desc, plan) > (size_t)SPARK_STATIC_WORKSPACE_BYTES) plan.counter_stride = 1;
    if (workspace_bytes_of(desc, plan) > (size_t)SPARK_STATIC_WORKSPACE_BYTES) return SPARK_ERR_WORKSPACE_TOO_SMALL;
    void *ws = scratch_address();
    if (!ws) return SPARK_ERR_HIP;
    // the array keeps whatever the last call on this GPU left: the counters must start at zero (a small fill
    // kernel, not a memset node, so the call can be captured into a graph); partial states are written before
    // they are read
    if (spark::launch_zero_counters(static_cast<uint32_t *>(ws), (int)(counter_bytes(desc, plan.counter_stride) / sizeof(uint32_t)),
                                    static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return SPARK_ERR_HIP;
    return decode_common(desc, q_bf16, packed, v_bf16, nullptr, cu_seqlens, out, ws, SPARK_STATIC_WORKSPACE_BYTES,
                         hip_stream, nullptr, nullptr, nullptr, 0, 0, false, &plan);
}

}  // extern "C"
