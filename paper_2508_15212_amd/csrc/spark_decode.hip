// Host side of decode attention: parameter block, choice of the query-group instantiation, counter reset.
// The kernel template is in spark_decode_kernel.h; its instantiations are compiled in spark_decode_g*.hip.
#include "spark_decode_kernel.h"

namespace spark {

extern template hipError_t launch_g<1>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<2>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<4>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<8>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<16>(const DecodeParams &, int, hipStream_t);

// Whether a call gains by the blocks of sixteen wavefronts of spark_decode_short.h.  Such a block takes four tiles at a time, four
// lanes a row, all in one compute unit, whose LDS then bounds it; 256 of them, a pass, take 1024 tiles (over all KV heads).  It gains
//   - by the walk, with long rows and with eight query heads, whose walk by one lane has few gathers in flight (not where the
//     row length has an instantiation): up to a pass, or a quarter more;
//   - by the merge, where a (sequence, KV head) pair has many partials, half as many here, folded by sixteen wavefronts: that is
//     with many tiles a sequence.
// It loses where a second pass is begun for little.  Time against blocks of four wavefronts (outlier channels, jittered rows; KV
// heads, lengths, tiles a sequence, passes):
//                                            G = 1, T = 32 / 48 / 60   G = 2, 32 / 48 / 75   G = 4, 32 / 48 / 60   G = 8, 32 / 48 / 75   G = 8, 26 / 38 / 64
//   8 heads  1 x 4096              64   0.5    1.00 / 0.96 / 0.95        1.06 / 1.02 / 1.00    1.02 / 1.00 / 0.98    0.95 / 0.93 / 0.93    1.04 / 1.04 / 1.05
//            1 x 6500             102   0.8    0.95 / 0.92 / 0.90        0.99 / 0.97 / 0.95    0.97 / 0.96 / 0.96    0.91 / 0.91 / 0.90    0.99 / 1.00 / 1.00
//            1 x 10000            157   1.2    0.91 / 0.90 / 0.90        0.96 / 0.96 / 0.95    0.98 / 0.98 / 0.97    0.92 / 0.92 / 0.90    0.98 / 0.99 / 0.99
//            1 x 16384            256   2.0    0.97 / 0.97 / 0.99        0.97 / 1.00 / 1.05    1.00 / 1.02 / 1.04    0.90 / 0.92 / 0.95    0.93 / 0.95 / 1.02
//            2 x 6000 to 10000    125   2.0    1.04 / 1.03 / 1.05        1.03 / 1.07 / 1.11    1.04 / 1.07 / 1.08    0.94 / 0.97 / 1.00    0.98 / 1.00 / 1.09
//            4 x 700 to 3900       36   1.1    1.03 / 0.98 / 0.95        1.05 / 1.04 / 0.98    1.06 / 1.02 / 0.99    0.97 / 0.95 / 0.90    1.06 / 1.05 / 1.00
//            6 x 2000 to 3000      39   1.8    1.15 / 1.11 / 1.12        1.19 / 1.19 / 1.20    1.16 / 1.15 / 1.15    1.11 / 1.09 / 1.09    1.15 / 1.18 / 1.19
//            8 x 300 to 800         8   0.5    1.01 / 0.98 / 0.96        1.04 / 1.04 / 1.00    1.04 / 1.00 / 0.99    0.96 / 0.95 / 0.93    1.07 / 1.08 / 1.08
//   4 heads  1 x 32768            512   2.0    0.79 / 0.80 / 0.82        0.81 / 0.84 / 0.89    0.86 / 0.88 / 0.90    0.75 / 0.77 / 0.80    0.76 / 0.78 / 0.85
//   2 heads  8 x 3000 to 6000      70   1.1    0.94 / 0.86 / 0.90        0.97 / 0.96 / 0.93    0.96 / 0.95 / 0.94    0.91 / 0.89 / 0.86    0.97 / 0.97 / 0.95
//            1 x 65536           1024   2.0    0.57 / 0.58 / 0.59        0.63 / 0.65 / 0.68    0.70 / 0.72 / 0.75    0.59 / 0.61 / 0.64    0.60 / 0.62 / 0.66
// Long rows, 8 heads, four / sixteen (us): 1 x 1024: G = 4, T = 90 15.6 / 13.5, T = 127 17.1 / 14.3, G = 2, T = 127 15.2 / 13.7, G = 1,
// T = 70 11.2 / 10.5; 1 x 16384: G = 4, T = 90 24.8 / 26.0, G = 1, T = 70 21.0 / 21.2.
static bool short_call_pays(const SparkLayout &L, int G)
{
    const bool instantiated = row_length_instantiated(L), long_rows = L.T > (G == 2 ? 80 : 64);
    const int64_t pass = 256 * 4, tiles = L.n_tiles * L.n_kv_heads, per_sequence = L.n_tiles / L.batch;
    if (G <= 4 && instantiated) return false;
    if (G <= 4 && long_rows) return tiles <= pass;
    if (tiles > 2 * pass) return false;
    if (G == 8 && !instantiated) return tiles <= pass * 5 / 4 || per_sequence > 64;
    if (tiles < (G == 4 ? 288 : 512)) return false;
    if (tiles > pass * 3 / 2) return per_sequence >= (G == 1 || L.T <= 40 ? 256 : 512);
    if (per_sequence >= 96) return true;
    if (tiles > pass * 5 / 4) return false;
    if (tiles > pass && per_sequence > 64) return true;
    return (G == 1 && (L.T >= 44 || per_sequence >= 64)) || (G == 4 && L.T >= 44);
}

// The balanced mode and the blocks of sixteen wavefronts: dense values, degenerate recovery, rows of one length (`plain`),
// query groups up to 8 (else chunks by blocks of four).
// Short calls: all blocks are resident at once, one a compute unit.  Chunks get as much longer as that takes, where blocks of
// four wavefronts would have to do the same, or where that is half a pass (of four tiles a place) on average; with more (8 x 800 to
// 1500 tokens and appended rows, T = 32, 6.6 tiles a place) four / sixteen wavefronts a block took 14.6 / 16.1 us.
DecodePlan decode_form(DecodePlan plan, const SparkLayout &L, int Hq, bool plain, int ntail)
{
    const int G = Hq / L.n_kv_heads;
    if (plan.short_call == 2) return plan;
    if (!plain || G > 8) plan.warm_waves = 0;
    plan.short_call = 0;
    if (!plain || G > 8 || plan.warm_waves > 0 || !short_call_pays(L, G)) return plan;
    const int64_t room = 256 / L.n_kv_heads - (int64_t)L.batch * ntail;      // chunks there are places for
    if (plan.nchunk_max <= room) {
        plan.short_call = 1;
    } else if (plan.fixed_splits == 0 && L.batch <= 64 && room >= 2 * L.batch &&
               (plan.chunk_limit > 0 || L.n_tiles + 2 * L.batch <= 4 * room * 3 / 2)) {
        plan.short_call = 1;
        plan.chunk_limit = plan.nchunk_max = (int)room;
    }
    return plan;
}

// Whether the blocks of a call with appended rows set priorities (set_priority).  The appended rows' blocks come last in the grid.  With
// more blocks than the 512 that are resident at once they start as others end, which happens early without priorities and at the very
// end with them.  That costs more than priorities gain while a block has seven tiles or fewer.  Time with / without priorities against the
// same without either and with counters side by side, mean (largest) of 2 to 31 sequences of 300 to 16000 tokens, 64 to 1024 rows of room,
// G = 1 to 16, two to eight KV heads, T = 26 / 48 / 64, by tiles of a block:
//   5          1.017 / 1.006   1.012 / 1.003   1.020 / 1.006   (1.07 / 1.04)
//   7          1.010 / 1.003   1.012 / 0.999   1.006 / 1.005   (1.08 / 1.03)
//   8 and 9    1.011 / 1.004   1.003 / 1.003   0.987 / 1.000   (1.07 / 1.03)
//   10 to 12   0.995 / 1.005   0.988 / 1.005   0.959 / 1.002   (1.08 / 1.03)
//   13 to 16   1.021 / 1.008   0.999 / 1.002   0.979 / 1.004   (1.08 / 1.07)
//   17 to 39   1.002 / 1.003   0.981 / 1.002   0.975 / 1.000   (1.07 / 1.05)
// 12 of 500 to 3000 tokens, 256 rows, G = 4, T = 64 / 26: with 26.6 / 22.8 us, without 23.8 / 20.7; 8 of 1500 to 7000 tokens, T = 64: with
// 29.1, without 32.9.  Tried: the appended rows' blocks first in the grid (1.02 to 1.05 of last), the others' levels below theirs (no change).
static bool priorities_pay(int chunk_tiles, int64_t nblocks)
{
    return nblocks <= 544 || chunk_tiles >= 8;
}

// Zeroes the arrival counters of a fresh workspace.
__global__ void spark_zero_kernel(uint32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Timeline buffer of the measurement aid spark_decode_timeline (process-wide; NULL = off)
namespace {
unsigned long long *g_timeline = nullptr;
size_t g_timeline_blocks = 0;
}  // namespace

void set_decode_timeline(unsigned long long *device_words, size_t blocks)
{
    g_timeline = device_words;
    g_timeline_blocks = device_words ? blocks : 0;
}

hipError_t launch_decode_attn(const uint16_t *q, const uint8_t *packed, const uint16_t *v, int64_t v_tok_stride,
                              int64_t v_head_stride, const uint8_t *packed_v, const SparkLayout *Lv,
                              const int32_t *cu, float *part_acc, float *part_ml,
                              uint32_t *counters, int Hq, const DecodePlan &cut, float softmax_scale, const SparkLayout &L,
                              void *out, int out_f32, const uint16_t *tail_k, const uint16_t *tail_v,
                              const int32_t *tail_len, int tail_cap, int rec, uint64_t seed, hipStream_t st)
{
    DecodeParams P;
    P.q = q;
    P.packed = packed;
    P.v = v;
    P.packed_v = packed_v;
    P.Lv = Lv ? *Lv : L;
    P.v_tok_stride = v_tok_stride;
    P.v_head_stride = v_head_stride;
    P.cu = cu;
    P.part_acc = part_acc;
    P.part_ml = part_ml;
    P.counters = counters;
    P.out = out;
    P.out_f32 = out_f32;
    P.Hq = Hq;
    P.Hkv = L.n_kv_heads;
    const bool plain = !packed_v && rec == 0 && !L.topp;
    const DecodePlan plan = decode_form(cut, L, Hq, plain, tail_k ? cut.tail_slots : 0);
    P.fixed_splits = plan.fixed_splits;
    P.chunk_tiles = plan.chunk_tiles;
    P.nchunk_max = plan.nchunk_max;
    P.chunk_limit = plan.chunk_limit;
    P.short_call = plan.short_call;
    P.warm_waves = plan.warm_waves;
    P.counter_stride = plan.counter_stride;
    P.tail_slots = plan.tail_slots;
    P.ntail = tail_k ? plan.tail_slots : 0;
    P.tail_base = (int64_t)plan.chunk_ids * Hq;
    P.tail_k = tail_k;
    P.tail_v = tail_v;
    P.tail_len = tail_len;
    P.tail_cap = tail_cap;
    P.rec = rec;
    P.seed_lo = (uint32_t)seed;
    P.seed_hi = (uint32_t)(seed >> 32);
    P.scale_log2 = softmax_scale * 1.44269504088896340736f;
    P.L = L;
    const int G = P.Hq / P.Hkv;
    const int nblocks = P.Hkv * ((P.warm_waves > 0 ? P.warm_waves / kDecodeWaves : P.nchunk_max) + L.batch * P.ntail);
    const int chunks = P.chunk_limit > 0 && P.chunk_limit < P.nchunk_max ? P.chunk_limit : P.nchunk_max;
    const bool prior = !tail_k || !plain || priorities_pay(P.chunk_tiles, (int64_t)P.Hkv * (chunks + (int64_t)L.batch * P.ntail));
    P.full_share = prior ? P.chunk_tiles : kNoPriority;
    P.trace = (g_timeline != nullptr && (size_t)nblocks <= g_timeline_blocks) ? g_timeline : nullptr;
    switch (G) {
        case 1: return launch_g<1>(P, nblocks, st);
        case 2: return launch_g<2>(P, nblocks, st);
        case 4: return launch_g<4>(P, nblocks, st);
        case 8: return launch_g<8>(P, nblocks, st);
        case 16: return launch_g<16>(P, nblocks, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_zero_counters(uint32_t *counters, int n_words, hipStream_t st)
{
    hipLaunchKernelGGL(spark_zero_kernel, dim3((n_words + 255) / 256), dim3(256), 0, st, counters, n_words);
    return hipGetLastError();
}

}  // namespace spark
