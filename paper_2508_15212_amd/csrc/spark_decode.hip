// Host side of decode attention: parameter block, choice of the query-group instantiation, counter reset.
// The kernel template is in spark_decode_kernel.h; its instantiations are compiled in spark_decode_g*.hip.
#include "spark_decode_kernel.h"

namespace spark {

extern template hipError_t launch_g<1>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<2>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<4>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<8>(const DecodeParams &, int, hipStream_t);
extern template hipError_t launch_g<16>(const DecodeParams &, int, hipStream_t);

// Whether a call's tiles (over all KV heads) are few enough, and not too few, for the blocks of sixteen wavefronts of
// spark_decode_short.h.  Such a block takes four tiles at a time with four lanes a row, but all in one compute unit, whose LDS then
// bounds it; blocks of four wavefronts are as fast or faster for the row lengths that have an instantiation, except where
// eight query heads leave registers for small groups of entries only, and for very small calls of short rows.  One sequence, 8 KV
// heads, four / sixteen wavefronts a block (us; 1024 tokens are 128 tiles):
//   G = 4, T = 33:  1024 11.1 / 11.5   4096 13.2 / 12.6   8192 15.5 / 14.8   16384 21.3 / 20.2   32768 26.8 / 28.2
//          T = 90:  100 12.7 / 8.4   1024 15.6 / 13.5   8192 19.2 / 17.3   16384 24.8 / 26.0     T = 127:  1024 17.7 / 14.5
//   G = 8, T = 30:  1024 13.2 / 12.8   4096 16.2 / 14.5   16384 26.6 / 22.9    T = 80:  1024 19.1 / 15.6   16384 31.5 / 29.7
//          T = 26 (instantiated):  1024 11.9 / 12.2   8192 18.1 / 17.2   16384 25.4 / 22.5     T = 64:  8192 20.8 / 20.0
//   G = 2, T = 30:  2048 10.4 / 11.0   8192 14.1 / 13.4   T = 70:  1024 11.7 / 12.3   T = 127:  1024 15.8 / 14.0
//   G = 1, T = 30:  1024 8.8 / 9.5   4096 11.0 / 10.6   8192 13.6 / 12.3   T = 70:  1024 11.2 / 10.5   16384 21.0 / 21.2
static bool short_call_tiles(const SparkLayout &L, int G, int64_t tiles)
{
    if (row_length_instantiated(L)) return G == 8 && tiles >= 512 && tiles <= 2048;
    const bool long_rows = L.T > (G == 2 ? 80 : 64);
    const int64_t least = long_rows || G == 8 ? 0 : (G == 4 ? 288 : 512);
    return tiles >= least && tiles <= (long_rows && G <= 4 ? 1024 : 2048);
}

// The balanced mode and the blocks of sixteen wavefronts: dense values, degenerate recovery, rows of one length (`plain`),
// query groups up to 8 (else chunks by blocks of four).
// Short calls: all blocks are resident at once, one a compute unit.  Chunks get as much longer as that takes, where blocks of
// four wavefronts would have to do the same, or where that is half a pass (of four tiles) on average.  T = 32, four / sixteen
// wavefronts a block (us): 6 x 2000 to 3000 tokens 21.6 / 18.6; with 5.5 tiles a place (4 x 700 to 3900 tokens and appended
// rows) 15.1 / 14.5, with 6.6 (8 x 800 to 1500 and appended rows) 14.6 / 16.1.
DecodePlan decode_form(DecodePlan plan, const SparkLayout &L, int Hq, bool plain, int ntail)
{
    const int G = Hq / L.n_kv_heads;
    if (!plain || G > 8) plan.warm_waves = 0;
    plan.short_call = 0;
    if (!plain || G > 8 || plan.warm_waves > 0 || !short_call_tiles(L, G, L.n_tiles * L.n_kv_heads)) return plan;
    const int64_t room = 256 / L.n_kv_heads - (int64_t)L.batch * ntail;      // chunks there are places for
    if (plan.nchunk_max <= room) {
        plan.short_call = 1;
    } else if (plan.fixed_splits == 0 && L.batch <= 64 && room >= 2 * L.batch &&
               (plan.chunk_limit > 0 || L.n_tiles + 2 * L.batch <= 6 * room)) {
        plan.short_call = 1;
        plan.chunk_limit = plan.nchunk_max = (int)room;
    }
    return plan;
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

hipError_t launch_zero_counters(uint32_t *counters, int n, hipStream_t st)
{
    hipLaunchKernelGGL(spark_zero_kernel, dim3((n + 255) / 256), dim3(256), 0, st, counters, n);
    return hipGetLastError();
}

}  // namespace spark
