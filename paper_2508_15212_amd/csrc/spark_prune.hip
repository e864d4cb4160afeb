// Prefill-time channel pruning of the key cache for gfx950 (wave64).
//
// [Sec. "Problem Formulation and Analysis": saliency w = |q^j| * |k^j|, Eq. (7), Top_T;
//  Sec. "SparK": mean query over the observation window, mask and pruned keys;
//  App. "Caching Pruned Channel Statistics": mean saliency of the pruned set.]
//
// Kernels
//   spark_window_stat_kernel  a[b,h,j] = mean_g | mean_t Q_win[b,g,t,j] |  in float64, stored
//                             as float32 together with 1/a (G*128 threads per (b, h)); short calls
//                             do this in the pruning launch (see prune_launches).
//   spark_prune_kernel        top-T selection and packing, SIXTEEN LANES A ROW: a wavefront takes four rows at a time (a
//                             step; two steps a group), lane i of sixteen holds channels 8i .. 8i + 7.  A reduction
//                             over a row is four lane moves that serve four rows, slots and sums are per lane, and
//                             next to nothing of a row goes through the scalar unit.  Per row:
//     1. saliencies as float32 bit patterns; their top 15 bits (exponent, seven mantissa bits; fewer for the
//        smallest and the largest T) are the DIGIT.
//     2. one counting pass over 120 LDS bins of one digit each, 0.94 octaves around the place where the T-th largest is
//        expected: the row's mean digit, i.e. the logarithm of its geometric mean, plus an offset that follows the
//        rows before.  (Over rows of Gaussian keys the T-th digit stays within 0.44 octaves of that in 98.5 to
//        99.9 %; of the row's mean saliency in 93 to 99 %, of the row before in 41 to 99 %, which is why the window
//        can be this narrow and the digit this fine.)
//     3. the bin where the count reaches T gives the cut; in one row of ten it holds a key too many or two, which are
//        taken off one by one.  What does not fit (a T-th key outside the window, ties, crowded bins) is settled by
//        a bounded bisection of the bit pattern.
//     4. the lane's kept entries go to the row's place in LDS with 16-bit stores under the channels' masks, and sixteen
//        rows leave together in the tile's 16-byte sections.
//   What bounds it: vector issue.  45 vector and 19 scalar instructions a row (with one row at a time, two channels a lane,
//   41 and 37, and both units were at their limit).  One sequence of 131072 tokens x 8 KV heads, T = 26: 101 -> 87 us
//   (4.0 TB/s); 64 ragged sequences, T = 64: 66 -> 61 us; 40003 tokens, int8 codes: 46 -> 40 us; values, T_v = 38:
//   36 -> 34 us; 1024 tokens (one wavefront took a whole tile): 23 -> 10 us.  (Back to back on one input, of which a part
//   stays in the memory-side cache.  With inputs that rotate, 8 x 32768 tokens, T = 26: 191 -> 175 us.)  Four steps a group (fewer instructions,
//   43, but registers for four wavefronts per SIMD only) took 93 us instead of 86.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "spark_kernels.h"
#include "spark_layout.h"
#include "spark_wave.h"

namespace spark {

// ---------------------------------------------------------------- window statistic

// header of a key cache, by 64 threads
__device__ __forceinline__ void write_key_header(uint8_t *packed, const SparkLayout &L, int j)
{
    uint32_t v = 0;
    if (j == 0) v = SPARK_MAGIC;
    if (j == 1) v = (uint32_t)L.T;
    if (j == 2) v = (uint32_t)L.int8;
    if (j == 3) v = (uint32_t)L.batch;
    if (j == 4) v = (uint32_t)L.n_kv_heads;
    if (j == 5) v = (uint32_t)L.total_tokens;
    if (j == 6) v = (uint32_t)L.ndw;
    if (j == 8) v = (uint32_t)L.stats;      // (word 7 = 0: a key cache)
    reinterpret_cast<uint32_t *>(packed)[j] = v;
}

// grid = batch * Hkv blocks, min(G, 8) * 128 threads: thread (g, j) sums head g's window column j in
// float64 (t ascending), thread (0, j) then adds the G absolute means in g order -- the same order
// of operations as a plain loop nest.  Every sum of bf16 inputs this short is exact in float64, so
// the single rounding to float32 at the end decides a's bits.
__global__ __launch_bounds__(8 * SPARK_D) void spark_window_stat_kernel(const uint16_t *__restrict__ qwin,
                                                                     int Hq, int Hkv, int W,
                                                                     uint8_t *__restrict__ packed,
                                                                     SparkLayout L)
{
    __shared__ double absmean[16][SPARK_D];
    const int bh = blockIdx.x;
    if (L.topp) {          // the directory of the value streams starts empty (see spark_topp_prune_kernel)
        uint32_t *const dir = reinterpret_cast<uint32_t *>(packed + L.off_dir);
        const int64_t n = (int64_t)L.n_kv_heads * (L.n_tiles + 1);
        for (int64_t i = (int64_t)bh * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) dir[i] = 0u;
    }
    const int b = bh / Hkv, h = bh % Hkv;
    const int j = threadIdx.x % SPARK_D, g0 = threadIdx.x / SPARK_D;
    const int G = Hq / Hkv, GT = blockDim.x / SPARK_D;      // GT = min(G, 8) head slots
    for (int g = g0; g < G; g += GT) {
        const uint16_t *src = qwin + ((int64_t)(b * Hq + h * G + g) * W) * SPARK_D + j;
        double qs = 0.0;
        int t = 0;
        for (; t + 8 <= W; t += 8) {          // eight loads in flight, added in order
            uint16_t x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = src[(int64_t)(t + u) * SPARK_D];
#pragma unroll
            for (int u = 0; u < 8; ++u) qs += (double)bf16_bits_to_float(x[u]);
        }
        for (; t < W; ++t) qs += (double)bf16_bits_to_float(src[(int64_t)t * SPARK_D]);
        absmean[g][j] = fabs(qs / (double)W);
    }
    __syncthreads();
    if (g0 != 0) return;
    double s = 0.0;
    for (int gg = 0; gg < G; ++gg) s += absmean[gg][j];
    const float a32 = (float)(s / (double)G);
    float *a_out = reinterpret_cast<float *>(packed + L.off_a);
    float *inva_out = reinterpret_cast<float *>(packed + L.off_inva);
    a_out[(int64_t)bh * SPARK_D + j] = a32;
    inva_out[(int64_t)bh * SPARK_D + j] = (a32 != 0.0f) ? (1.0f / a32) : 0.0f;
    if (bh == 0 && j < 64) write_key_header(packed, L, j);
}

// ---------------------------------------------------------------- top-T selection + pack

constexpr int kPruneWaves = 4;      // wavefronts per block, each on its own rows
constexpr int kSteps = 2;           // a GROUP is what a wavefront takes at a time: two STEPS of four rows, sixteen lanes a row
constexpr int kGroup = 4 * kSteps;
constexpr int kStageRows = 16;      // a STAGE: the rows put together in LDS before they are written out
constexpr int kOverBins = 8;        // bins that collect the keys above the window (lane 0's)
constexpr int kBins = 128;          // eight a lane; the window is the 120 digits that follow
constexpr int kBinStride = kBins + 16;      // words per row of a step: the bins, then one spare word per lane
constexpr int kHistWords = 4 * kBinStride;  // per wavefront

// Bits of a key below its digit.  The T-th of 128 saliencies strays further from the row's mean the closer T is to either
// end, and fewer keys are near it.  With 128 digits an octave the window misses it in at most one step of four rows in 30
// from T = 12 to 99, but in 30 % at 112, 70 % at 120, 93 % at 127, and in 30 to 85 % at 8 and below where some channels are
// much larger than the others.  Half, a quarter and an eighth of the digits cut that to under 1 % (T = 1: 4 %; 120: under
// 1 %; 127: 4 %); in the middle they would only leave more keys of the T-th one's bin to be taken off one by one.
// 131072 tokens x 8 heads, eight large channels, one digit / this (us): T = 4 141 / 78, 8 100 / 80, 104 110 / 105, 112
// 126 / 109, 120 148 / 110, 127 176 / 116; values at 4 138 / 73, 8 90 / 78, 120 138 / 105.  (Few values of rows without
// large channels are the worse for it: 4 of 128 78 / 85, 8 80 / 79.)
__host__ inline uint32_t digit_shift_of(int T)
{
    if (T < 12) return T < 5 ? 18u : 17u;
    if (T < 100) return 16u;
    return T < 116 ? 17u : (T < 126 ? 18u : 19u);
}

// c - 4 a for a below 2^23 (one instruction)
__device__ __forceinline__ int minus_4x(uint32_t a, int c)
{
    int r;
    asm("v_mad_i32_i24 %0, %1, -4, %2" : "=v"(r) : "v"(a), "v"(c));
    return r;
}
// x clamped to [lo, hi] (one instruction; lo <= hi)
__device__ __forceinline__ int clamp_i32(int x, int lo, int hi)
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo), "v"(hi));
    return r;
}

// words per row in the LDS staging area: the row as it is stored (bf16 values also where int8 codes will be), rounded
// up to an odd number of 16-byte sections, so that lanes which read one section of sixteen rows meet no bank conflict
__host__ __device__ inline int spark_stage_words(const SparkLayout &L)
{
    int w = L.val0 + (L.T + 1) / 2;
    if (w < L.ndw) w = L.ndw;
    return 4 * (((w + 3) / 4) | 1);
}

__host__ __device__ inline size_t spark_prune_lds_bytes(const SparkLayout &L)
{
    return (size_t)kPruneWaves * (kStageRows * spark_stage_words(L) + kHistWords) * 4;
}

// WINDOW: sequences that can have a token in one tile, and the LDS for their channel weights besides
__host__ __device__ inline int spark_window_slots(const SparkLayout &L) { return L.batch < SPARK_TILE_TOKENS ? L.batch : SPARK_TILE_TOKENS; }
__host__ inline size_t spark_window_lds_bytes(const SparkLayout &L)
{
    return spark_prune_lds_bytes(L) + (size_t)spark_window_slots(L) * (SPARK_D * sizeof(float) + sizeof(int));
}

// The kept ones of a lane's eight channels (x: two a word; kb: the channels' wave masks) go to the 16-bit places in LDS
// from byte address `slot` on; returns the sum of the other ones' saliencies (their float32 bits in key).  Stores run
// under the masks and additions under their complements; all lanes are active before and after.
template <bool SUM>
__device__ __forceinline__ float stage_row(uint32_t slot, const uint4 &x, const uint64_t (&kb)[8], const uint32_t (&key)[8])
{
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;      // (sums by pairs: smaller rounding errors than one running sum's)
#define SPARK_STAGE(STORE, X, C)             \
    "s_mov_b64 exec, %[k" C "]\n\t"          \
    STORE " %[p], %[" X "]\n\t"              \
    "v_add_u32 %[p], 2, %[p]\n\t"
#define SPARK_STAGE_SUM(STORE, X, C, S)      \
    SPARK_STAGE(STORE, X, C)                 \
    "s_not_b64 exec, exec\n\t"               \
    "v_add_f32 %[" S "], %[" S "], %[w" C "]\n\t"
#define SPARK_STAGE_ONLY(STORE, X, C, S) SPARK_STAGE(STORE, X, C)
#define SPARK_STAGE_ALL(M)                                                                                         \
    M("ds_write_b16", "x0", "0", "s0") M("ds_write_b16_d16_hi", "x0", "1", "s1") M("ds_write_b16", "x1", "2", "s2") \
    M("ds_write_b16_d16_hi", "x1", "3", "s3") M("ds_write_b16", "x2", "4", "s0")                                   \
    M("ds_write_b16_d16_hi", "x2", "5", "s1") M("ds_write_b16", "x3", "6", "s2")                                   \
    M("ds_write_b16_d16_hi", "x3", "7", "s3")
    if constexpr (SUM) {
        asm volatile(SPARK_STAGE_ALL(SPARK_STAGE_SUM) "s_mov_b64 exec, -1"
                     : [p] "+v"(slot), [s0] "+v"(s0), [s1] "+v"(s1), [s2] "+v"(s2), [s3] "+v"(s3)
                     : [x0] "v"(x.x), [x1] "v"(x.y), [x2] "v"(x.z), [x3] "v"(x.w), [k0] "s"(kb[0]), [k1] "s"(kb[1]),
                       [k2] "s"(kb[2]), [k3] "s"(kb[3]), [k4] "s"(kb[4]), [k5] "s"(kb[5]), [k6] "s"(kb[6]), [k7] "s"(kb[7]),
                       [w0] "v"(key[0]), [w1] "v"(key[1]), [w2] "v"(key[2]), [w3] "v"(key[3]), [w4] "v"(key[4]),
                       [w5] "v"(key[5]), [w6] "v"(key[6]), [w7] "v"(key[7])
                     : "memory", "scc");
    } else {
        asm volatile(SPARK_STAGE_ALL(SPARK_STAGE_ONLY) "s_mov_b64 exec, -1"
                     : [p] "+v"(slot)
                     : [x0] "v"(x.x), [x1] "v"(x.y), [x2] "v"(x.z), [x3] "v"(x.w), [k0] "s"(kb[0]), [k1] "s"(kb[1]),
                       [k2] "s"(kb[2]), [k3] "s"(kb[3]), [k4] "s"(kb[4]), [k5] "s"(kb[5]), [k6] "s"(kb[6]), [k7] "s"(kb[7])
                     : "memory");
    }
#undef SPARK_STAGE_ALL
#undef SPARK_STAGE_ONLY
#undef SPARK_STAGE_SUM
#undef SPARK_STAGE
    return (s0 + s1) + (s2 + s3);
}

// keys >= x of a row (the same in its sixteen lanes)
__device__ __forceinline__ uint32_t count_ge(const uint32_t (&key)[8], uint32_t x)
{
    uint32_t n = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) n += key[c] >= x ? 1u : 0u;
    return row16_sum(n);
}

constexpr uint32_t kCloseEnough = 3;      // keys too many that are taken off one by one

// Brings lo <= the T-th largest key of the row < hi together until hi - lo <= `width` or fewer than `few` keys are
// >= lo (count: that number).  low / high: whether lo and hi are such bounds on entry (where neither is, they are
// equal); a bound that is not known is looked for from the other one in steps that double.
__device__ __forceinline__ void bracket(const uint32_t (&key)[8], uint32_t T, uint32_t &lo, uint32_t &hi, uint32_t &count,
                                        bool low, bool high, uint32_t width, uint32_t few)
{
    uint32_t step = 1u << 22;
    for (int it = 0; it < 64; ++it) {         // (at most ten doublings, then 32 halvings)
        const bool active = !low || !high || (count >= few && hi - lo > width);
        if (__ballot(active) == 0ull) break;
        const uint32_t down = hi > step ? hi - step : 0u;
        const uint32_t up = lo < 0x80000000u - step ? lo + step : 0x80000000u;
        const uint32_t mid = !low ? down : (!high ? up : lo + ((hi - lo) >> 1));
        const uint32_t n = count_ge(key, mid);
        if (active) {
            if (n >= T || mid == 0u) {
                lo = mid;
                count = n;
                low = true;
            } else {
                hi = mid;
                high = true;
            }
            high = high || mid >= 0x80000000u;          // (nothing finite is up there: the loop ends whatever the keys are)
            step = step < (1u << 30) ? 2u * step : step;
        }
    }
}

// The channel weights of one (sequence, KV head) by a block of the pruning kernel: the sums of spark_window_stat_kernel in the
// same order, two channels a thread.  absmean: G * 128 doubles of LDS, a_out: 128 floats of LDS.  Whole block; ends in a barrier.
__device__ __forceinline__ void block_window_stat(const uint16_t *__restrict__ qwin, int Hq, int G, int W, int b, int h,
                                                  double *absmean, float *a_out)
{
    for (int p = threadIdx.x; p < G * (SPARK_D / 2); p += kPruneWaves * 64) {
        const int g = p / (SPARK_D / 2), j2 = 2 * (p % (SPARK_D / 2));
        const char *src = reinterpret_cast<const char *>(qwin + ((int64_t)(b * Hq + h * G + g) * W) * SPARK_D + j2);
        double s0 = 0.0, s1 = 0.0;
        auto add_rows = [&](auto n, int t) __attribute__((always_inline)) {
            uint32_t x[decltype(n)::value];
#pragma unroll
            for (int u = 0; u < decltype(n)::value; ++u) x[u] = *reinterpret_cast<const uint32_t *>(src + (t + u) * (2 * SPARK_D));
#pragma unroll
            for (int u = 0; u < decltype(n)::value; ++u) {
                s0 += (double)bf16_bits_to_float(x[u] & 0xFFFFu);
                s1 += (double)__uint_as_float(x[u] & 0xFFFF0000u);
            }
        };
        int t = 0;
        for (; t + 32 <= W; t += 32) add_rows(std::integral_constant<int, 32>(), t);
        for (; t + 8 <= W; t += 8) add_rows(std::integral_constant<int, 8>(), t);
        for (; t < W; ++t) add_rows(std::integral_constant<int, 1>(), t);
        absmean[g * SPARK_D + j2] = fabs(s0 / (double)W);
        absmean[g * SPARK_D + j2 + 1] = fabs(s1 / (double)W);
    }
    __syncthreads();
    if (threadIdx.x < SPARK_D) {
        double s = 0.0;
        for (int gg = 0; gg < G; ++gg) s += absmean[gg * SPARK_D + threadIdx.x];
        a_out[threadIdx.x] = (float)(s / (double)G);
    }
    __syncthreads();
}

// The first n_whole tiles (over all heads) take one wavefront each, the next n_half two, the others four; a wavefront takes its
// rows a group (eight) at a time and writes them out a stage (sixteen, two groups) at a time.
// MODE: bit 0 = int8 codes + scale instead of bf16 kept entries; bit 1 = the rows also carry the all-channel mean
// and standard deviation of the row's saliencies (App. "Caching Pruned Channel Statistics", for the sampled recovery).
// VALUES: the rows are value-cache rows (App. "Pruning Value Cache Channels"): the score of a channel is
// |v| itself, there is no channel weight, no sequence bookkeeping and no statistic of the pruned set.
// WINDOW: short calls (a block is a tile, four wavefronts), where the window statistic's own launch would be a third of
// the time: a block computes the channel weights of the sequences in its tile itself, in LDS, while its rows are on their way;
// batch * Hkv further blocks store them for the reader of the cache.
// (128 registers there, and 2 spilled; 76 to 80 without.)
template <int MODE, bool VALUES, bool WINDOW = false>
__global__ __launch_bounds__(kPruneWaves * 64, WINDOW ? 4 : 6) void spark_prune_kernel(
    const uint16_t *__restrict__ k, int64_t k_tok_stride, int64_t k_head_stride, const int32_t *__restrict__ cu,
    uint8_t *__restrict__ packed, SparkLayout L, uint32_t n_whole, uint32_t n_half, uint32_t digit_shift,
    const uint16_t *__restrict__ qwin, int Hq, int W)
{
    static_assert(!(VALUES && WINDOW), "values have no channel weights");
    constexpr bool INT8 = (MODE & 1) != 0, STATS = (MODE & 2) != 0;
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    // the wavefront index is the same in all 64 lanes; saying so keeps everything derived from it in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wt = blockIdx.x * kPruneWaves + (uint32_t)wave;       // (the host checks that tiles fit 30 bits)
    if (VALUES && wt == 0) {
        // header of a value cache (the key cache's is written with the channel weights)
        uint32_t v = 0;
        if (lane == 0) v = SPARK_MAGIC;
        if (lane == 1) v = (uint32_t)L.T;
        if (lane == 4) v = (uint32_t)L.n_kv_heads;
        if (lane == 5) v = (uint32_t)L.total_tokens;
        if (lane == 6) v = (uint32_t)L.ndw;
        if (lane == 7) v = 1u;   // value cache
        reinterpret_cast<uint32_t *>(packed)[lane] = v;
    }
    // (WINDOW: weights of the tile's sequences, in order, and which sequences they are, behind the wavefronts' areas)
    float *const a_lds = reinterpret_cast<float *>(smem + spark_prune_lds_bytes(L));
    const int a_slots = spark_window_slots(L);
    int *const seq_lds = reinterpret_cast<int *>(a_lds + a_slots * SPARK_D);
    const int G = WINDOW ? Hq / L.n_kv_heads : 1;
    if constexpr (WINDOW) {
        const int64_t bh = (int64_t)blockIdx.x - L.n_tiles * L.n_kv_heads;
        if (bh >= 0) {                                   // (block-uniform)
            block_window_stat(qwin, Hq, G, W, (int)(bh / L.n_kv_heads), (int)(bh % L.n_kv_heads), reinterpret_cast<double *>(smem), a_lds);
            if (threadIdx.x < SPARK_D) {
                const float a32 = a_lds[threadIdx.x];
                reinterpret_cast<float *>(packed + L.off_a)[bh * SPARK_D + threadIdx.x] = a32;
                reinterpret_cast<float *>(packed + L.off_inva)[bh * SPARK_D + threadIdx.x] = (a32 != 0.0f) ? (1.0f / a32) : 0.0f;
                if (bh == 0 && threadIdx.x < 64) write_key_header(packed, L, threadIdx.x);
            }
            return;
        }
    }
    // tile number over the heads, and which share of the tile
    uint32_t gt = wt, lg_per_tile = 0, share = 0;
    if (wt >= n_whole) {
        const uint32_t after_whole = wt - n_whole, after_half = after_whole - 2u * n_half;
        lg_per_tile = after_whole < 2u * n_half ? 1u : 2u;
        const uint32_t i = lg_per_tile == 1u ? after_whole : after_half;
        gt = n_whole + (lg_per_tile == 1u ? 0u : n_half) + (i >> lg_per_tile);
        share = i & ((1u << lg_per_tile) - 1u);
    }
    if (gt >= (uint32_t)(L.n_tiles * L.n_kv_heads)) return;     // the whole wavefront leaves; no block barrier is used
    const int h = (int)(gt / (uint32_t)L.n_tiles);
    const int64_t tile = gt - (uint32_t)h * (uint32_t)L.n_tiles;
    const int rows = SPARK_TILE_TOKENS >> lg_per_tile;          // (a multiple of kStageRows)
    int t0 = (int)share * rows;                                 // first row of the stage in hand
    const int t_end = t0 + rows;
    const int64_t n0 = tile * SPARK_TILE_TOKENS;
    const int64_t left = L.total_tokens - n0;
    const int nvalid = left < SPARK_TILE_TOKENS ? (int)left : SPARK_TILE_TOKENS;
    const uint32_t T = (uint32_t)L.T;
    const int row = lane >> 4, sub = lane & 15;          // this lane: channels 8 sub .. 8 sub + 7 of row 4 s + row of the group
    const int sw = spark_stage_words(L);
    uint32_t *const stage = reinterpret_cast<uint32_t *>(smem) + (size_t)wave * (kStageRows * sw + kHistWords);
    const uint32_t stage_a = lds_address(stage);
    const uint32_t hist_a = stage_a + 4u * (uint32_t)(kStageRows * sw);

    // Row addresses: a wave-uniform base and one 32-bit offset per lane and step.  Rows past the last token repeat it.
    const char *const kbase = reinterpret_cast<const char *>(k + n0 * k_tok_stride + (int64_t)h * k_head_stride);
    const uint32_t stride_b = (uint32_t)k_tok_stride * 2u;   // bytes per token row (the host checks the range)
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const uint32_t lane_b = (uint32_t)row * stride_b + 16u * (uint32_t)sub;
    auto load_rows = [&](int t) __attribute__((always_inline)) -> uint4 {
        u32x4 v;
        if (nvalid == SPARK_TILE_TOKENS)
            v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(kbase + (size_t)((uint32_t)t * stride_b) + lane_b));
        else
            v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(kbase + ((uint32_t)min(t + row, nvalid - 1) * stride_b + 16u * sub)));
        return make_uint4(v.x, v.y, v.z, v.w);
    };
    uint4 x[kSteps];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) x[s] = load_rows(t0 + 4 * s);

    // sequence of this lane's row: the largest b with cu[b] <= its token (skips empty sequences), found for the first row
    int b = 0, seq_end_t = 0x7FFFFFFF;
    float a[8];
    const float *const a_all = reinterpret_cast<const float *>(packed + L.off_a) + (int64_t)h * SPARK_D + 8 * sub;
    int a_slot = 0;
    auto load_a = [&]() __attribute__((always_inline)) {
        const float4 *src = reinterpret_cast<const float4 *>(a_all + (int64_t)b * L.n_kv_heads * SPARK_D);
        if constexpr (WINDOW) {
            while (seq_lds[a_slot] != b) ++a_slot;       // (every sequence with a token in the tile is there)
            src = reinterpret_cast<const float4 *>(a_lds + a_slot * SPARK_D + 8 * sub);
        }
        const float4 lo = src[0], hi = src[1];
        a[0] = lo.x; a[1] = lo.y; a[2] = lo.z; a[3] = lo.w;
        a[4] = hi.x; a[5] = hi.y; a[6] = hi.z; a[7] = hi.w;
    };
    auto sequence_of = [&](int64_t token) __attribute__((always_inline)) {
        int lo = 0, hi = L.batch;     // invariant: cu[lo] <= token < cu[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (cu[mid] <= token) lo = mid; else hi = mid;
        }
        return lo;
    };
    if constexpr (WINDOW) {
        int sb = sequence_of(n0), end = cu[sb + 1];
        for (int i = 0;; ++i) {
            block_window_stat(qwin, Hq, G, W, sb, h, reinterpret_cast<double *>(smem), a_lds + i * SPARK_D);
            if (threadIdx.x == 0) seq_lds[i] = sb;
            if (end >= n0 + nvalid || i == a_slots - 1) break;
            const int from = end;
            do {
                ++sb;
                end = cu[sb + 1];
            } while (end <= from);
        }
        __syncthreads();
    }
    if constexpr (!VALUES) {
        b = sequence_of(n0 + (t0 < nvalid ? t0 : nvalid - 1));
        seq_end_t = (int)((int64_t)cu[b + 1] - n0);   // total < 2^31
        load_a();
    }

    // the staging area is zero where no kept value goes (the padding, the upper half of the last word for odd T)
    for (int i = lane; i < kStageRows * sw; i += 64) stage[i] = 0u;

    const uint32_t bins_a = hist_a + 4u * (uint32_t)(row * kBinStride);          // this row's bins
    const int lo_clamp = (int)(bins_a + 4u * (uint32_t)(sub & (kOverBins - 1))); // where a key above the window counts
    const int hi_clamp = (int)(bins_a + 4u * (uint32_t)(kBins + sub));           // this lane's spare word, past the bins
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
    lds_u32x4 *const my_bins = (lds_u32x4 *)(uintptr_t)(bins_a + 32u * (uint32_t)sub);
    const uint32_t row_a = stage_a + 4u * (uint32_t)(row * sw);                  // staged row of step 0
    const uint32_t step_a = 16u * (uint32_t)sw;                                  // four staged rows
    uint8_t *const tile_out = packed + L.off_tiles + ((int64_t)h * L.n_tiles + tile) * L.tile_bytes;
    // Digit (exponent and seven mantissa bits) of the T-th largest key, above the mean digit of the row: digits are
    // logarithms, so this is a ratio to the geometric mean of the row's saliencies.  Follows the rows.
    int offset = 0;
    bool have_offset = false;

    // One counting pass: clear_bins(), add_digits() for one or two rows a lane, bins_reached().
    auto clear_bins = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) my_bins[j] = u32x4{0u, 0u, 0u, 0u};
        prune_lds_sync();
    };
    auto add_digits = [&](const uint32_t (&digit)[8], int top, uint32_t one) __attribute__((always_inline)) {
        const int top_a = (int)bins_a + 4 * top;         // (top: the digit of bin 0)
#pragma unroll
        for (int c = 0; c < 8; ++c)
            __hip_atomic_fetch_add(lds_word((uint32_t)clamp_i32(minus_4x(digit[c], top_a), lo_clamp, hi_clamp)), one,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    };
    // Keys with a digit not below the bin's, step s in half s of the word, plus 2^15 - T: the half's sign says that the
    // count has reached T.  Returns in how many of the row's bins it has (half s: the row of step s).  A byte permute
    // turns the four signs of two words into bytes of all ones, and a dot product of bytes counts them.
    static_assert(kSteps == 2, "two steps in the halves of a word");
    auto bins_reached = [&]() __attribute__((always_inline)) -> uint32_t {
        prune_lds_sync();
        const u32x4 b0 = my_bins[0], b1 = my_bins[1];
        prune_lds_sync();
        const uint32_t h8[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
        const uint32_t all = ((b0.x + b0.y) + (b0.z + b0.w)) + ((b1.x + b1.y) + (b1.z + b1.w));
        uint32_t cum = row16_inclusive_sum(all) - all + (32768u - T) * 0x00010001u;
        int reached = 0;                               // of this lane's eight bins: step 0 + 16 step 1
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            const uint32_t c0 = cum + h8[j], c1 = c0 + h8[j + 1];
            cum = c1;
            reached = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_perm(c1, c0, 0x0B0A0908u), (int)0xF0FFF0FFu, reached, false);
        }
        return row16_sum(((uint32_t)reached & 15u) | (((uint32_t)reached & 0xF0u) << 12));
    };
    // The rare rest, in any row: T-th key outside the window, many keys in its bin, keys equal to it.  p, count: keys >= p;
    // bin: where the counting pass ended.  Leaves the kept keys' masks in kb and the T-th key, or one just below, in p.
    auto settle = [&](const uint32_t (&ks)[8], uint32_t &p, uint32_t count, int bin, uint64_t (&kb)[8]) __attribute__((always_inline)) {
        bool tied = false;
        uint32_t keep_eq = 0;          // tied: how many of the keys == p are kept
        {
            const bool low = count >= T, inside = bin >= kOverBins;
            uint32_t hi = low ? (inside ? p + (1u << digit_shift) : 0x80000000u) : min(p, 0x80000000u);
            bracket(ks, T, p, hi, count, low, !low || inside, 1u, T + kCloseEnough + 1u);
        }
        for (uint32_t it = 0; it <= kCloseEnough; ++it) {
            const bool over = count > T && !tied;
            if (__ballot(over) == 0ull) break;
            uint32_t dist[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) dist[c] = ks[c] - p;
            const uint32_t next = p + row16_min(min8(dist)) + 1u;
            const uint32_t n = count_ge(ks, next);
            if (over) {
                tied = n < T;
                keep_eq = T - n;
                p = tied ? next - 1u : next;
                count = tied ? count : n;
            }
        }
        uint32_t eq = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) eq += ks[c] == p ? 1u : 0u;
        uint32_t rank = row16_inclusive_sum(eq) - eq;
        const bool odd = !tied && count != T;      // (keys that are no numbers: any T channels)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const bool is_eq = tied && ks[c] == p;                 // (the lowest channels get the places that are left)
            const bool keep = is_eq ? rank < keep_eq : ks[c] >= p;
            rank += is_eq ? 1u : 0u;
            kb[c] = __ballot(odd ? 8u * sub + c < T : keep);
        }
    };
    constexpr int kTop = (kBins - kOverBins) / 2 + kOverBins;      // digit of bin 0 above the window's centre

    for (; t0 < t_end; t0 += kStageRows) {
        uint32_t mu_reg = 0, all_reg = 0, sq_reg = 0;      // lane 16 row + i: sums of staged row 4 i + row
#pragma nounroll
        for (int g0 = 0; g0 < kStageRows; g0 += kGroup) {
            const int tg = t0 + g0;
            if (tg >= nvalid) break;
            uint32_t key[kSteps][8];
            int mean[kSteps];
            if (have_offset) clear_bins();
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                if constexpr (!VALUES) {
                    const int t = tg + 4 * s + row;
                    if (t >= seq_end_t && t < nvalid) {      // (lanes of a row move on together)
                        do {
                            ++b;
                            seq_end_t = (int)((int64_t)cu[b + 1] - n0);
                        } while (t >= seq_end_t);
                        load_a();
                        // finish these loads here, inside the rare branch: otherwise the wait for them lands after
                        // the join and drains the prefetched rows on every step
                        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
                    }
                }
                const uint32_t xw[4] = {x[s].x, x[s].y, x[s].z, x[s].w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if constexpr (VALUES) {
                        // |v|, and in the sixteen bits that a bf16 magnitude leaves free the channel, lower ones
                        // above: no two keys of a row are equal, and equal magnitudes go to the lower channel
                        key[s][2 * c] = ((xw[c] << 16) & 0x7FFF0000u) | (uint32_t)(SPARK_D - 1 - 8 * sub - 2 * c);
                        key[s][2 * c + 1] = (xw[c] & 0x7FFF0000u) | (uint32_t)(SPARK_D - 2 - 8 * sub - 2 * c);
                    } else {
                        // saliency: one float32 multiply, never fused
                        key[s][2 * c] = __float_as_uint(__fmul_rn(a[2 * c], fabsf(__uint_as_float(xw[c] << 16))));
                        key[s][2 * c + 1] = __float_as_uint(__fmul_rn(a[2 * c + 1], fabsf(__uint_as_float(xw[c] & 0xFFFF0000u))));
                    }
                }
                uint32_t digit[8], dsum = 0;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    digit[c] = key[s][c] >> digit_shift;
                    dsum += digit[c];
                }
                mean[s] = (int)(row16_sum(dsum) >> 7);
                if (s == 0 && !have_offset) {
                    // first rows: the T-th key to an eighth of an octave, from a counting pass over fifteen octaves
                    uint32_t wide[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) wide[c] = key[0][c] >> 20;
                    clear_bins();
                    const uint32_t finer = 20u - digit_shift;
                    add_digits(wide, (mean[0] >> finer) + kTop, 1u);
                    const int bin = kBins - (int)(bins_reached() & 0xFFFFu);
                    offset = (((mean[0] >> finer) + kTop - bin) << finer) + (1 << (finer - 1u)) - mean[0];
                    have_offset = true;
                    clear_bins();
                }
                add_digits(digit, mean[s] + offset + kTop, 1u << (16 * s));
            }
            const uint32_t reached = bins_reached();
            int learned = 0;
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                const uint32_t (&ks)[8] = key[s];
                const int bin = kBins - (int)((reached >> (16 * s)) & 0xFFFFu);       // (kBins: below the window)
                uint32_t p = (uint32_t)(mean[s] + offset + kTop - max(bin, kOverBins - 1)) << digit_shift;
                uint64_t kb[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) kb[c] = __ballot(ks[c] >= p);
                uint32_t m = byte_of_masks(kb);
                uint32_t upto = row16_inclusive_sum((uint32_t)__popc(m));
                if ((__ballot(upto != T) & 0x8000800080008000ull) != 0ull) {
                    // some row's bin did not end exactly at T keys, or its T-th key lies outside the window
                    uint32_t count = row16_last(upto);
                    // usual: one to three keys too many, which are taken off one by one, the smallest first
                    bool few = __ballot(count < T || count > T + kCloseEnough) == 0ull, done = false;
                    for (uint32_t it = 0; few && it < kCloseEnough; ++it) {
                        uint32_t dist[8];
#pragma unroll
                        for (int c = 0; c < 8; ++c) dist[c] = ks[c] - p;               // (keys < p wrap round)
                        const uint32_t next = p + row16_min(min8(dist)) + 1u;          // past the smallest key left
                        const uint32_t cut = count > T ? next : p;
#pragma unroll
                        for (int c = 0; c < 8; ++c) kb[c] = __ballot(ks[c] >= cut);
                        m = byte_of_masks(kb);
                        upto = row16_inclusive_sum((uint32_t)__popc(m));
                        done = (__ballot(upto != T) & 0x8000800080008000ull) == 0ull;
                        const uint32_t n = row16_last(upto);
                        few = !done && __ballot(n < T) == 0ull;        // (fewer than T: equal keys went together)
                        if (done || few) {
                            p = cut;
                            count = n;
                        }
                    }
                    if (__builtin_expect(!done, 0)) settle(ks, p, count, bin, kb);
                    if (__builtin_expect(!done, 0)) {
                        m = byte_of_masks(kb);
                        upto = row16_inclusive_sum((uint32_t)__popc(m));
                    }
                }
                learned += (int)(p >> digit_shift) - mean[s];
                const uint32_t ra = row_a + (uint32_t)(g0 / 4 + s) * step_a;
                *(lds_u8 *)(uintptr_t)(ra + (uint32_t)sub) = (uint8_t)m;
                const uint32_t slot = ra + 4u * (uint32_t)L.val0 + 2u * (upto - (uint32_t)__popc(m));
                const float pruned = stage_row<!VALUES>(slot, x[s], kb, ks);
                if (tg + kGroup < t_end) x[s] = load_rows(tg + kGroup + 4 * s);       // (its registers are free now)
                if constexpr (!VALUES) {
                    const uint32_t sum = __float_as_uint(row16_sum_f32(pruned));
                    mu_reg = sub == g0 / 4 + s ? sum : mu_reg;
                }
                if constexpr (STATS) {
                    // (sums by pairs, for the same reason)
                    float v[8], d[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) v[c] = __uint_as_float(ks[c]);
                    const float w = row16_sum_f32(((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]))) * (1.0f / (float)SPARK_D);
#pragma unroll
                    for (int c = 0; c < 8; ++c) d[c] = v[c] - w;
                    const float q = (fmaf(d[0], d[0], d[1] * d[1]) + fmaf(d[2], d[2], d[3] * d[3])) +
                                    (fmaf(d[4], d[4], d[5] * d[5]) + fmaf(d[6], d[6], d[7] * d[7]));
                    const uint32_t sq = __float_as_uint(row16_sum_f32(q));
                    all_reg = sub == g0 / 4 + s ? __float_as_uint(w) : all_reg;
                    sq_reg = sub == g0 / 4 + s ? sq : sq_reg;
                }
            }
            offset = (2 * offset + learned) >> 2;              // half the old, half the mean of the two new ones
        }
        if constexpr (!VALUES) {
            if (sub < kStageRows / 4 && t0 < nvalid) {
                uint32_t *const r = stage + (4 * sub + row) * sw;
                r[4] = __float_as_uint(T < SPARK_D ? __uint_as_float(mu_reg) / (float)(SPARK_D - (int)T) : 0.0f);
                if constexpr (STATS) {
                    r[INT8 ? 6 : 5] = all_reg;
                    r[INT8 ? 7 : 6] = __float_as_uint(sqrtf(__uint_as_float(sq_reg) * (1.0f / (float)SPARK_D)));
                }
            }
        }
        prune_lds_sync();
        // ---- the staged rows leave: lane = (row of the stage, one of four sections at a time)
        {
            const int rw = lane & 15, part = lane >> 4;
            uint32_t *const r = stage + rw * sw;
            if constexpr (INT8) {
                // absmax scale and round-to-nearest-even codes, decided in float32, by four lanes a row.  The staged
                // bf16 words are read two at a time (four values; val0 is even, rows are 16-byte aligned, and the
                // words behind the last kept value are zero up to the row's end).
                const uint2 *const vals2 = reinterpret_cast<const uint2 *>(r + L.val0);
                const int nquad = ((int)T + 3) / 4;
                uint2 v[8];
                float amax = 0.0f;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    v[i] = make_uint2(0u, 0u);
                    if (4 * i < nquad) {                                // (wave-uniform)
                        if (4 * i + part < nquad) v[i] = vals2[4 * i + part];
                        amax = fmaxf(fmaxf(amax, fabsf(bf16_bits_to_float(v[i].x & 0xFFFFu))), fabsf(bf16_bits_to_float(v[i].x >> 16)));
                        amax = fmaxf(fmaxf(amax, fabsf(bf16_bits_to_float(v[i].y & 0xFFFFu))), fabsf(bf16_bits_to_float(v[i].y >> 16)));
                    }
                }
                prune_lds_sync();
                {
                    const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(amax), __float_as_uint(amax), false, false);
                    amax = fmaxf(__uint_as_float(r16[0]), __uint_as_float(r16[1]));
                    const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(amax), __float_as_uint(amax), false, false);
                    amax = fmaxf(__uint_as_float(r32[0]), __uint_as_float(r32[1]));
                }
                const float scale = __fdiv_rn(amax, 127.0f);
                // The code is rint(fl32(v / scale)).  The exact division costs ten instructions a value, so the
                // integer is first taken from v times an approximate reciprocal: that product and the exactly
                // rounded quotient both lie within 3.1e-5 of v / scale (|v / scale| <= 127, reciprocal to one
                // unit in the last place, two roundings), so unless the product comes within 6e-5 of a half
                // integer the two round to the same integer; otherwise (and when the reciprocal is not
                // finite) the lane divides exactly.
                const float rs = __builtin_amdgcn_rcpf(scale);
                auto code_of = [&](uint32_t bits) -> uint32_t {
                    const float val = bf16_bits_to_float(bits);
                    const float qa = val * rs;
                    float qf = rintf(qa);
                    if (!(fabsf(qa - qf) < 0.5f - 6e-5f)) qf = rintf(__fdiv_rn(val, scale));
                    // (|v| <= amax and scale = fl32(amax / 127), so |qf| <= 127 already: no clamp is needed)
                    return (uint32_t)(int)qf & 0xFFu;
                };
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (4 * i < nquad) {
                        uint32_t word = 0;
                        if (scale != 0.0f)
                            word = code_of(v[i].x & 0xFFFFu) | (code_of(v[i].x >> 16) << 8) | (code_of(v[i].y & 0xFFFFu) << 16) |
                                   (code_of(v[i].y >> 16) << 24);
                        if (4 * i + part < nquad) r[L.val0 + 4 * i + part] = word;
                    }
                }
                if (part == 0) {
                    r[5] = __float_as_uint(scale);
                    if (L.val0 + L.nv < L.ndw) r[L.val0 + L.nv] = 0u;
                }
                prune_lds_sync();
            }
            const int t = t0 + rw;
            // Rows past the last token carry a well-formed mask (channels 0..T-1) and zeros, so that a reader that
            // walks exactly T bits never runs off the mask.
            auto low_bits = [](int n) { return n <= 0 ? 0u : (n >= 32 ? 0xFFFFFFFFu : ((1u << n) - 1u)); };
            // (written once, read by another kernel much later: non-temporal, like the loads)
            for (int q = part; q < L.nq + L.tail2; q += 4) {
                const uint4 s = *reinterpret_cast<const uint4 *>(r + 4 * q);
                u32x4 v = {s.x, s.y, s.z, s.w};
                if (t >= nvalid) {
                    v = u32x4{0u, 0u, 0u, 0u};
                    if (q == 0) v = u32x4{low_bits((int)T), low_bits((int)T - 32), low_bits((int)T - 64), low_bits((int)T - 96)};
                }
                if (q < L.nq)
                    __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(tile_out + (size_t)q * 1024 + t * 16));
                else
                    __builtin_nontemporal_store(u32x2{v.x, v.y}, reinterpret_cast<u32x2 *>(tile_out + (size_t)q * 1024 + t * 8));
            }
            prune_lds_sync();      // the staging rows are reused
        }
    }
}

// ---------------------------------------------------------------- canonical export

// one thread per (token, KV head) row
__global__ void spark_unpack_kernel(const uint8_t *__restrict__ packed, SparkLayout L,
                                    uint32_t *mask_out, void *vals_out, float *mu_out,
                                    float *scale_out, float *a_out, float *mu_all_out, float *sigma_out)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t rows = L.total_tokens * L.n_kv_heads;
    if (a_out && idx < (int64_t)L.batch * L.n_kv_heads * SPARK_D)
        a_out[idx] = reinterpret_cast<const float *>(packed + L.off_a)[idx];
    if (idx >= rows) return;
    const int64_t n = idx / L.n_kv_heads;
    const int h = (int)(idx % L.n_kv_heads);
    const uint8_t *tile = packed + L.off_tiles + ((int64_t)h * L.n_tiles + n / SPARK_TILE_TOKENS) * L.tile_bytes;
    const int t = (int)(n % SPARK_TILE_TOKENS);
    auto word = [&](int d) {
        return *reinterpret_cast<const uint32_t *>(tile + spark_tile_word_offset(L, t, d));
    };
    if (mask_out)
        for (int m = 0; m < 4; ++m) mask_out[idx * 4 + m] = word(m);
    if (mu_out && !L.values) mu_out[idx] = __uint_as_float(word(4));
    if (L.stats) {
        if (mu_all_out) mu_all_out[idx] = __uint_as_float(word(L.int8 ? 6 : 5));
        if (sigma_out) sigma_out[idx] = __uint_as_float(word(L.int8 ? 7 : 6));
    }
    if (L.int8) {
        if (scale_out) scale_out[idx] = __uint_as_float(word(5));
        if (vals_out) {
            int8_t *o = reinterpret_cast<int8_t *>(vals_out) + idx * L.T;
            for (int i = 0; i < L.T; ++i) o[i] = (int8_t)((word(L.val0 + i / 4) >> (8 * (i & 3))) & 0xFF);
        }
    } else if (vals_out) {
        uint16_t *o = reinterpret_cast<uint16_t *>(vals_out) + idx * L.T;
        for (int i = 0; i < L.T; ++i) o[i] = (uint16_t)((word(L.val0 + i / 2) >> (16 * (i & 1))) & 0xFFFF);
    }
}


// ---------------------------------------------------------------- host-side launch

namespace {

// every tile of the cache in one launch
template <bool VALUES>
hipError_t launch_tiles(const uint16_t *x, int64_t tok_stride, int64_t head_stride, const int32_t *cu,
                        uint8_t *packed, const SparkLayout &L, hipStream_t st)
{
    const int64_t tiles = L.n_tiles * L.n_kv_heads;
    if (tiles == 0) return hipSuccess;
    if (tiles >= ((int64_t)1 << 30)) return hipErrorInvalidValue;
    // Wavefronts per tile.  One has the least set-up, but a wavefront that starts late and works on 64 rows lasts long
    // after the others are done (10 us with the chip to itself).  So wavefronts start in the order of their work: whole tiles
    // first, then halves of 1536 tiles, at the end quarters of 512 (2048 wavefronts, a third of what is resident).  No whole tiles
    // where the halves and quarters are resident together, or nearly (3072 tiles, 7168 wavefronts), and quarters only where tiles
    // are few (1408, 5632 wavefronts; values 1280).  Us, the window kernel included, one / two / four wavefronts for every tile (the
    // rule before took four up to 1536 tiles, two up to 10240) -> whole tiles, halves, quarters:
    //   keys: 2000 27 / 23 / 24 -> 21   5008 (int8) 46 / 42 / 43 -> 39   8000 55 / 52 -> 46   16384 88 / 90 -> 83
    //         4544 (ragged, T = 64) 64 / 62 -> 59   32768 161 / 167 -> 157
    //   values: 2000 24 / 19 / 18 -> 18   5008 34 / 33 / 34 -> 31   8000 49 / 47 -> 44   16384 85 / 87 -> 81
    //   keys, four -> halves and quarters: 625 15.3 -> 17.2   1024 17.3 -> 18.0   1250 17.9 -> 18.6; int8 codes: 625 16.5 -> 18.8   1250 19.8 -> 20.2
    //   the same as a ratio, mean of fifteen T from 24 to 96 (each 0.92 to 1.15): 1290 1.02   1340 1.02   1400 1.01   1460 1.01   1530 1.00;
    //   int8 codes 1.04, 1.03, 1.01, 1.02, 1.00; values (T_v = 26 / 64 / 100) 1281 1.01 / 1.00 / 1.04   1400 0.95 / 0.95 / 1.02
    //   two -> with whole tiles -> without: 2150 (T = 26) 22.6 -> 23.8 -> 20.8   2400 (T = 64, int8) 28.5 -> 28.4 -> 25.8   2560 (T = 96) 26.1 -> 27.4 -> 24.8
    //         3072 (T = 26 / 64 / 96) 26.3 / 26.2 / 29.0 -> 25.1 / 25.5 / 27.8 -> 25.4 / 24.5 / 27.1   values 2200 (T_v = 64) 18.9 -> 20.2 -> 18.8
    // Quarters of 256, 384, 768, 1536 and 3072 tiles and halves of 512 to 6144 were tried: 0 to 3 % slower.
    const int64_t n_quarter = tiles <= (VALUES ? 1280 : 1408) ? tiles : 512;
    const int64_t n_half = tiles <= 3072 || tiles - n_quarter < 1536 ? tiles - n_quarter : 1536;
    const int64_t n_whole = tiles - n_quarter - n_half;
    const int64_t waves = n_whole + 2 * n_half + 4 * (tiles - n_whole - n_half);
    auto launch = [&](auto kern) -> hipError_t {
        hipLaunchKernelGGL(kern, dim3((unsigned)((waves + kPruneWaves - 1) / kPruneWaves)), dim3(kPruneWaves * 64),
                           spark_prune_lds_bytes(L), st, x, tok_stride, head_stride, cu, packed, L, (uint32_t)n_whole, (uint32_t)n_half,
                           digit_shift_of(L.T), (const uint16_t *)nullptr, 0, 0);
        return hipGetLastError();
    };
    switch (VALUES ? 0 : (L.int8 ? 1 : 0) + (L.stats ? 2 : 0)) {
        case 0: return launch(&spark_prune_kernel<0, VALUES>);
        case 1: return launch(&spark_prune_kernel<1, false>);
        case 2: return launch(&spark_prune_kernel<2, false>);
        default: return launch(&spark_prune_kernel<3, false>);
    }
}

}  // namespace

hipError_t launch_window_stat(const uint16_t *qwin, uint8_t *packed, const SparkLayout &L, int Hq, int W, hipStream_t st)
{
    hipLaunchKernelGGL(spark_window_stat_kernel, dim3(L.batch * L.n_kv_heads),
                       dim3(((Hq / L.n_kv_heads) < 8 ? (Hq / L.n_kv_heads) : 8) * SPARK_D), 0, st, qwin, Hq,
                       L.n_kv_heads, W, packed, L);
    return hipGetLastError();
}

// The window statistic and the pruning in one launch: four wavefronts a tile, then a block per (sequence, KV head).
static hipError_t launch_window_and_tiles(const uint16_t *k, int64_t tok_stride, int64_t head_stride, const uint16_t *qwin, const int32_t *cu,
                                          uint8_t *packed, const SparkLayout &L, int Hq, int W, hipStream_t st)
{
    static_assert(kPruneWaves == 4, "a block is a tile");
    const unsigned blocks = (unsigned)((L.n_tiles + L.batch) * L.n_kv_heads);
    auto launch = [&](auto kern) -> hipError_t {
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(kPruneWaves * 64), spark_window_lds_bytes(L), st, k, tok_stride, head_stride, cu, packed, L, 0u, 0u,
                           digit_shift_of(L.T), qwin, Hq, W);
        return hipGetLastError();
    };
    switch ((L.int8 ? 1 : 0) + (L.stats ? 2 : 0)) {
        case 0: return launch(&spark_prune_kernel<0, false, true>);
        case 1: return launch(&spark_prune_kernel<1, false, true>);
        case 2: return launch(&spark_prune_kernel<2, false, true>);
        default: return launch(&spark_prune_kernel<3, false, true>);
    }
}

// Whether the window statistic goes into the pruning launch: calls whose blocks, one a tile, are all resident at once (three a
// compute unit, four would fit their registers; fewer where they take more LDS).  A launch of its own costs 4 us with the gap before the
// next; in the tile's block it costs 1 to 2 us per sequence that the tile spans (a block's loads, one after the other:
// therefore 256 tokens a sequence on average) and reads the window once per tile (therefore a bound on that: 32 MB).  One
// sequence, 8 KV heads, two launches / one (us):
//   G = 4, W = 32: 100 tokens 11.6 / 10.6   1024 13.2 / 10.5   2048 13.2 / 10.7   4096 14.6 / 12.5   5000 15.3 / 14.0
//   G = 8, W = 64: 1024 15.8 / 13.9   G = 1, W = 16: 2048 13.5 / 11.2   one KV head, 16384 tokens: 12.3 / 10.5
//   8 sequences of 260 tokens 13.7 / 12.6, of 300 to 700 14.4 / 12.9; prune and first decode step of 1024 tokens 23.3 / 21.2
// The line: 6000 tokens (760 blocks) 15.2 / 14.8, five of 1000 to 2000 (980 blocks) 16.5 / 17.1; with more blocks than are
// resident, 8192 tokens where there was room for 768, 17.1 / 19.9.
int prune_launches(const SparkLayout &L, int Hq, int W)
{
    const int64_t tiles = L.n_tiles * L.n_kv_heads, blocks = tiles + (int64_t)L.batch * L.n_kv_heads;
    const int G = Hq / L.n_kv_heads;
    const int64_t by_lds = (int64_t)(160 * 1024 / spark_window_lds_bytes(L));
    const bool one = tiles > 0 && blocks <= 256 * (by_lds < 3 ? by_lds : 3) && G <= 8 && L.total_tokens >= 256 * (int64_t)L.batch &&
                     tiles * G * W <= 131072;
    return one ? 1 : 2;
}

hipError_t launch_prune(const uint16_t *k, int64_t k_tok_stride, int64_t k_head_stride, const uint16_t *qwin,
                        const int32_t *cu, uint8_t *packed, const SparkLayout &L, int Hq, int W, hipStream_t st)
{
    // (a block reads two window columns at a time)
    if (prune_launches(L, Hq, W) == 1 && (reinterpret_cast<uintptr_t>(qwin) & 3u) == 0u) return launch_window_and_tiles(k, k_tok_stride, k_head_stride, qwin, cu, packed, L, Hq, W, st);
    const hipError_t e = launch_window_stat(qwin, packed, L, Hq, W, st);
    if (e != hipSuccess) return e;
    return launch_tiles<false>(k, k_tok_stride, k_head_stride, cu, packed, L, st);
}

hipError_t launch_prune_values(const uint16_t *v, int64_t v_tok_stride, int64_t v_head_stride, uint8_t *packed,
                               const SparkLayout &L, hipStream_t st)
{
    return launch_tiles<true>(v, v_tok_stride, v_head_stride, nullptr, packed, L, st);
}

hipError_t launch_unpack(const uint8_t *packed, const SparkLayout &L, uint32_t *mask_out, void *vals_out,
                         float *mu_out, float *scale_out, float *a_out, float *mu_all_out, float *sigma_out,
                         hipStream_t st)
{
    int64_t n = L.total_tokens * L.n_kv_heads;
    const int64_t na = (int64_t)L.batch * L.n_kv_heads * SPARK_D;
    if (a_out && na > n) n = na;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(spark_unpack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, packed, L,
                       mask_out, vals_out, mu_out, scale_out, a_out, mu_all_out, sigma_out);
    return hipGetLastError();
}

}  // namespace spark
