// The top-p variant of the prefill pruning for gfx950 (wave64).
//
// [Sec. "Adaptive Variants of SparK": per token, the fewest most salient channels whose saliencies together
//  account for 99 % of the row's total saliency are kept; no fixed pruning ratio.]
//
// The count of a row is an integer decided by sums, so the sums are integers too: every saliency of a row is
// expressed in units of the last place of the row's largest saliency, rounded down (q < 2^24, a row's total
// below 2^31), and with p in basis points the row keeps the smallest m >= 1 whose m largest saliencies have
//     10000 * sum q  >=  p * (total of q),      i.e.   sum q >= need := ceil(p * total / 10000).
// Exact in any summation order, which is what a parallel reduction needs.  Ties: lower channel first.
//
// Everything works on tiles of 64 tokens, four wavefronts of sixteen rows each, FOUR ROWS AT A TIME: sixteen lanes a row,
// eight channels a lane, so that a reduction over a row is four lane moves that serve four rows, and nothing of a row has
// to be wave-uniform.
//   select_tile   per row a selection ON SUMS: every lane adds the q of its channels to 128 LDS bins of an eighth of an
//                 octave each, from the row's largest key down; a prefix sum over the bins gives the bin in which the
//                 running sum reaches `need`, and the keys of that bin are then taken one by one, largest first (1.4 of them
//                 on average, 2.0 for the slowest of four rows; with four bins an octave 1.7 and 2.8).  A bin of which
//                 four keys or more are needed is first cut into 64 finer ones, up to three times.  Writes the rows'
//                 fixed part (mask, mean saliency of the pruned channels, count).
//   write_tile    takes the dense key rows again; every lane finds the slots of its eight channels from the row's mask byte, the
//                 kept entries of sixteen rows are put together in LDS and leave as whole words of the value stream.
//   spark_topp_prune_kernel   both, for small and large calls, in one launch: a block selects a tile and then writes one that
//                 was selected about 2048 tiles (over all heads) earlier; one block in up to 32 turns the lengths
//                 that the blocks before it have filed into the directory's sums.
//   spark_topp_select_kernel, spark_topp_scan_kernel, spark_topp_pack_kernel   the same one after the other, for calls in
//                 between (measurements beside the launch).
// What bounds them (one sequence of 65536 tokens x 8 KV heads, 51 kept channels a row): the selection by vector issue, 75 to 80
// instructions a row, 62 us alone; the writing by memory, 31 us alone for 134 MB read and 54 MB written.  In one launch they
// overlap: 96 -> 84 us for the whole call (calls back to back).  Tried: every block writing its own tile (137 us: it waits for the slowest
// block in front, holding its place), blocks that stay and write a tile late from LDS (109 us), 8 blocks per compute unit
// (spills, 109 us), 6 (90 us).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spark_kernels.h"
#include "spark_layout.h"
#include "spark_wave.h"

namespace spark {

namespace {

constexpr int kWaves = 4;            // wavefronts per block, one tile a block, sixteen rows a wavefront
constexpr int kRowsPerWave = SPARK_TILE_TOKENS / kWaves;
constexpr int kSteps = kRowsPerWave / 4;      // four rows at a time

// First counting level: eight bins an octave over the sixteen octaves below the top of the largest key's.
constexpr int kBins = 128;
constexpr int kBinsPerLane = kBins / 16;
constexpr int kBinStride = kBins + 16;        // words per row: the bins, then one spare word per lane for keys further down

// a saliency (float32 bits, sign clear) in units of 2^(emax - 150), rounded down; emax >= 1 and not below its exponent
__device__ __forceinline__ uint32_t quantise(uint32_t bits, int emax)
{
    const int e = max((int)(bits >> 23), 1);
    const uint32_t mant = bits - ((uint32_t)(e - 1) << 23);      // (the implied bit is in place; below 2^24)
    return mant >> min(emax - e, 31);
}

// Where the running sum over the sixteen lanes' bins (NB a lane, in order) reaches `need`: the number of bins in
// front of that one, and the sum over them.  What is missing to `need`, less one, is followed instead of the sum: its sign
// says that a bin has reached it (a byte permute makes bytes of all ones of two signs, a dot product of bytes counts
// them), and its smallest value above -1, taken as unsigned, gives the sum.
template <int NB>
__device__ __forceinline__ void find_bin(const uint32_t *bins, uint32_t before, uint32_t need, uint32_t &n, uint32_t &above)
{
    uint32_t r = need - 1u - before, least = r;
    int reached = 0;
#pragma unroll
    for (int j = 0; j < NB; j += 2) {
        const uint32_t r0 = r - bins[j], r1 = r0 - bins[j + 1];
        r = r1;
        least = min(least, min(r0, r1));
        reached = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_perm(r1, r0, 0x0C0C0B09u), 0x0000FFFF, reached, false);
    }
    n = 16u * NB - row16_sum((uint32_t)reached);
    above = need - 1u - row16_min(least);
}

// Sum of the saliencies (float32 bits in key) that are NOT in the channels' wave masks.  The additions run under the masks'
// complements; all lanes are active before and after.
__device__ __forceinline__ float sum_pruned(const uint64_t (&kb)[8], const uint32_t (&key)[8])
{
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;      // (sums by pairs: smaller rounding errors than one running sum's)
#define SPARK_SUM(C, S) "s_not_b64 exec, %[k" C "]\n\tv_add_f32 %[" S "], %[" S "], %[w" C "]\n\t"
    asm volatile(SPARK_SUM("0", "s0") SPARK_SUM("1", "s1") SPARK_SUM("2", "s2") SPARK_SUM("3", "s3") SPARK_SUM("4", "s0")
                 SPARK_SUM("5", "s1") SPARK_SUM("6", "s2") SPARK_SUM("7", "s3") "s_mov_b64 exec, -1"
                 : [s0] "+v"(s0), [s1] "+v"(s1), [s2] "+v"(s2), [s3] "+v"(s3)
                 : [k0] "s"(kb[0]), [k1] "s"(kb[1]), [k2] "s"(kb[2]), [k3] "s"(kb[3]), [k4] "s"(kb[4]), [k5] "s"(kb[5]),
                   [k6] "s"(kb[6]), [k7] "s"(kb[7]), [w0] "v"(key[0]), [w1] "v"(key[1]), [w2] "v"(key[2]), [w3] "v"(key[3]),
                   [w4] "v"(key[4]), [w5] "v"(key[5]), [w6] "v"(key[6]), [w7] "v"(key[7])
                 : "scc");
#undef SPARK_SUM
    return (s0 + s1) + (s2 + s3);
}

// What a tile's directory entry holds while the streams are being written: 0 (as cleared), the words of its own tile, or
// the words of all tiles up to it, which is what it holds in the end.  No tile has more than 64 * 64 words or fewer than
// one.  (A sum of kOwnWords or more would be taken for the words of a tile, and waited for without end: calls whose streams have
// room for that many do not come here, see topp_prune_launches.)
constexpr uint32_t kOwnWords = 0xFFFFE000u;
__device__ __forceinline__ uint32_t dir_load(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void dir_store(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Words of all tiles up to the one whose entry is dir[last], by one wavefront: from that entry back, own words are added until
// an entry holds a sum or there are no more.  Waits for entries that have not been filed.  after: words of the `lane` entries
// behind dir[last - lane].
__device__ __forceinline__ uint32_t words_up_to(const uint32_t *dir, int64_t last, int lane, uint32_t &after)
{
    const int64_t end = last;
    uint32_t sum = 0;
    for (;;) {
        const int64_t i = last - lane;                   // lane 0: the nearest
        const uint32_t v = i > 0 ? dir_load(dir + i) : 0u;
        const uint64_t sums = __ballot(i <= 0 || (v != 0u && v < kOwnWords));
        const int n = sums != 0ull ? (int)__builtin_ctzll(sums) : 64;           // own words to be added, then a sum
        if (__ballot(lane < n && v == 0u) != 0ull) {
            __builtin_amdgcn_s_sleep(8);                 // (what many ask for at a time comes late)
            continue;
        }
        const uint32_t add = lane < n ? v - kOwnWords : (lane == n ? v : 0u);
        const uint32_t upto = wave_inclusive_sum(add);
        if (last == end) after = upto - add;
        sum += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        if (n < 64) return sum;
        last -= 64;
    }
}

// The kept ones of a lane's eight channels (x: two channels a word; m: their mask byte) go to the 16-bit places in
// LDS that end at byte address `end`, in order.  The stores run under the channels' wave masks, taken off the byte
// from its top bit on; all lanes are active before and after.
__device__ __forceinline__ void stage_kept(uint32_t m, uint32_t end, const uint4 &x)
{
    m <<= 24;
    asm volatile(
#define SPARK_STAGE(STORE, X)                  \
    "v_add_co_u32 %[m], vcc, %[m], %[m]\n\t"   \
    "s_mov_b64 exec, vcc\n\t"                  \
    "v_add_u32 %[p], -2, %[p]\n\t"             \
    STORE " %[p], " X "\n\t"                   \
    "s_mov_b64 exec, -1\n\t"
        SPARK_STAGE("ds_write_b16_d16_hi", "%[x3]")
        SPARK_STAGE("ds_write_b16", "%[x3]")
        SPARK_STAGE("ds_write_b16_d16_hi", "%[x2]")
        SPARK_STAGE("ds_write_b16", "%[x2]")
        SPARK_STAGE("ds_write_b16_d16_hi", "%[x1]")
        SPARK_STAGE("ds_write_b16", "%[x1]")
        SPARK_STAGE("ds_write_b16_d16_hi", "%[x0]")
        SPARK_STAGE("ds_write_b16", "%[x0]")
#undef SPARK_STAGE
        : [m] "+v"(m), [p] "+v"(end)
        : [x0] "v"(x.x), [x1] "v"(x.y), [x2] "v"(x.z), [x3] "v"(x.w)
        : "memory", "vcc");
}

}  // namespace

// header of the cache, by sixteen lanes (the channel weights are written by the window kernel that runs before)
__device__ __forceinline__ void write_header(uint8_t *packed, const SparkLayout &L, int p_bp)
{
    const int lane = threadIdx.x;
    uint32_t v = 0;
    if (lane == 0) v = SPARK_MAGIC;
    if (lane == 3) v = (uint32_t)L.batch;
    if (lane == 4) v = (uint32_t)L.n_kv_heads;
    if (lane == 5) v = (uint32_t)L.total_tokens;
    if (lane == 6) v = (uint32_t)L.ndw;
    if (lane == 9) v = 1u;   // top-p cache
    if (lane == 10) v = (uint32_t)p_bp;
    reinterpret_cast<uint32_t *>(packed)[lane] = v;
}

// Selects the kept channels of a tile's rows: masks, means and counts; returns the words that the wavefront's rows take in the
// stream.  SAME_LAUNCH: another block of this launch reads them, so they are stored with device scope.
template <bool SAME_LAUNCH>
__device__ __forceinline__ uint32_t select_tile(const uint16_t *__restrict__ k, int64_t k_tok_stride, int64_t k_head_stride,
                                                const int32_t *__restrict__ cu, uint8_t *__restrict__ packed, const SparkLayout &L,
                                                int p_bp, int h, int64_t tile, uint32_t *wave_lds)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane >> 4, sub = lane & 15;          // this lane: channels 8 sub .. 8 sub + 7 of row 4 s + row
    const int64_t n0 = tile * SPARK_TILE_TOKENS;
    const int64_t left = L.total_tokens - n0;
    const int nvalid = left < SPARK_TILE_TOKENS ? (int)left : SPARK_TILE_TOKENS;
    const int t0 = wave * kRowsPerWave;
    uint8_t *tile_out = packed + L.off_tiles + ((int64_t)h * L.n_tiles + tile) * L.tile_bytes;
    uint32_t my_mu = 0, my_cnt = 0;      // lane 16 row + s (s < kSteps): mean pruned saliency and count of row t0 + 4 s + row
    uint32_t masks = 0;                  // mask byte of step s in byte s

    if (t0 < nvalid) {
        // all of the wavefront's rows are requested at once; rows past the last token repeat it
        uint4 x[kSteps];
        const uint16_t *kbase = k + n0 * k_tok_stride + (int64_t)h * k_head_stride + 8 * sub;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int t = t0 + 4 * s + row;
            x[s] = *reinterpret_cast<const uint4 *>(kbase + (int64_t)(t < nvalid ? t : nvalid - 1) * k_tok_stride);
        }
        // sequence of the first row: largest b with cu[b] <= its token (skips empty sequences)
        int b = 0, seq_end_t;
        {
            int hi = L.batch;     // invariant: cu[b] <= n0 + t0 < cu[hi]
            while (hi - b > 1) {
                const int mid = (b + hi) >> 1;
                if (cu[mid] <= n0 + t0) b = mid; else hi = mid;
            }
            seq_end_t = (int)((int64_t)cu[b + 1] - n0);
        }
        const float *a_all = reinterpret_cast<const float *>(packed + L.off_a) + (int64_t)h * SPARK_D + 8 * sub;
        float a[8];
        auto load_a = [&]() __attribute__((always_inline)) {
            const float4 *src = reinterpret_cast<const float4 *>(a_all + (int64_t)b * L.n_kv_heads * SPARK_D);
            const float4 lo = src[0], hi = src[1];
            a[0] = lo.x; a[1] = lo.y; a[2] = lo.z; a[3] = lo.w;
            a[4] = hi.x; a[5] = hi.y; a[6] = hi.z; a[7] = hi.w;
        };
        load_a();
        uint32_t *const hist = wave_lds + row * kBinStride;
        const uint32_t hist_a = lds_address(hist);
        const uint32_t below = ((uint32_t)(kBins + sub) << 20) | 0xFFFFFu;      // the lane's spare word, as a distance

#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int t = t0 + 4 * s + row;
            if (t >= seq_end_t && t < nvalid) {      // (lanes of a row move on together; b stays behind in rows past the end)
                do {
                    ++b;
                    seq_end_t = (int)((int64_t)cu[b + 1] - n0);
                } while (t >= seq_end_t);
                load_a();
            }
            // saliency: one float32 multiply, never fused
            uint32_t key[8];
            {
                const uint32_t xw[4] = {x[s].x, x[s].y, x[s].z, x[s].w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    key[2 * c] = __float_as_uint(__fmul_rn(a[2 * c], fabsf(__uint_as_float(xw[c] << 16))));
                    key[2 * c + 1] = __float_as_uint(__fmul_rn(a[2 * c + 1], fabsf(__uint_as_float(xw[c] & 0xFFFF0000u))));
                }
            }
            const uint32_t kmax = row16_max(max(max(max(key[0], key[1]), max(key[2], key[3])), max(max(key[4], key[5]), max(key[6], key[7]))));
            const int emax = max((int)(kmax >> 23), 1);
            // Bins are laid out from the top of the largest key's octave down: bin (top - key) >> 20 holds an eighth of
            // an octave.
            const uint32_t top = kmax | 0x7FFFFFu;
            uint32_t q[8], total = 0;
            // In units of the largest key's last place, rounded down: a product with a power of two, which is exact, and a
            // conversion that cuts off.  (Rows whose largest key is too small for that power, and keys that are no numbers, are
            // taken apart instead.)
            const bool plain = __ballot(kmax - (24u << 23) >= (255u - 24u) << 23) == 0ull;
            const float unit = __uint_as_float((uint32_t)(277 - emax) << 23);
            auto units_of = [&](uint32_t bits) __attribute__((always_inline)) {
                uint32_t u;
                if (__builtin_expect(plain, 1)) u = (uint32_t)(__uint_as_float(bits) * unit); else u = quantise(bits, emax);
                return u;
            };
            if (__builtin_expect(plain, 1)) {
#pragma unroll
                for (int c = 0; c < 8; ++c) q[c] = (uint32_t)(__uint_as_float(key[c]) * unit);
            } else {
#pragma unroll
                for (int c = 0; c < 8; ++c) q[c] = quantise(key[c], emax);
            }
            uint4 *const my_bins = reinterpret_cast<uint4 *>(hist + kBinsPerLane * sub);
            my_bins[0] = my_bins[1] = make_uint4(0u, 0u, 0u, 0u);
            prune_lds_sync();
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const uint32_t bin = min(top - key[c], below) >> 20;
                uint32_t at;
                asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(at) : "v"(bin), "v"(hist_a));     // (written out: the compiler takes one more)
                __hip_atomic_fetch_add(lds_word(at), q[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                total += q[c];
            }
            prune_lds_sync();
            const uint4 b0 = my_bins[0], b1 = my_bins[1];
            prune_lds_sync();
            total = row16_sum(total);
            const uint32_t bins[kBinsPerLane] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            const uint32_t mine = ((b0.x + b0.y) + (b0.z + b0.w)) + ((b1.x + b1.y) + (b1.z + b1.w));
            // need = ceil(total * p / 10000) without a 64-bit division: total = 10000 A + B (A < 2^18, B * p < 2^27)
            const uint32_t tA = total / 10000u, tB = total - __umul24(tA, 10000u);
            const uint32_t need = __umul24(tA, (uint32_t)p_bp) + (__umul24(tB, (uint32_t)p_bp) + 9999u) / 10000u;
            uint32_t n, above;                       // above: sum over the keys >= hi
            find_bin<kBinsPerLane>(bins, row16_inclusive_sum(mine) - mine, need, n, above);
            uint32_t hi = top - (n << 20) + 1u;
            // Where four or more keys of the bin are needed it is cut into 64 finer ones (at most three times).  (A row
            // whose sum lies below all the bins comes here with every key below them undecided: a cut then takes
            // off an eighth of an octave at most, and the rest is done key by key.)
            const uint32_t four_keys = 3u << 24 >> (n >> 3);       // (a key of the bin is worth less than a third of it)
#pragma nounroll
            for (int sh = 14; sh > 0; sh -= 6) {
                if (__builtin_expect(__ballot(need - above >= four_keys) == 0ull, 1)) break;
                *reinterpret_cast<uint4 *>(hist + 4 * sub) = make_uint4(0u, 0u, 0u, 0u);
                prune_lds_sync();
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const uint32_t i = (hi - 1u - key[c]) >> sh;      // (keys >= hi wrap round)
                    if (i < 64u) atomicAdd(&hist[i], q[c]);
                }
                prune_lds_sync();
                const uint4 v = *reinterpret_cast<const uint4 *>(hist + 4 * sub);
                prune_lds_sync();
                const uint32_t fine[4] = {v.x, v.y, v.z, v.w};
                const uint32_t sum4 = v.x + v.y + v.z + v.w;
                uint32_t n2, more;
                find_bin<4>(fine, row16_inclusive_sum(sum4) - sum4, need - above, n2, more);
                hi -= n2 << sh;
                above += more;
            }
            // The keys below hi, largest first, until `need` is reached: theta is the smallest kept one.
            uint32_t theta, q_theta;
            int n_eq;                // keys == theta of the four rows (4: no ties)
            for (int it = 0;; ++it) {
                uint32_t dist[8], upper = hi - 1u;
                asm("" : "+v"(upper));               // (a value of its own: one subtraction per key, nothing kept for it)
#pragma unroll
                for (int c = 0; c < 8; ++c) dist[c] = upper - key[c];        // (keys >= hi wrap round)
                theta = upper - row16_min(min8(dist));
                q_theta = units_of(theta);
                n_eq = 0;
#pragma unroll
                for (int c = 0; c < 8; ++c) n_eq += __popcll(__ballot(key[c] == theta));
                const bool open = above + q_theta < need;
                if (__builtin_expect(__ballot(open) == 0ull || it == SPARK_D, 1)) break;    // (a row has 128 keys)
                uint32_t all = above + q_theta;
                if (__builtin_expect(n_eq != 4, 0)) {
                    uint32_t eq = 0;
#pragma unroll
                    for (int c = 0; c < 8; ++c) eq += key[c] == theta ? 1u : 0u;
                    all = above + row16_sum(eq) * q_theta;
                    if (__ballot(open && all < need) == 0ull) break;
                }
                const bool further = open && all < need;
                above = further ? all : above;
                hi = further ? theta : hi;
            }
            // kept: keys > theta, and of those == theta as many as it takes, lowest channels first
            uint64_t kb[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) kb[c] = __ballot(key[c] >= theta);
            if (__builtin_expect(n_eq != 4, 0)) {
                uint32_t eq = 0;
#pragma unroll
                for (int c = 0; c < 8; ++c) eq += key[c] == theta ? 1u : 0u;
                const uint32_t eq_upto = row16_inclusive_sum(eq), eq_row = row16_last(eq_upto);
                uint32_t n_tie = 1, acc = above + q_theta, rank = eq_upto - eq;
                while (acc < need && n_tie < eq_row) {
                    acc += q_theta;
                    ++n_tie;
                }
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const bool tied = key[c] == theta;
                    kb[c] = __ballot(key[c] > theta || (tied && rank < n_tie));
                    rank += tied ? 1u : 0u;
                }
            }
            const uint32_t m = byte_of_masks(kb);
            const uint32_t cnt = row16_sum((uint32_t)__popc(m));
            const uint32_t psum = __float_as_uint(row16_sum_f32(sum_pruned(kb, key)));
            masks |= (t < nvalid ? m : 0u) << (8 * s);       // (rows past the last token: empty mask)
            if (sub == s) {
                my_mu = psum;
                my_cnt = cnt;
            }
        }
    }

    // ---- the rows' fixed part (rows past the last token: mean 0, count 0).  The mask bytes are put in order in LDS.
    prune_lds_sync();
#pragma unroll
    for (int s = 0; s < kSteps; ++s) reinterpret_cast<uint8_t *>(wave_lds)[64 * s + lane] = (uint8_t)(masks >> (8 * s));
    prune_lds_sync();
    uint32_t *const mask_out = reinterpret_cast<uint32_t *>(tile_out) + t0 * 4 + lane;
    if constexpr (SAME_LAUNCH) dir_store(mask_out, wave_lds[lane]); else *mask_out = wave_lds[lane];
    prune_lds_sync();
    const int t = t0 + 4 * sub + row;
    const bool valid = sub < kSteps && t < nvalid;
    if (sub < kSteps) {
        const float mu = my_cnt < SPARK_D ? __uint_as_float(my_mu) / (float)(SPARK_D - my_cnt) : 0.0f;
        uint64_t *const fixed_out = reinterpret_cast<uint64_t *>(tile_out + 1024 + t * 8);
        const uint64_t fixed = valid ? (uint64_t)__float_as_uint(mu) | ((uint64_t)my_cnt << 32) : 0ull;
        if constexpr (SAME_LAUNCH) __hip_atomic_store(fixed_out, fixed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); else *fixed_out = fixed;
    }
    // (every row rounded up to a whole word)
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(valid ? (my_cnt + 1u) / 2u : 0u), 63);
}

// The dense rows of a tile that are to be written, requested: sixteen a wavefront, rows past the last token repeat it.
__device__ __forceinline__ void request_rows(const uint16_t *__restrict__ k, int64_t k_tok_stride, int64_t k_head_stride, const SparkLayout &L,
                                             int h, int64_t tile, uint4 (&x)[kSteps])
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n0 = tile * SPARK_TILE_TOKENS;
    const int64_t left = L.total_tokens - n0;
    const int nvalid = left < SPARK_TILE_TOKENS ? (int)left : SPARK_TILE_TOKENS;
    const uint16_t *kbase = k + n0 * k_tok_stride + (int64_t)h * k_head_stride + 8 * (lane & 15);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        const int t = wave * kRowsPerWave + 4 * s + (lane >> 4);
        x[s] = *reinterpret_cast<const uint4 *>(kbase + (int64_t)(t < nvalid ? t : nvalid - 1) * k_tok_stride);
    }
}

// Writes the kept entries (rows in x) of a tile whose rows have been selected, by any block, to its place in the head's
// stream: every lane finds the slots of its eight channels from the row's mask byte, the entries of sixteen rows are put
// together in LDS and leave as whole words.  `sum`: words of all tiles up to it.
template <bool SAME_LAUNCH>
__device__ __forceinline__ void write_tile(const uint4 (&x)[kSteps], uint8_t *__restrict__ packed, const SparkLayout &L, int h, int64_t tile,
                                           uint32_t sum, uint32_t *wave_lds)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane >> 4, sub = lane & 15;
    const int t0 = wave * kRowsPerWave;
    if (t0 >= L.total_tokens - tile * SPARK_TILE_TOKENS) return;       // (no block barrier is used)
    const uint8_t *tp = packed + L.off_tiles + ((int64_t)h * L.n_tiles + tile) * L.tile_bytes;
    const uint32_t *const mask_in = reinterpret_cast<const uint32_t *>(tp) + t0 * 4 + lane;
    const uint32_t *const cnt_in = reinterpret_cast<const uint32_t *>(tp + 1024 + lane * 8 + 4);
    const uint32_t word_of_mask = SAME_LAUNCH ? dir_load(mask_in) : *mask_in, cnt = SAME_LAUNCH ? dir_load(cnt_in) : *cnt_in;
    prune_lds_sync();
    wave_lds[lane] = word_of_mask;
    prune_lds_sync();
    uint32_t m[kSteps];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) m[s] = reinterpret_cast<const uint8_t *>(wave_lds)[64 * s + lane];   // (past the last token: empty)
    prune_lds_sync();
    const uint32_t upto = wave_inclusive_sum((cnt + 1u) / 2u);       // lane = token: words of the tile's rows 0 .. token
    const uint32_t base = sum - (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    const uint32_t first = t0 ? (uint32_t)__builtin_amdgcn_readlane((int)upto, t0 - 1) : 0u;
    const uint32_t nwords = (uint32_t)__builtin_amdgcn_readlane((int)upto, t0 + kRowsPerWave - 1) - first;
    const uint32_t stage_a = lds_address(wave_lds);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        const int t = t0 + 4 * s + row;
        const uint32_t last = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * t, (int)upto) - first - 1u;    // the row's last word
        const uint32_t kept = (uint32_t)__popc(m[s]);
        const uint32_t kept_upto = row16_inclusive_sum(kept), kept_row = row16_last(kept_upto);
        // (its upper half stays 0 where the count is odd; the entries are stored after it)
        if (sub == 0 && kept_row != 0u) *lds_word(stage_a + 4u * last) = 0u;
        prune_lds_sync();
        stage_kept(m[s], stage_a + 4u * (last + 1u) - 2u * (kept_row + (kept_row & 1u)) + 2u * kept_upto, x[s]);
    }
    prune_lds_sync();
    uint32_t *dst = reinterpret_cast<uint32_t *>(packed + L.off_vals) + (int64_t)h * L.vals_head_words + base + first;
    for (uint32_t i = lane; i < nwords; i += 64) dst[i] = wave_lds[i];
}

// Blocks take tickets of their head in the order in which they start: ticket i selects tile i, files its words in the
// directory, and then writes the entries of tile i - lag, whose place in the stream is known by then as a rule; `lag` more
// tickets only write.  Every group-th ticket turns the words of the last `group` tiles into sums.
// Every wait ends, however few blocks are resident, because nobody waits for a block that may not have started: who makes sums
// waits for words that smaller tickets file before they wait for anything; who writes tile i - lag waits for a sum that a
// smaller ticket makes (group <= lag, or lag = 0 and group = 1: its own).
// (A directory entry is read by few: a line that many ask for is handed out about every 10 ns.  Every block adding up its own
// place from the entries before it: 133 us instead of the 87 us of 65536 tokens x 8 heads.)
__global__ __launch_bounds__(kWaves * 64, 7) void spark_topp_prune_kernel(
    const uint16_t *__restrict__ k, int64_t k_tok_stride, int64_t k_head_stride, const int32_t *__restrict__ cu,
    uint8_t *__restrict__ packed, SparkLayout L, int p_bp, int lag, int group)
{
    // per wavefront: counting bins of four rows, or the kept entries of sixteen
    __shared__ __align__(16) uint32_t lds_all[kWaves][kRowsPerWave * SPARK_D / 2];
    static_assert(4 * kBinStride <= kRowsPerWave * SPARK_D / 2, "one area for both");
    __shared__ uint32_t words_of_wave[kWaves];
    __shared__ uint32_t ticket, sum_of_late;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = (int)(blockIdx.x % (uint32_t)L.n_kv_heads);
    uint32_t *const dir = reinterpret_cast<uint32_t *>(packed + L.off_dir) + (int64_t)h * (L.n_tiles + 1);
    if (blockIdx.x == 0 && threadIdx.x < 16) write_header(packed, L, p_bp);
    // The tickets are counted in the directory's first entry, which the last taker sets back to 0.
    if (threadIdx.x == 0) {
        const uint32_t t = __hip_atomic_fetch_add(dir, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((int64_t)t == L.n_tiles + lag - 1) dir_store(dir, 0u);
        ticket = t;
    }
    __syncthreads();
    const int64_t mine = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)ticket);
    uint32_t *const wave_lds = lds_all[wave];
    uint32_t words = 0;
    if (mine < L.n_tiles) words = select_tile<true>(k, k_tok_stride, k_head_stride, cu, packed, L, p_bp, h, mine, wave_lds);
    const int64_t late = mine - lag;                     // the tile to be written
    uint4 x[kSteps];
    if (late >= 0) request_rows(k, k_tok_stride, k_head_stride, L, h, late, x);
    uint32_t sum = 0;                                    // (wavefront 0: words of all tiles up to `late`)
    if (mine < L.n_tiles) {
        if (lane == 0) words_of_wave[wave] = words;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);         // the rows' fixed part has been acknowledged
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t all = 0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) all += words_of_wave[w];
            dir_store(dir + mine + 1, kOwnWords + all);
        }
        const int in_group = (int)(mine % group);
        if (wave == 0 && (in_group == group - 1 || mine == L.n_tiles - 1)) {
            uint32_t after;
            sum = words_up_to(dir, mine + 1, lane, after);
            if (lane <= in_group) dir_store(dir + mine + 1 - lane, sum - after);
        }
    }
    if (late < 0) return;
    // A sum that is there says that the tile's own block has filed its words, after its rows' fixed part had reached the
    // point where all the chip's caches agree.  (The tile's place is this sum less its own words: the entry in front may
    // still be on its way when this one is there.)  One wavefront asks for all four, and not too often: what many ask for
    // at a time comes late.
    if (wave == 0) {
        if (late != mine) {
            for (;;) {
                sum = (uint32_t)__builtin_amdgcn_readfirstlane((int)dir_load(dir + late + 1));
                if (sum != 0u && sum < kOwnWords) break;
                __builtin_amdgcn_s_sleep(8);
            }
        }
        if (lane == 0) sum_of_late = sum;
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    write_tile<true>(x, packed, L, h, late, (uint32_t)__builtin_amdgcn_readfirstlane((int)sum_of_late), wave_lds);
}

// ---- the same in three launches: selection (a block per tile), directory (a block per head), writing (a block per tile)

__global__ __launch_bounds__(kWaves * 64, 7) void spark_topp_select_kernel(
    const uint16_t *__restrict__ k, int64_t k_tok_stride, int64_t k_head_stride, const int32_t *__restrict__ cu,
    uint8_t *__restrict__ packed, SparkLayout L, int p_bp)
{
    __shared__ __align__(16) uint32_t hist_all[kWaves][4 * kBinStride];
    __shared__ uint32_t words_of_wave[kWaves];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = (int)(blockIdx.x / (uint32_t)L.n_tiles);
    const int64_t tile = blockIdx.x % (uint32_t)L.n_tiles;
    if (blockIdx.x == 0 && threadIdx.x < 16) write_header(packed, L, p_bp);
    const uint32_t words = select_tile<false>(k, k_tok_stride, k_head_stride, cu, packed, L, p_bp, h, tile, hist_all[wave]);
    if ((threadIdx.x & 63) == 0) words_of_wave[wave] = words;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t all = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) all += words_of_wave[w];
        reinterpret_cast<uint32_t *>(packed + L.off_dir)[(int64_t)h * (L.n_tiles + 1) + tile + 1] = all;
    }
}

// One block per KV head: dir[h][0] = 0, dir[h][t + 1] = words of tiles 0 .. t (they arrive as per-tile counts).
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void spark_topp_scan_kernel(uint8_t *__restrict__ packed, SparkLayout L)
{
    __shared__ uint32_t wave_sum[kScanThreads / 64];
    uint32_t *dir = reinterpret_cast<uint32_t *>(packed + L.off_dir) + (int64_t)blockIdx.x * (L.n_tiles + 1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n = L.n_tiles;
    if (threadIdx.x == 0) dir[0] = 0u;
    uint32_t run = 0;                                    // words of the tiles in front of this pass's
    for (int64_t i0 = 0; i0 < n; i0 += kScanThreads) {
        const int64_t i = i0 + threadIdx.x;
        const uint32_t upto = wave_inclusive_sum(i < n ? dir[i + 1] : 0u);
        if (lane == 63) wave_sum[wave] = upto;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kScanThreads / 64; ++w) {
            const uint32_t v = wave_sum[w];
            before += w < wave ? v : 0u;
            all += v;
        }
        if (i < n) dir[i + 1] = run + before + upto;
        run += all;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kWaves * 64) void spark_topp_pack_kernel(const uint16_t *__restrict__ k, int64_t k_tok_stride,
                                                                      int64_t k_head_stride, uint8_t *__restrict__ packed,
                                                                      SparkLayout L)
{
    __shared__ __align__(16) uint32_t stage_all[kWaves][kRowsPerWave * SPARK_D / 2];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = (int)(blockIdx.x / (uint32_t)L.n_tiles);
    const int64_t tile = blockIdx.x % (uint32_t)L.n_tiles;
    uint4 x[kSteps];
    request_rows(k, k_tok_stride, k_head_stride, L, h, tile, x);
    const uint32_t sum = reinterpret_cast<const uint32_t *>(packed + L.off_dir)[(int64_t)h * (L.n_tiles + 1) + tile + 1];
    write_tile<false>(x, packed, L, h, tile, sum, stage_all[wave]);
}

// canonical export, one thread per (token, KV head) row
__global__ void spark_topp_unpack_kernel(const uint8_t *__restrict__ packed, SparkLayout L, uint32_t *mask_out,
                                         int32_t *count_out, uint16_t *vals_out, float *mu_out, float *a_out)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t rows = L.total_tokens * L.n_kv_heads;
    if (a_out && idx < (int64_t)L.batch * L.n_kv_heads * SPARK_D)
        a_out[idx] = reinterpret_cast<const float *>(packed + L.off_a)[idx];
    if (idx >= rows) return;
    const int64_t n = idx / L.n_kv_heads;
    const int h = (int)(idx % L.n_kv_heads);
    const int64_t tile = n / SPARK_TILE_TOKENS;
    const int t = (int)(n % SPARK_TILE_TOKENS);
    const uint8_t *tp = packed + L.off_tiles + ((int64_t)h * L.n_tiles + tile) * L.tile_bytes;
    const uint32_t cnt = *reinterpret_cast<const uint32_t *>(tp + 1024 + t * 8 + 4);
    if (mask_out)
        for (int m = 0; m < 4; ++m) mask_out[idx * 4 + m] = *reinterpret_cast<const uint32_t *>(tp + t * 16 + m * 4);
    if (mu_out) mu_out[idx] = *reinterpret_cast<const float *>(tp + 1024 + t * 8);
    if (count_out) count_out[idx] = (int32_t)cnt;
    if (vals_out) {
        uint32_t before = 0;
        for (int u = 0; u < t; ++u) before += (*reinterpret_cast<const uint32_t *>(tp + 1024 + u * 8 + 4) + 1u) / 2u;
        const uint32_t base = reinterpret_cast<const uint32_t *>(packed + L.off_dir)[(int64_t)h * (L.n_tiles + 1) + tile];
        const uint32_t *src = reinterpret_cast<const uint32_t *>(packed + L.off_vals) + (int64_t)h * L.vals_head_words + base + before;
        uint16_t *o = vals_out + idx * SPARK_D;
        for (uint32_t i = 0; i < (uint32_t)SPARK_D; ++i)
            o[i] = i < cnt ? (uint16_t)((src[i >> 1] >> (16 * (i & 1))) & 0xFFFFu) : (uint16_t)0;
    }
}

// ---------------------------------------------------------------- host-side launch

// One launch or three.  In one, few tiles (lag 0: a block writes its own tile) save two launches, and many tiles (a lag of
// about as many as the chip has in flight) hide the writing, which waits for memory, behind the selection, which is bound
// by vector issue.  In between, where all blocks select at once and then all write, the way from a tile's words to its place
// (two trips through memory, or one for every 64 tiles of a head) costs more than the launches; and with few heads the count of
// the tickets (11.5 ns each) does.  Three launches / one (us, 51 kept channels a row, window kernel included):
//   8 heads, tiles:  64 17.8 / 15.3   256 18.0 / 17.1   512 20.2 / 27   1024 23.9 / 39   2048 35.6 / 34.3   4096 56.5 / 49.7   8192 96.3 / 84.2
//   1 head:  64 16.3 / 15.1   96 16.7 / 15.8   127 16.8 / 16.6   256 17.0 / 19.3   1024 24 / 63
//   2 heads:  128 16.5 / 15.8   192 16.9 / 16.4   224 17.1 / 17.2   254 16.8 / 17.4   2048 37 / 57
//   4 heads:  256 18.3 / 17.2   2048 35.8 / 35.6   4096 57.0 / 52.8   8192 98 / 87      16 heads:  4096 56.7 / 49.3
//   64 heads:  2048 36.0 / 32.8      1024 heads:  2048 41.0 / 34.5      4096 heads:  8192 129 / 111
// Heads of 67.1 million tokens and more, whose streams have room for kOwnWords words, take three: there the directory's words are
// sums only.
int topp_prune_launches(const SparkLayout &L)
{
    const int64_t tiles = L.n_tiles * L.n_kv_heads;
    if (tiles == 0) return 0;
    if (L.vals_head_words >= (int64_t)kOwnWords) return 3;
    return (tiles <= 256 && L.n_tiles <= 112) || (tiles >= 2048 && L.n_kv_heads >= 4) ? 1 : 3;
}

hipError_t launch_prune_topp(const uint16_t *k, int64_t k_tok_stride, int64_t k_head_stride, const int32_t *cu,
                             uint8_t *packed, const SparkLayout &L, int p_bp, hipStream_t st)
{
    if (L.n_tiles == 0) return hipSuccess;
    const int64_t tiles = L.n_tiles * L.n_kv_heads;
    const dim3 threads(kWaves * 64);
    if (topp_prune_launches(L) == 1) {
        const int lag = tiles <= 256 ? 0 : (L.n_kv_heads < 2048 ? 2048 / L.n_kv_heads : 1);
        const int group = lag < 4 ? 1 : (lag < 64 ? lag / 2 : 32);
        const int64_t tickets = L.n_tiles + lag;
        hipLaunchKernelGGL(spark_topp_prune_kernel, dim3((unsigned)(tickets * L.n_kv_heads)), threads, 0, st, k, k_tok_stride,
                           k_head_stride, cu, packed, L, p_bp, lag, group);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(spark_topp_select_kernel, dim3((unsigned)tiles), threads, 0, st, k, k_tok_stride, k_head_stride, cu, packed,
                       L, p_bp);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(spark_topp_scan_kernel, dim3(L.n_kv_heads), dim3(kScanThreads), 0, st, packed, L);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(spark_topp_pack_kernel, dim3((unsigned)tiles), threads, 0, st, k, k_tok_stride, k_head_stride, packed, L);
    return hipGetLastError();
}

hipError_t launch_unpack_topp(const uint8_t *packed, const SparkLayout &L, uint32_t *mask_out, int32_t *count_out,
                              uint16_t *vals_out, float *mu_out, float *a_out, hipStream_t st)
{
    int64_t n = L.total_tokens * L.n_kv_heads;
    const int64_t na = (int64_t)L.batch * L.n_kv_heads * SPARK_D;
    if (a_out && na > n) n = na;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(spark_topp_unpack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, packed, L, mask_out,
                       count_out, vals_out, mu_out, a_out);
    return hipGetLastError();
}

}  // namespace spark
