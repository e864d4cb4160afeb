// Decode attention for short calls on gfx950: sixteen tokens a wavefront, in blocks of SIXTEEN wavefronts, one per compute unit, or
// of FOUR, one per tile.
// (Included by spark_decode_kernel.h, whose parameter block, chunk numbering and partial slots it shares.)
//
// A short call is a chain of latencies; the longest was the walk of a lane over all kept entries of its row, one of 64 a
// wavefront takes (4 of the 10 us of 1024 tokens with 64 kept channels).  Here
//   rows     come as they are stored, 16 bytes a lane, and are parked in the wavefront's LDS;
//   scores   FOUR lanes a row, one mask word each: lane (tg, cn) walks word tg of row cn, a few entries at a time, and a
//            lane-swap reduction hands lane row tg the scores of query heads tg, 4 + tg.  Softmax: a row of sixteen lanes;
//   output   both bf16 parts of the probabilities side by side in one 16x16x32 product (K = 2 x 16 tokens);
//   merge    all wavefronts share the partials of the block that counts in last.
// Bound by the round trips (sequence table, rows, partial, count, merge) and, in blocks with four tiles, by the table
// gathers in the compute unit's LDS (24 to 36 cycles each), which a block per tile spreads over four times as many compute
// units.  What each takes and what it measured stand beside the rules: short_call_pays in spark_decode.hip (sixteen), fine_plan in
// spark_api.hip (four); 4 sequences of 700 to 3900 tokens with 256 appended rows each, eight query heads, by sixteen wavefronts: T = 30
// 18.0 -> 17.0 us, T = 127 29.2 -> 24.9 us; 1024 tokens, four query heads, T = 64, by a block per tile: 11.4 -> 9.7 us.  (128
// registers; four query heads spill 4 of them, eight spill 8.)
#pragma once

namespace spark {

constexpr int kShortRows = 16;          // tokens a wavefront takes at a time

template <int G, int INT8, int BW>
__global__ __launch_bounds__(BW * 64, 4) void spark_decode_short_kernel(DecodeParams P)
{
    static_assert(G <= 8, "eight query heads at most");
    static_assert(BW * kShortRows == (BW == 4 ? kFineTailRows : 256), "a block of appended rows is one pass");
    constexpr int GP = 8 * ((G + 1 + 3) / 8) + 4;                // floats per table entry (as in spark_decode_kernel)
    constexpr int NH = (G + 3) / 4;                              // query heads per lane row: tg, 4 + tg
    constexpr int kMaxSections = 18;                             // 16-byte sections of the longest row (128 entries, statistics)
    constexpr int kLoads = (kMaxSections + 3) / 4;
    constexpr int kEntries = G <= 4 ? 4 : 2;                     // walked at a time, bounded by registers
    // A row's stride is an odd number of sections.  A lane that is through with its entries reads on, 32 entries at most.
    constexpr int kRowWords = kShortRows * 4 * (kMaxSections | 1) + 20;
    static_assert(kRowWords >= G * SPARK_D && kRowWords % 4 == 0, "accumulators fit, 16-byte aligned");

    __shared__ __align__(16) float qt[SPARK_D * GP];
    __shared__ __align__(16) uint32_t area[BW][kRowWords];       // rows, then the accumulators
    __shared__ __align__(16) uint16_t pbuf[BW][G][32];           // two parts of the probabilities
    __shared__ __align__(16) uint16_t pthird[BW][G][16];         // the third one (appended rows)
    __shared__ float red_m[BW][G], red_l[BW][G];
    __shared__ int last_flag;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tg = lane >> 4, cn = lane & 15;
    if (P.trace != nullptr) {
        stamp(P, 0, wall_clock64());
        stamp(P, 6, ((unsigned long long)__builtin_amdgcn_s_getreg(20 | (31 << 11)) << 32) |     // XCC_ID
                        (unsigned long long)__builtin_amdgcn_s_getreg(4 | (31 << 11)));              // HW_ID
        stamp(P, 7, 0ull);
    }
    const SparkLayout &L = P.L;
    const int nmain = P.nchunk_max * P.Hkv;
    const bool is_tail = (int)blockIdx.x >= nmain;               // block-uniform
    const int tb = (int)blockIdx.x - nmain;
    const int gid = is_tail ? -1 : (int)(blockIdx.x / P.Hkv);
    const int h = is_tail ? (tb / P.ntail) % P.Hkv : (int)(blockIdx.x % P.Hkv);
    const int tail_b = is_tail ? (tb / P.ntail) / P.Hkv : -1;
    int tail_rows = is_tail ? P.tail_len[tail_b] : 0;
    const SeqChunks sc = locate_chunks(P, L.batch, gid, tail_b, lane);
    if (sc.n == 0) return;                                       // past the last chunk: the whole block leaves
    const int b = sc.b, nmerge = sc.n + P.ntail;

    f32x4 acc[8];                        // head 4 tg + r, channel 8 cn + e
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 vx[4];                         // rows 4 i + tg, channels 8 cn .. 8 cn + 7
    // B operand e: channel 8 cn + e of the four rows, twice (one half of K for each part of the probabilities)
    auto add_output = [&](const bf16x8 &A, const bf16x8 *A2) __attribute__((always_inline)) {
#pragma unroll
        for (int cp = 0; cp < 4; ++cp) {
            const uint32_t x0 = u4c(vx[0], cp), x1 = u4c(vx[1], cp), x2 = u4c(vx[2], cp), x3 = u4c(vx[3], cp);
            const uint32_t e0 = __builtin_amdgcn_perm(x1, x0, 0x05040100u), e1 = __builtin_amdgcn_perm(x3, x2, 0x05040100u);
            const uint32_t o0 = __builtin_amdgcn_perm(x1, x0, 0x07060302u), o1 = __builtin_amdgcn_perm(x3, x2, 0x07060302u);
            const bf16x8 even = __builtin_bit_cast(bf16x8, u32x4{e0, e1, e0, e1}), odd = __builtin_bit_cast(bf16x8, u32x4{o0, o1, o0, o1});
            if (A2 != nullptr) {                                 // (small parts first)
                acc[2 * cp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*A2, even, acc[2 * cp], 0, 0, 0);
                acc[2 * cp + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*A2, odd, acc[2 * cp + 1], 0, 0, 0);
            }
            acc[2 * cp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, even, acc[2 * cp], 0, 0, 0);
            acc[2 * cp + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, odd, acc[2 * cp + 1], 0, 0, 0);
        }
    };
    auto row16_max_f32 = [](float x) __attribute__((always_inline)) {
        x = dpp_max_step<0x128, 0xF>(x);
        x = dpp_max_step<0x124, 0xF>(x);
        x = dpp_max_step<0x122, 0xF>(x);
        return dpp_max_step<0x121, 0xF>(x);
    };
    auto row16_add_f32 = [](float x) __attribute__((always_inline)) {
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, true));
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, true));
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xF, 0xF, true));
        return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xF, 0xF, true));
    };
    // place of token cn = 4 i + tg' in a probability operand: K = 8 tg' + i (+ 4: the second part)
    const int ppos = 8 * (cn & 3) + (cn >> 2);

    if (!is_tail) {
        const int s0 = sc.s0, s1 = sc.s1, split = gid - sc.first;
        // parts (sixteen tokens) of this block's chunk: the tiles are cut as for spark_decode_kernel
        int p_begin = 0, p_end = 0;
        if (s1 > s0) {
            const int tf = s0 / SPARK_TILE_TOKENS, tl = (s1 - 1) / SPARK_TILE_TOKENS;
            const int chunk = (tl - tf + sc.n) / sc.n;           // ceil((tl - tf + 1) / n)
            p_begin = max(4 * (tf + split * chunk), s0 / kShortRows);
            p_end = min(4 * (tf + (split + 1) * chunk), (s1 - 1) / kShortRows + 1);
        }
        float inva_r = 0.0f;
        uint16_t q_r[G];
        if (tid < SPARK_D) {
            inva_r = reinterpret_cast<const float *>(P.packed + L.off_inva)[((int64_t)b * P.Hkv + h) * SPARK_D + tid];
#pragma unroll
            for (int g = 0; g < G; ++g) q_r[g] = P.q[((int64_t)b * P.Hq + h * G + g) * SPARK_D + tid];
        }
        const uint8_t *tiles = P.packed + L.off_tiles + (int64_t)h * L.n_tiles * L.tile_bytes;
        const uint16_t *vbase = P.v + (int64_t)h * P.v_head_stride + cn * 8;
        const int nsec = L.nq + L.tail2, sw = 4 * (nsec | 1);
        u32x4 x[kLoads];                 // section 4 u + tg of row cn
        auto load_row = [&](int part) __attribute__((always_inline)) {
            const uint8_t *tp = tiles + (int64_t)(part >> 2) * L.tile_bytes;
            const int t = (part & 3) * kShortRows + cn;
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int qd = 4 * u + tg;
                if (4 * u < nsec) {                              // (wave-uniform)
                    if (qd < L.nq) {
                        x[u] = *reinterpret_cast<const u32x4 *>(tp + qd * 1024 + t * 16);
                    } else if (qd < nsec) {                      // the 2-word section at the end of the row
                        const uint2 y = *reinterpret_cast<const uint2 *>(tp + L.nq * 1024 + t * 8);
                        x[u] = u32x4{y.x, y.y, 0u, 0u};
                    }
                }
            }
        };
        auto load_v = [&](int part) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int n = part * kShortRows + 4 * i + tg;          // (rows outside the sequence get p = 0)
                n = min(max(n, s0), s1 - 1);
                vx[i] = *reinterpret_cast<const uint4 *>(vbase + (int64_t)n * P.v_tok_stride);
            }
        };
        int part = p_begin + wave;
        if (part < p_end) {
            load_row(part);
            load_v(part);
        }
        if (tid < SPARK_D) {
#pragma unroll
            for (int g = 0; g < G; ++g) qt[tid * GP + g] = bf16lo(q_r[g]) * P.scale_log2;
            qt[tid * GP + G] = inva_r;
        }
        __syncthreads();
        float m[NH], l[NH], R[NH];       // of head 4 i + tg
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            m[i] = -INFINITY;
            l[i] = 0.0f;
            float r = 0.0f;
            const int g = min(4 * i + tg, G - 1);
#pragma unroll
            for (int k = 0; k < 8; ++k) r += qt[(cn + 16 * k) * GP + g] * qt[(cn + 16 * k) * GP + G];
            R[i] = row16_add_f32(r);
        }
        if (P.trace != nullptr) { stamp(P, 1, wall_clock64()); stamp(P, 5, (unsigned long long)((p_end - p_begin + 3) / 4)); }
        uint32_t *const rows = area[wave];
        const uint32_t *const row = rows + cn * sw;
        for (; part < p_end; part += BW) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u)
                if (4 * u + tg < nsec) *reinterpret_cast<u32x4 *>(&rows[cn * sw + 4 * (4 * u + tg)]) = x[u];
            const bool more = part + BW < p_end;        // (wave-uniform)
            if (more) load_row(part + BW);
            wave_lds_sync();
            // ---- scores: this lane's mask word of its row, a few entries at a time
            const u32x4 mk = *reinterpret_cast<const u32x4 *>(row);
            uint32_t left = row[tg];
            const float mu = __uint_as_float(row[4]);
            const float scale_row = INT8 ? __uint_as_float(row[5]) : 1.0f;
            const int before = (tg > 0 ? __popc(mk.x) : 0) + (tg > 1 ? __popc(mk.y) : 0) + (tg > 2 ? __popc(mk.z) : 0);
            const uint8_t *pv = reinterpret_cast<const uint8_t *>(row + L.val0) + (INT8 ? before : 2 * before);
            const float *const qw = qt + 32 * tg * GP;
            float s[4 * NH];
#pragma unroll
            for (int g = 0; g < 4 * NH; ++g) s[g] = 0.0f;
            while (__ballot(left != 0u) != 0ull) {
                float ev[kEntries][G + 1], kv[kEntries];
                bool on[kEntries];
#pragma unroll
                for (int u = 0; u < kEntries; ++u) {
                    on[u] = left != 0u;
                    const float *e = qw + __builtin_ctz(left | 0x80000000u) * GP;
                    left &= left - 1u;
#pragma unroll
                    for (int g = 0; g <= G; ++g) ev[u][g] = e[g];
                    kv[u] = INT8 ? (float)(int)reinterpret_cast<const int8_t *>(pv)[u] * scale_row
                                 : __uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(pv)[u] << 16);
                }
                pv += INT8 ? kEntries : 2 * kEntries;
#pragma unroll
                for (int u = 0; u < kEntries; ++u) {
                    const float d = on[u] ? fmaf(-mu, ev[u][G], kv[u]) : 0.0f;
#pragma unroll
                    for (int g = 0; g < G; ++g) s[g] = fmaf(ev[u][g], d, s[g]);
                }
            }
            // ---- online softmax (log2 domain): lane row tg = query heads tg, 4 + tg, lane cn = token
            const int n = part * kShortRows + cn;
            const bool valid = n >= s0 && n < s1;
            float alpha[NH];
            bool moved = false;
#pragma unroll
            for (int i = 0; i < NH; ++i) {
                float v = reduce_scatter_rows(s[4 * i], s[4 * i + 1], s[4 * i + 2], s[4 * i + 3]);
                v = valid ? fmaf(mu, R[i], v) : -INFINITY;
                const float mnew = fmaxf(m[i], row16_max_f32(v));
                const float msafe = (mnew == -INFINITY) ? 0.0f : mnew;
                alpha[i] = fast_exp2(m[i] - msafe);              // m = -inf -> 0
                moved = moved || mnew != m[i];
                m[i] = mnew;
                const float p = fast_exp2(v - msafe);            // v = -inf -> 0
                l[i] = fmaf(l[i], alpha[i], p);
                const __bf16 ph = (__bf16)p;
                const __bf16 pl = (__bf16)(p - (float)ph);
                if (4 * i + tg < G) {
                    pbuf[wave][4 * i + tg][ppos] = __builtin_bit_cast(uint16_t, ph);
                    pbuf[wave][4 * i + tg][ppos + 4] = __builtin_bit_cast(uint16_t, pl);
                }
            }
            if (__ballot(moved) != 0ull) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float al = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha[0]), 16 * r));
                    if constexpr (NH > 1) {
                        const float al1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha[NH - 1]), 16 * r));
                        al = tg == 0 ? al : al1;
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e][r] *= al; // (rows without a query head stay 0)
                }
            }
            wave_lds_sync();
            uint4 a = {0, 0, 0, 0};
            if (cn < G) a = *reinterpret_cast<const uint4 *>(&pbuf[wave][cn][8 * tg]);
            add_output(__builtin_bit_cast(bf16x8, a), nullptr);
            if (more) load_v(part + BW);
            wave_lds_sync();             // rows and probabilities are rewritten by the next pass
        }
        if (P.trace != nullptr) stamp(P, 2, wall_clock64());
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            const float lt = row16_add_f32(l[i]);
            if (cn == 0 && 4 * i + tg < G) { red_m[wave][4 * i + tg] = m[i]; red_l[wave][4 * i + tg] = lt; }
        }
    } else {
        // ---- appended rows, sixteen a wavefront: as in tail_partial
        float s_scale;
        uint4 qx[4];
        bf16x8 Aq[4];
        tail_query_rows<G>(P, b, h, cn, tg, qx);
        const float q_scale = split_scale(P.scale_log2, s_scale);
        tail_rows = tail_rows < 0 ? 0 : (tail_rows > P.tail_cap ? P.tail_cap : tail_rows);
        const int c0 = (tb % P.ntail) * (BW * kShortRows) + wave * kShortRows;
        const int nval = min(tail_rows - c0, kShortRows);
        float m[4], l[4];                // of head 4 tg + r
#pragma unroll
        for (int r = 0; r < 4; ++r) { m[r] = -INFINITY; l[r] = 0.0f; }
        if (P.trace != nullptr) { stamp(P, 1, wall_clock64()); stamp(P, 5, 0ull); }
        if (nval > 0) {                  // (wave-uniform); rows past the last one: the last one
            const int64_t row0 = ((int64_t)b * P.tail_cap + c0) * P.Hkv + h, step = P.Hkv;
            uint4 kx[4];
            const uint16_t *krow = P.tail_k + (row0 + (int64_t)min(cn, nval - 1) * step) * SPARK_D + 8 * tg;
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) kx[kb] = *reinterpret_cast<const uint4 *>(krow + 32 * kb);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                vx[i] = *reinterpret_cast<const uint4 *>(P.tail_v + (row0 + (int64_t)min(4 * i + tg, nval - 1) * step) * SPARK_D + 8 * cn);
            f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                tail_query_operand<G>(qx[kb], cn, q_scale, Aq[kb]);
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Aq[kb], __builtin_bit_cast(bf16x8, kx[kb]), s, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = cn < nval ? s[r] * s_scale : -INFINITY;
                m[r] = row16_max_f32(v);                         // finite: row 0 is there
                const float p = fast_exp2(v - m[r]);
                l[r] = p;
                // three parts of eight bits each, cut off: exactly p
                const float hi = __uint_as_float(__float_as_uint(p) & 0xFFFF0000u), rest = p - hi;
                const float mid = __uint_as_float(__float_as_uint(rest) & 0xFFFF0000u), lo = rest - mid;
                const int g = 4 * tg + r;
                if (g < G) {
                    pbuf[wave][g][ppos] = (uint16_t)(__float_as_uint(hi) >> 16);
                    pbuf[wave][g][ppos + 4] = (uint16_t)(__float_as_uint(mid) >> 16);
                    pthird[wave][g][4 * (cn & 3) + (cn >> 2)] = (uint16_t)(__float_as_uint(lo) >> 16);
                }
            }
            wave_lds_sync();
            uint4 a = {0, 0, 0, 0}, third = {0, 0, 0, 0};
            if (cn < G) {
                a = *reinterpret_cast<const uint4 *>(&pbuf[wave][cn][8 * tg]);
                const uint2 y = *reinterpret_cast<const uint2 *>(&pthird[wave][cn][4 * tg]);
                third.x = y.x;
                third.y = y.y;
            }
            const bf16x8 A2 = __builtin_bit_cast(bf16x8, third);
            add_output(__builtin_bit_cast(bf16x8, a), &A2);
            tail_infinite_values(P.tail_v + row0 * SPARK_D + 8 * cn, step * SPARK_D, nval,
                                 [&](int n) __attribute__((always_inline)) {
                                     const int at = 8 * (n & 3) + (n >> 2);
                                     f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                                     for (int r = 0; r < 4; ++r) {
                                         const int g = 4 * tg + r;
                                         if (g < G)
                                             p[r] = (bf16lo(pbuf[wave][g][at]) + bf16lo(pbuf[wave][g][at + 4])) +
                                                    bf16lo(pthird[wave][g][4 * (n & 3) + (n >> 2)]);
                                     }
                                     return p;
                                 }, acc);
        }
        if (P.trace != nullptr) stamp(P, 2, wall_clock64());
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float lt = row16_add_f32(l[r]);
            if (cn == 0 && 4 * tg + r < G) { red_m[wave][4 * tg + r] = m[r]; red_l[wave][4 * tg + r] = lt; }
        }
    }

    // ---- merge the wavefronts, write the partial
    {
        float *mine = reinterpret_cast<float *>(area[wave]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * tg + r < G) {
#pragma unroll
                for (int e = 0; e < 8; e += 4)
                    *reinterpret_cast<f32x4 *>(&mine[(4 * tg + r) * SPARK_D + 8 * cn + e]) = f32x4{acc[e][r], acc[e + 1][r], acc[e + 2][r], acc[e + 3][r]};
            }
    }
    __syncthreads();
    auto store_out = [&](int g, int ch, float A, float Lsum) __attribute__((always_inline)) {
        const float o = (Lsum > 0.0f) ? (A / Lsum) : 0.0f;
        const int64_t oi = ((int64_t)b * P.Hq + h * G + g) * SPARK_D + ch;
        if (P.out_f32)
            reinterpret_cast<float *>(P.out)[oi] = o;
        else
            reinterpret_cast<uint16_t *>(P.out)[oi] = __builtin_bit_cast(uint16_t, (__bf16)o);
    };
    // partial slot of (query head of the pair, i-th partial)
    auto slot_of = [&](int g, int i) -> int64_t {
        return i < sc.n ? (int64_t)(sc.first + i) * P.Hq + h * G + g
                        : P.tail_base + ((int64_t)b * P.Hq + h * G + g) * P.tail_slots + (i - sc.n);
    };
    for (int idx = tid; idx < G * SPARK_D; idx += BW * 64) {
        const int g = idx / SPARK_D, ch = idx % SPARK_D;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < BW; ++w) M = fmaxf(M, red_m[w][g]);
        const float Ms = (M == -INFINITY) ? 0.0f : M;
        float Lsum = 0.0f, A = 0.0f;
#pragma unroll
        for (int w = 0; w < BW; ++w) {
            const float f = fast_exp2(red_m[w][g] - Ms);
            Lsum = fmaf(red_l[w][g], f, Lsum);
            A = fmaf(reinterpret_cast<const float *>(area[w])[g * SPARK_D + ch], f, A);
        }
        if (nmerge == 1) {               // the only block of this (batch, KV head)
            store_out(g, ch, A, Lsum);
        } else {
            const int64_t slot = slot_of(g, is_tail ? sc.n + tb % P.ntail : gid - sc.first);
            st_agent(&P.part_acc[slot * SPARK_D + ch], A);
            if (ch == 0) { st_agent(&P.part_ml[slot * 2], M); st_agent(&P.part_ml[slot * 2 + 1], Lsum); }
        }
    }
    if (P.trace != nullptr) { const unsigned long long now = wall_clock64(); stamp(P, 3, now); stamp(P, 4, now); }
    if (nmerge == 1) return;             // (block-uniform)

    // ---- the last block of this (batch, KV head) to get here merges: stores acknowledged, then counted (see
    // spark_decode_kernel).  A wavefront folds every (BW / G)-th partial of one query head, or all partials of some heads.
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
    if (tid == 0) {
        const uint32_t old = atomicInc(&P.counters[(b * P.Hkv + h) * P.counter_stride], (uint32_t)(nmerge - 1));
        last_flag = (old == (uint32_t)(nmerge - 1));
    }
    __syncthreads();
    if (P.trace != nullptr) stamp(P, 4, wall_clock64());
    if (!last_flag) return;
    {
        constexpr int kShare = BW > G ? BW / G : 1, kHeads = BW < G ? G / BW : 1;       // wavefronts per query head, heads per wavefront
        constexpr int RN = BW == 4 ? 32 : 16;                    // partials in flight
#pragma unroll 1
        for (int hd = 0; hd < kHeads; ++hd) {
            const int g = (wave + BW * hd) % G, first = wave / G;
            const uint64_t *pa = reinterpret_cast<const uint64_t *>(P.part_acc + 2 * lane);
            const uint64_t *pm = reinterpret_cast<const uint64_t *>(P.part_ml);
            float M = -INFINITY, Lsum = 0.0f, A0 = 0.0f, A1 = 0.0f;
            for (int i0 = first; i0 < nmerge; i0 += RN * kShare) {
                const int left = (nmerge - i0 + kShare - 1) / kShare, nn = left < RN ? left : RN;
                float mi = -INFINITY, li = 0.0f;
                if (lane < nn) {
                    const uint64_t ml = __hip_atomic_load(pm + slot_of(g, i0 + kShare * lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    mi = __uint_as_float((uint32_t)ml);
                    li = __uint_as_float((uint32_t)(ml >> 32));
                }
                uint64_t av[RN];
#pragma unroll
                for (int k = 0; k < RN; ++k) {                       // (past the end: the last one, its factor is 0)
                    const int i = i0 + kShare * (k < nn ? k : nn - 1);
                    av[k] = k < nn ? __hip_atomic_load(pa + slot_of(g, i) * (SPARK_D / 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
                }
                const float Mn = fmaxf(M, wave_max(mi));
                const float Ms = (Mn == -INFINITY) ? 0.0f : Mn;
                const float fo = fast_exp2(M - Ms), fi = fast_exp2(mi - Ms);
                M = Mn;
                Lsum = fmaf(Lsum, fo, wave_sum(li * fi));
                A0 *= fo;
                A1 *= fo;
#pragma unroll
                for (int k = 0; k < RN; ++k) {
                    const float f = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fi), k));
                    A0 = fmaf(__uint_as_float((uint32_t)av[k]), f, A0);
                    A1 = fmaf(__uint_as_float((uint32_t)(av[k] >> 32)), f, A1);
                }
            }
            // (accumulators of the block's own wavefronts have been read by all: two barriers ago)
            reinterpret_cast<float2 *>(area[wave])[hd * (SPARK_D / 2) + lane] = make_float2(A0, A1);
            if (lane == 0) { red_m[wave][hd] = M; red_l[wave][hd] = Lsum; }
        }
        __syncthreads();
        for (int idx = tid; idx < G * SPARK_D; idx += BW * 64) {
            const int gg = idx / SPARK_D, ch = idx % SPARK_D, w0 = gg % BW, hd = gg / BW;
            float Mx = -INFINITY;
#pragma unroll
            for (int k = 0; k < kShare; ++k) Mx = fmaxf(Mx, red_m[w0 + G * k][hd]);
            const float Ms = (Mx == -INFINITY) ? 0.0f : Mx;
            float Ls = 0.0f, A = 0.0f;
#pragma unroll
            for (int k = 0; k < kShare; ++k) {
                const float f = fast_exp2(red_m[w0 + G * k][hd] - Ms);
                Ls = fmaf(red_l[w0 + G * k][hd], f, Ls);
                A = fmaf(reinterpret_cast<const float *>(area[w0 + G * k])[hd * SPARK_D + ch], f, A);
            }
            store_out(gg, ch, A, Ls);
        }
    }
    if (P.trace != nullptr) { stamp(P, 4, wall_clock64()); stamp(P, 7, 1ull); }
}

template <int G, int BW>
static hipError_t launch_short(const DecodeParams &P, int nblocks, hipStream_t st)
{
    if (P.L.int8)
        hipLaunchKernelGGL((spark_decode_short_kernel<G, 1, BW>), dim3(nblocks), dim3(BW * 64), 0, st, P);
    else
        hipLaunchKernelGGL((spark_decode_short_kernel<G, 0, BW>), dim3(nblocks), dim3(BW * 64), 0, st, P);
    return hipGetLastError();
}

}  // namespace spark
