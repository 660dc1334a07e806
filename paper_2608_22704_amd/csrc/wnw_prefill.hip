// Prefill compression on the device (Method, "Prefill Compression"): the text-to-audio attention
// sums that rank a head's audio positions, and the keep selection from them (per segment, or
// over the whole audio of a head for the global variant).
//
// p[b][l][kv][tau] = sum over the text tokens t and the g q-heads of KV-head kv of the softmax
// weight that text token t puts on audio position tau; text token t attends to every audio row
// and to text rows 0..t.  Per KV-head this is S = Q K^T with Q the g * T_t text query rows and K
// the T_a + T_t key rows, a dense contraction, so both passes run on the bf16 matrix cores (fp32
// accumulation):
//   pass 1 (prefill_rowstats_kernel): per query row, STAT_BIAS minus the log-sum-exp of its logits over
//           its causal key set (base 2);
//   pass 2 (prefill_colsum_kernel): per audio key, the sum over all query rows of
//           exp(s - lse).  Audio keys are visible to every text row, so pass 2 needs no mask.
// The streamed operand of either pass (K rows, then query rows) goes straight from global to shared
// memory, three 16 KB tiles deep, and the tile loop is unrolled over the three buffers so that no
// vector instruction computes an address.
//
// What bounds it: per logit and pass, an FMA, an exponential and an addition next to 256 flop on the
// matrix cores, and the chip's power: on 240 KV-heads, 15000 keys and 2048 rows the clock falls to
// 1.6-1.7 GHz, with the matrix cores busy 50-57 % of the cycles and vector instructions issued on 45 % of
// them (counting four cycles each; an exponential holds the unit longer).  There both passes took 4.06-4.4 ms
// staged through registers with 16 x 16 products in pass 1, and take 3.41-3.63 ms now, 3.9 on the
// benchmark's inputs (3.8 TFLOP executed: 1.0-1.1 PFLOP/s; a bf16 matrix product of 8192 reaches 1.18 on the card);
// on 72 KV-heads, 3607 keys and 1176 rows 205-215 us, now 178-187 us.  There the tiles in flight are not quite
// kept there: the fragments loaded before the loop are first used in it, and the compiler waits for every load
// in the first of three tiles of each round.  A loop that takes one product's terms between the next one's
// matrix instructions, at two work-groups a compute unit, was slower (3.9 ms): three work-groups overlap the two
// units better.
#include "wnw_internal.h"
#include "wnw_lds.h"

#include <algorithm>
#include <type_traits>

#include <math.h>

namespace wnw {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr float LOG2E = 1.4426950408889634f;
constexpr float C2 = 0.08838834764831845f * LOG2E;   // logit scale 1 / sqrt(128), base 2
// Added to every exponent of pass 2: 32 lets terms down to 2^-158 count, for sums that fp32 holds from 2^-126
// up, and costs half the rounding of 64 (error against 64 bits 8.2e-7 with 64).
constexpr float STAT_BIAS = 32.f;
constexpr int PT = 64;                                // rows per tile in shared memory
constexpr int PBUF = 3;                               // tiles in shared memory, two of them in flight
constexpr int PPF = PT * (D / 8) / NT;                // 16-byte pieces per lane and tile

// 2^x by the hardware instruction alone: outputs below 2^-126 flush to zero (exp2f adds a
// range fix-up of ~3 instructions per call for them).
__device__ inline float exp2_hw(float x)
{
    return __builtin_amdgcn_exp2f(x);
}

__device__ inline bf16x8_t as_bf8(uint4 u)
{
    return __builtin_bit_cast(bf16x8_t, u);
}

__device__ inline f32x4_t mfma16(bf16x8_t a, bf16x8_t b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Work-group w is dispatched to accelerator die (XCD) w % 8, each with its own L2.  The
// returned order gives the work-groups of one die consecutive logical indices, so the blocks
// of one KV-head (which share its K or Q rows) run on one die and share its L2.
__device__ inline int xcd_order(int w, int n)
{
    const int q = n / 8, r = n % 8, x = w % 8;
    return x * q + min(x, r) + w / 8;
}

// Merge of two (max, sum) pairs of base-2 softmax statistics.
__device__ inline void merge_ms(float &m, float &l, float m2, float l2)
{
    const float mm = fmaxf(m, m2);
    const float a = m == -INFINITY ? 0.f : l * exp2f(m - mm);
    const float b = m2 == -INFINITY ? 0.f : l2 * exp2f(m2 - mm);
    m = mm;
    l = a + b;
}

// Pass 1.  Grid: ceil(g * T_t / (128 NB)) row blocks for each of the B * L * H_kv KV-heads, in XCD
// order.  Wave w owns query rows r0 + 32 NB w .. + 32 NB (NB blocks of 32, the B operands, in
// registers) of KV-head (b, lk); rows r = j * T_t + t (q-head j of the group, text token t).  The
// result of 32 keys against 32 rows (see wnw_lds.h) leaves every lane sixteen keys of ONE row, so a
// row's running (max, sum) is a single pair per lane and block; the two lanes of a row merge at the
// end.  NB = 2 halves the shared-memory reads per product; NB = 1 is for launches of few work-groups
// (72 KV-heads, 1176 rows, 3754 keys: 112 us with 1, 121 with 2, 146 with 16 x 16 products).
template <int NB, bool DIRECT>
__global__ __launch_bounds__(NT, NB == 2 ? 2 : 3) void prefill_rowstats_kernel(Geometry g, const uint16_t *__restrict__ K,
                                                                              const uint16_t *__restrict__ qt,
                                                                              float *__restrict__ stat)
{
    constexpr int ROWS = 4 * 32 * NB;
    const int R = g.G * g.Tt, nrb = (R + ROWS - 1) / ROWS;
    const int v = xcd_order(blockIdx.x, gridDim.x), hd = v / nrb, rblk = v - hd * nrb;
    const int b = hd / (g.L * g.Hkv), lk = hd - b * g.L * g.Hkv, l = lk / g.Hkv, kv = lk - l * g.Hkv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const uint16_t *Kh = K + (size_t)hd * g.T * D;
    const size_t qbase = (((size_t)b * g.L + l) * g.Hq + (size_t)kv * g.G) * g.Tt;
    const uint16_t *Qh = qt + qbase * D;
    const int rw = rblk * ROWS + wave * 32 * NB + col;   // this lane's row of block 0

    __shared__ alignas(256) uint4 kbuf[PBUF][PT * (D / 8)];
    const unsigned tile0 = lds_address(&kbuf[0][0]);
    const TileLoader<PT, PPF, DIRECT> ld(wave, lane, 1);
    auto issue = [&](int t, int buf) { ld.load(Kh, t * PT, g.T, tile0 + (unsigned)buf * (PT * D * 2)); };
    bf16x8_t qf[NB][8];
    int lim[NB];                                      // causal limit (last visible key) of the row
    float nm[NB], sum[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int r = rw + n * 32;
#pragma unroll
        for (int s = 0; s < 8; ++s)
            qf[n][s] = as_bf8(r < R ? *(const uint4 *)(Qh + (size_t)r * D + 16 * s + 8 * half) : make_uint4(0, 0, 0, 0));
        lim[n] = r < R ? g.Ta + r % g.Tt : -1;
        nm[n] = INFINITY;
        sum[n] = 0.f;
    }
    // Statistics are base 2 and scaled, the running maximum kept negated (nm = -m) for the
    // exponent's FMA.  Every row sum holds a term of at least 2^0, so exponentials that flush
    // below 2^-126 change nothing.
    auto take = [&](f32x16_t (&x)[NB], int k0) {
        if (k0 + 32 <= g.Ta) {
            // audio keys: every one visible to every row, no mask.  The terms are first taken against
            // the running maximum as it stands; only when a row's terms add up to more than 2^20 (or
            // its maximum is still -inf, which gives +inf) does the wavefront raise the maxima and
            // take the keys again.  Sums stay far inside fp32's range either way.
            float t[NB], tall = 0.f;
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                float a[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = exp2_hw(fmaf(x[n][i], C2, nm[n]));
#pragma unroll
                for (int i = 4; i < 16; ++i) a[i & 3] += exp2_hw(fmaf(x[n][i], C2, nm[n]));
                t[n] = (a[0] + a[1]) + (a[2] + a[3]);
                tall += t[n];
            }
            if (__any(tall > 0x1p20f)) {
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    float mt = x[n][0];
#pragma unroll
                    for (int i = 1; i < 16; ++i) mt = fmaxf(mt, x[n][i]);
                    const float mn = fmaxf(-nm[n], mt * C2);
                    float acc = sum[n] * exp2_hw(-nm[n] - mn);   // 0 before the first tile
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc += exp2_hw(fmaf(x[n][i], C2, -mn));
                    sum[n] = acc;
                    nm[n] = -mn;
                }
            } else {
#pragma unroll
                for (int n = 0; n < NB; ++n) sum[n] += t[n];
            }
        } else {
            // keys past a row's causal limit (text rows after its token, rows past the end, keys past
            // the cache) drop out
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                float mt = -INFINITY;
                bool nan = false;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    if (k0 + 8 * (i / 4) + 4 * half + i % 4 > lim[n]) x[n][i] = -INFINITY;
                    mt = fmaxf(mt, x[n][i]);
                    nan |= x[n][i] != x[n][i];
                }
                if (mt == -INFINITY && !nan) continue;   // every key masked for this row
                // a visible NaN (which the maximum passes over) makes the sum NaN, with a maximum that is kept
                const float mn = nan ? 0.f : fmaxf(-nm[n], mt * C2);
                float acc = sum[n] * exp2_hw(-nm[n] - mn);   // exp2(-inf) = 0 for an empty row
#pragma unroll
                for (int i = 0; i < 16; ++i) acc += exp2_hw(fmaf(x[n][i], C2, -mn));
                sum[n] = acc;
                nm[n] = -mn;
            }
        }
    };
    const int nt = (g.T + PT - 1) / PT;
#pragma unroll
    for (int i = 0; i < PBUF - 1; ++i) issue(i, i);
    const FragOffsets fo(lane);
    // one tile; `buf` is a constant, so every shared address is a lane's offset and an immediate
    auto tile = [&](int t, auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
        lds_loads_wait<(PBUF - 2) * PPF>();           // this wavefront's part of tile t has landed
        lds_tile_barrier();                           // everyone's has, and tile t - 1 is read
        issue(t + PBUF - 1, buf == 0 ? PBUF - 1 : buf - 1);
#pragma unroll
        for (int h = 0; h < PT / 32; ++h) {
            f32x16_t x[NB] = {};
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const bf16x8_t a = frag_read(tile0 + fo.o[s] + (unsigned)(buf * PT + h * 32) * (D * 2));
#pragma unroll
                for (int n = 0; n < NB; ++n) x[n] = mfma32(a, qf[n][s], x[n]);
            }
            take(x, t * PT + h * 32);
        }
    };
    for (int t = 0; t < nt; t += PBUF) {
        tile(t, std::integral_constant<int, 0>{});
        if (t + 1 < nt) tile(t + 1, std::integral_constant<int, 1>{});
        if (t + 2 < nt) tile(t + 2, std::integral_constant<int, 2>{});
    }
    static_assert(PBUF == 3, "the loop above names the buffers");
    lds_loads_wait<0>();                              // the loads past the last tile
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        float m = -nm[n], s = sum[n];
        const float m2 = __shfl_xor(m, 32), s2 = __shfl_xor(s, 32);
        merge_ms(m, s, m2, s2);
        const int r = rw + n * 32;
        if (half == 0 && r < R) stat[qbase + r] = (STAT_BIAS - m) - log2f(s);
    }
}

// Pass 2.  Grid: ceil(T_a / (64 KB)) key blocks for each of the B * L * H_kv KV-heads, in XCD order.
// Wave w owns audio keys k0 + 16 KB w .. + 16 KB (KB 16-key blocks, their K fragments held in
// registers, so each query fragment read from shared memory feeds KB MFMA chains); the work-group
// walks every query row of the KV-head in tiles of PT rows, and each lane adds exp2(s * C2 - lse) over
// the rows it holds for its key column.  v_mfma_f32_16x16x32_bf16 here: lane l holds A row l % 16 and B
// column l % 16 at k = 8 * (l / 16) .. + 8 (of 32); the 16x16 result holds column l % 16 of rows
// 4 * (l / 16) + i in element i, so a key's sum ends in four lanes (32 x 32 blocks leave it in 32: 118
// against 107 us on 72 KV-heads, 3607 keys, 1176 rows).
// KB = 4 feeds more products per fragment read; KB = 3 cuts a small cache into more work-groups
// (measured, both passes together: 240 KV-heads, 15000 keys, 2048 rows 3.59 ms with 4, 3.66 with 3; 72
// KV-heads, 3607 keys, 1176 rows 192 us with 4, 187 with 3).
template <int KB, bool DIRECT>
__global__ __launch_bounds__(NT, 3) void prefill_colsum_kernel(Geometry g, const uint16_t *__restrict__ K,
                                                               const uint16_t *__restrict__ qt,
                                                               const float *__restrict__ stat, float *__restrict__ p)
{
    constexpr int KEYS = 64 * KB;
    const int R = g.G * g.Tt, nkb = (g.Ta + KEYS - 1) / KEYS;
    const int v = xcd_order(blockIdx.x, gridDim.x), hd = v / nkb, kblk = v - hd * nkb;
    const int b = hd / (g.L * g.Hkv), lk = hd - b * g.L * g.Hkv, l = lk / g.Hkv, kv = lk - l * g.Hkv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const uint16_t *Kh = K + (size_t)hd * g.T * D;
    const size_t qbase = (((size_t)b * g.L + l) * g.Hq + (size_t)kv * g.G) * g.Tt;
    const uint16_t *Qh = qt + qbase * D;
    const int kw = kblk * KEYS + wave * 16 * KB;

    // Each wavefront loads its own copy of a tile's row statistics too, straight to shared memory like
    // the tile (a load into registers would make the compiler wait for the tiles in flight as well).
    __shared__ alignas(256) uint4 qbuf[PBUF][PT * (D / 8)];
    __shared__ alignas(16) float sbuf[PBUF][4][PT];
    static_assert(PT == 64, "one row statistic per lane and tile");
    const unsigned tile0 = lds_address(&qbuf[0][0]), stat0 = lds_address(&sbuf[0][wave][0]);
    const TileLoader<PT, PPF, DIRECT> ld(wave, lane, 1);
    auto issue = [&](int t, int buf) {
        ld.load(Qh, t * PT, R, tile0 + (unsigned)buf * (PT * D * 2));
        load_word_to_lds(stat + qbase, (unsigned)min(t * PT + lane, R - 1) * 4, stat0 + (unsigned)buf * (unsigned)sizeof(sbuf[0]));
    };
    bf16x8_t kf[KB][4];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int key = kw + kb * 16 + col;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            kf[kb][kk] = as_bf8(key < g.Ta ? *(const uint4 *)(Kh + (size_t)key * D + grp * 8 + 32 * kk)
                                           : make_uint4(0, 0, 0, 0));
    }
    // byte offsets of this lane's four fragments of tile rows 0 .. 15 (rows 16 n .. are 16 n rows further)
    unsigned fo[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) fo[kk] = (unsigned)(col * (D * 2) + ((4 * kk + grp) ^ col) * 16);
    float acc[KB] = {};
    // Terms are taken as 2^(x - lse + STAT_BIAS), with STAT_BIAS - lse from pass 1, and the sum scaled back
    // at the end, so that terms below 2^-126 still count without the exponential's range fix-up (terms
    // are at most 1 and sums of at most R of them stay far below the fp32 range).
    const int nt = (R + PT - 1) / PT;
#pragma unroll
    for (int i = 0; i < PBUF - 1; ++i) issue(i, i);
    // one tile; `buf` is a constant, so every shared address is a lane's offset and an immediate
    auto tile = [&](int t, auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
        lds_loads_wait<(PBUF - 2) * (PPF + 1)>();     // this wavefront's part of tile t has landed
        if (t * PT + PT > R && t * PT + lane >= R) sbuf[buf][wave][lane] = -INFINITY;   // past the last row: adds 0
        lds_tile_barrier();                           // everyone's has, and tile t - 1 is read
        issue(t + PBUF - 1, buf == 0 ? PBUF - 1 : buf - 1);
#pragma unroll
        for (int rb = 0; rb < PT / 16; ++rb) {
            bf16x8_t qf[4];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) qf[kk] = frag_read(tile0 + fo[kk] + (unsigned)(buf * PT + rb * 16) * (D * 2));
            const f32x4_t st = *(const f32x4_t *)&sbuf[buf][wave][rb * 16 + 4 * grp];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) sc = mfma16(qf[kk], kf[kb][kk], sc);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[kb] += exp2_hw(fmaf(sc[i], C2, st[i]));
            }
        }
    };
    for (int t = 0; t < nt; t += PBUF) {
        tile(t, std::integral_constant<int, 0>{});
        if (t + 1 < nt) tile(t + 1, std::integral_constant<int, 1>{});
        if (t + 2 < nt) tile(t + 2, std::integral_constant<int, 2>{});
    }
    lds_loads_wait<0>();                              // the loads past the last tile
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        acc[kb] += __shfl_xor(acc[kb], 16);
        acc[kb] += __shfl_xor(acc[kb], 32);
    }
    if (grp == 0)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int key = kw + kb * 16 + col;
            if (key < g.Ta) p[(size_t)hd * g.Ta + key] = ldexpf(acc[kb], -(int)STAT_BIAS);
        }
}

// Per-segment keep selection.  Grid (n_sub, B), one work-group per non-anchor head: position
// tau of segment j is kept iff fewer than keep(j) positions of the segment outrank it, by
// (score descending, position ascending); keep(j) is kfull, or klast for the last segment.
__global__ __launch_bounds__(NT) void prefill_keep_kernel(Geometry g, const int32_t *__restrict__ sub_lk,
                                                         const int2 *__restrict__ seg_keep,
                                                         const float *__restrict__ p, uint8_t *__restrict__ keep)
{
    const int hi = blockIdx.x, b = blockIdx.y, nsub = gridDim.x;
    const int lkh = sub_lk[hi];
    const int2 kc = seg_keep[hi];
    const float *ph = p + ((size_t)b * g.L * g.Hkv + lkh) * g.Ta;
    uint8_t *kh = keep + ((size_t)b * nsub + hi) * g.Ta;
    for (int tau = threadIdx.x; tau < g.Ta; tau += NT) {
        const int j = tau / g.cl, b0 = j * g.cl, e0 = min(b0 + g.cl, g.Ta);
        const int k = j == g.nc - 1 ? kc.y : kc.x;
        const float v = ph[tau];
        int rank = 0;
        for (int u = b0; u < e0; ++u) {
            const float w = ph[u];
            rank += (w > v) || (w == v && u < tau);
        }
        kh[tau] = isnan(v) ? 2 : rank < k;
    }
}

// Order-preserving key of a score: larger score, larger key; -0 and +0 are one key (they compare
// equal, so they tie and the lower position wins, as in the per-segment ranking).
__device__ inline uint32_t score_key(float v)
{
    uint32_t u = __float_as_uint(v);
    if (u == 0x80000000u) u = 0;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Global variant: one work-group per non-anchor head keeps the total of its per-segment counts,
// ranked over the whole audio.  A radix selection (four 8-bit digits, most significant first)
// finds the key v of the k-th best score and how many positions holding exactly v are kept;
// those go to the lowest positions (a block-wide prefix count in position order).
__global__ __launch_bounds__(NT) void prefill_keep_global_kernel(Geometry g, const int32_t *__restrict__ sub_lk,
                                                                const int2 *__restrict__ seg_keep,
                                                                const float *__restrict__ p, uint8_t *__restrict__ keep)
{
    const int hi = blockIdx.x, b = blockIdx.y, nsub = gridDim.x, tid = threadIdx.x;
    const int2 kc = seg_keep[hi];
    const int total = g.nc ? (g.nc - 1) * kc.x + kc.y : 0;
    const float *ph = p + ((size_t)b * g.L * g.Hkv + sub_lk[hi]) * g.Ta;
    uint8_t *kh = keep + ((size_t)b * nsub + hi) * g.Ta;
    __shared__ int hist[256];
    __shared__ uint32_t s_prefix;
    __shared__ int s_need, s_scan[NT];
    uint32_t prefix = 0, mask = 0;
    int need = total;
    if (total > 0) {
        for (int shift = 24; shift >= 0; shift -= 8) {
            hist[tid] = 0;   // NT == 256 bins
            __syncthreads();
            for (int t = tid; t < g.Ta; t += NT) {
                const uint32_t key = score_key(ph[t]);
                if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255], 1);
            }
            __syncthreads();
            if (tid == 0) {
                int cum = 0, d = 255;
                for (; d > 0; --d) {
                    if (cum + hist[d] >= need) break;
                    cum += hist[d];
                }
                s_prefix = prefix | ((uint32_t)d << shift);
                s_need = need - cum;
            }
            __syncthreads();
            prefix = s_prefix;
            need = s_need;
            mask |= 255u << shift;
            __syncthreads();
        }
    }
    // keep: key > v, or key == v among the first `need` such positions
    int base = 0;
    for (int t0 = 0; t0 < g.Ta; t0 += NT) {
        const int t = t0 + tid;
        const float v = t < g.Ta ? ph[t] : 0.f;
        const uint32_t key = score_key(v);
        const int tie = (total > 0 && t < g.Ta && key == prefix) ? 1 : 0;
        s_scan[tid] = tie;
        __syncthreads();
        for (int o = 1; o < NT; o <<= 1) {   // inclusive prefix sum
            const int add = tid >= o ? s_scan[tid - o] : 0;
            __syncthreads();
            s_scan[tid] += add;
            __syncthreads();
        }
        if (t < g.Ta) {
            const int before = base + s_scan[tid] - tie;
            kh[t] = isnan(v) ? 2 : (total > 0 && (key > prefix || (tie && before < need)));
        }
        base += s_scan[NT - 1];
        __syncthreads();
    }
}

// p = 0 (no text tokens): a fill kernel rather than a memset, so that the launch can sit in a
// captured graph.
__global__ __launch_bounds__(NT) void prefill_zero_kernel(float *__restrict__ p, long long n)
{
    for (long long i = (long long)blockIdx.x * NT + threadIdx.x; i < n; i += (long long)gridDim.x * NT) p[i] = 0.f;
}

}  // namespace

hipError_t launch_prefill_scores(const Geometry &g, const uint16_t *K, const uint16_t *q_text, float *lse,
                                 float *p, hipStream_t st)
{
    const int R = g.G * g.Tt;
    if (g.Ta == 0) return hipSuccess;
    if (R == 0) {
        const long long n = (long long)g.B * g.L * g.Hkv * g.Ta;
        hipLaunchKernelGGL(prefill_zero_kernel, dim3((unsigned)std::min<long long>((n + NT - 1) / NT, 4096)), dim3(NT), 0,
                           st, p, n);
        return hipGetLastError();
    }
    const long long nheads = (long long)g.B * g.L * g.Hkv;
    // Pass 1: work-groups of 256 rows from four of them a compute unit up, of 128 below.  Smaller ones cost from
    // 4.5 a unit up (72 KV-heads, 4096 rows, 7500 keys: +36 us of 1075; 240 KV-heads, 1200 rows, 3607 keys: +43 of 553) and
    // gain up to 1.4 (72 KV-heads, 1176 rows, 15000 keys: -11 of 677; 8 KV-heads, 1536 rows, 15000 keys: -109 of
    // 369).  Between, the rows that fill the last work-group decide (at 2.8 a unit -43 of 1249 us with 588 rows a head,
    // +24 of 655 with 2400; at 1.9 +7 to +13 of 71 to 150).
    const long long n1 = (long long)((R + 255) / 256) * nheads, n1s = (long long)((R + 127) / 128) * nheads;
    // Pass 2: KB = 4 from eight work-groups of 256 keys a compute unit up, 3 below.  KB = 3 costs 5 to 20 us from 8.4 a
    // unit up on 72 KV-heads (1075 us: +17; 2042: +43) and gains 5 to 17 at 4.2 (187 us: -5; 585: -17); with the last round
    // of work-groups nearly empty it goes the other way (240 KV-heads, 3607 keys: -9 to -21 of 308 to 928 at 14).
    const long long n2 = (long long)((g.Ta + 255) / 256) * nheads, n2s = (long long)((g.Ta + 191) / 192) * nheads;
    if (n1s > INT32_MAX || n2s > INT32_MAX) return hipErrorInvalidValue;
    // rows that are not aligned to the loads straight into shared memory: through registers (one variant each)
    const bool direct = (((uintptr_t)K | (uintptr_t)q_text) & 15) == 0;
    if (!direct)
        hipLaunchKernelGGL((prefill_rowstats_kernel<1, false>), dim3((unsigned)n1s), dim3(NT), 0, st, g, K, q_text, lse);
    else if (n1 >= 4LL * std::max(g.n_cu, 1))
        hipLaunchKernelGGL((prefill_rowstats_kernel<2, true>), dim3((unsigned)n1), dim3(NT), 0, st, g, K, q_text, lse);
    else
        hipLaunchKernelGGL((prefill_rowstats_kernel<1, true>), dim3((unsigned)n1s), dim3(NT), 0, st, g, K, q_text, lse);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!direct)
        hipLaunchKernelGGL((prefill_colsum_kernel<3, false>), dim3((unsigned)n2s), dim3(NT), 0, st, g, K, q_text, (const float *)lse, p);
    else if (n2 >= 8LL * std::max(g.n_cu, 1))
        hipLaunchKernelGGL((prefill_colsum_kernel<4, true>), dim3((unsigned)n2), dim3(NT), 0, st, g, K, q_text, (const float *)lse, p);
    else
        hipLaunchKernelGGL((prefill_colsum_kernel<3, true>), dim3((unsigned)n2s), dim3(NT), 0, st, g, K, q_text, (const float *)lse, p);
    return hipGetLastError();
}

hipError_t launch_prefill_keep(const Geometry &g, int n_sub, const int32_t *sub_lk, const int2 *seg_keep, bool global,
                               const float *p, uint8_t *keep, hipStream_t st)
{
    if (n_sub == 0 || g.Ta == 0) return hipSuccess;
    if (global)
        hipLaunchKernelGGL(prefill_keep_global_kernel, dim3(n_sub, g.B), dim3(NT), 0, st, g, sub_lk, seg_keep, p, keep);
    else
        hipLaunchKernelGGL(prefill_keep_kernel, dim3(n_sub, g.B), dim3(NT), 0, st, g, sub_lk, seg_keep, p, keep);
    return hipGetLastError();
}

}  // namespace wnw
