// Head triage arithmetic (Method, "Head Functional Triage via Offline Calibration", with the
// calibration score details of the appendix), on given inputs: the answer tokens' queries and a
// sample's keys, their aligned audio intervals, and the loss gradients at the audio keys.  The
// model, the alignment and the autograd that produce those are outside the library.
//
//   voice_hits_kernel   per (answer token, q-head): the K audio positions with the largest
//                       logit (softmax keeps the order), ties to the lower position, counted
//                       inside the token's interval.  voice_screen_kernel finds the candidates on the
//                       bf16 matrix cores and decides among them in double; voice_hits_kernel takes
//                       the rows it leaves.  Deciding logits are exact bf16 products summed in
//                       double; a sum of 128 products (16 significant bits each) rounds only when
//                       their magnitudes span more than ~30 binary orders, so the top-K decisions are
//                       in practice those of the exact logits.
//   key_sens_kernel     per (answer token, KV-head): the mean over audio positions of the L2 norm
//                       of the key gradient.  A streaming reduction (HBM-bound).
//   wnw_triage          (host) VS and HS means, VS * HS ranking, roles, normalised importance.
#include "wnw.h"
#include "wnw_internal.h"
#include "wnw_lds.h"
#include "wnw_screen.h"
#include "wnw_slots.h"

#include <float.h>
#include <math.h>

#include <algorithm>
#include <cstring>
#include <numeric>
#include <type_traits>
#include <vector>

namespace wnw {

namespace {

constexpr int VH_ROWS = 64;   // (token, q-head) rows per work-group (16 per wavefront)
constexpr int VH_TILE = 16;   // keys staged in LDS per iteration (as doubles): one MFMA key block
static_assert(VH_TILE * (D / 8) % NT == 0, "whole 16-byte pieces per thread");
constexpr int VH_KMAX = 8;    // largest K (the paper uses 4 and 8)
static_assert(VH_TILE % 16 == 0, "whole 16-key blocks per tile");
typedef double v4d __attribute__((ext_vector_type(4)));

__device__ inline void bf16x2(uint32_t u, double &lo, double &hi)
{
    lo = (double)__uint_as_float(u << 16);
    hi = (double)__uint_as_float(u & 0xffff0000u);
}

__device__ inline int vh_xcd_order(int w, int n)
{
    const int q = n / 8, r = n % 8, x = w % 8;
    return x * q + min(x, r) + w / 8;
}

// Voice hits, screened: the bf16 matrix cores bound every logit, and only the few keys that can
// be among a row's top K are evaluated in double.  Exactly the integers of voice_hits_kernel (below),
// which takes the rows that the screen cannot decide (hits = VH_OPEN on return).
//
// Bound.  A logit a from v_mfma_f32_32x32x16_bf16 differs from the exact e by at most
// m = 2^-14 * sum_d |q_d| kmax_d, kmax_d being the largest |k_d| of the keys (see wnw_screen.h).  Keys are split into
// groups (per lane and register pair) of which the largest a is kept; if T is the K-th
// largest of these maxima, K different keys have a >= T, hence e >= T - m, so a key of the
// exact top K, ties included, has a >= T - 2 m.
//   sweep A  every third key (every second for K > 4): T and kmax_d from a sample spread over the audio;
//   sweep B  every key: those with a >= T - 3 m go to the row's list, which leaves a key's own m twice the
//            sample's; kmax_d of every key is taken along;
//   if a list overflowed, or some kmax_d is over twice the sample's: both again, all from every key, with T - 2 m;
// (one maximum over all channels instead of kmax_d makes m many times too large for keys with a few large
// channels: with a constant 400 in one channel of normal keys most rows overflowed, 5.9 ms instead of the double
// kernel's 4.4);
// then the listed keys' logits in double (exact products, 16 lanes a key) and their ranks by
// (value descending, position ascending).  A row stays open when its list overflows even then
// (many keys within 2 m of each other, such as a zero query) or its values are not finite, too
// large or too small for the bound.
//
// What bounds it: nothing alone.  One 32 x 32 x 128 product per wavefront and tile is 8 matrix instructions
// against 10 KB read from shared memory, about 90 other vector instructions (the scan of sixteen logits, the
// channels' maxima, the lists) and a barrier; the matrix cores are busy 28 % of the cycles and vector
// instructions issued on 39 %.  The keys stream 1.3 to 2 times from HBM (1.2 GB on 240 KV-heads at 15000
// positions: 0.25 ms at the rate of a large copy).  240 KV-heads, 15000 positions, 256 rows each, K = 4: 4.37-4.5 ms
// with every logit in double, 0.46-0.49 ms here (0.54 while every tile waited for a shared maximum over all
// channels); the same with constants of up to 1000 in a channel.  Eight wavefronts: RB blocks of 32 rows
// times KS = 8 / RB shares of a tile's keys, so that a few rows still use the whole work-group.
constexpr int VH_OPEN = -1;
constexpr int VF_THREADS = 512;
constexpr int VF_CAP = 60;       // listed keys per row (60 keep two work-groups of RB = 4 in 160 KB)
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));

// Sum over the 16 lanes of a row of lanes (every lane ends with the same sum).
__device__ inline double sum16d(double v)
{
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o);
    return v;
}

template <int RB>
struct VfSmem {
    static constexpr int KS = 8 / RB;                 // shares of a tile's keys
    static constexpr int TILE = 32 * KS;              // keys per tile: one 32-key step per wavefront
    // tiles in shared memory, NBUF - 1 in flight: two work-groups a compute unit for RB = 4
    static constexpr int NBUF = RB == 1 ? 2 : 3;
    static constexpr int ROWS = 32 * RB;
    static constexpr int GRP = 16;                    // group maxima per row and share: 8 per lane, 2 lanes
    union {
        alignas(256) uint4 tile[NBUF][TILE * 16];     // see wnw_lds.h
        float gmax[ROWS][KS * GRP + 1];
    };
    int list[ROWS][VF_CAP];
    int cnt[ROWS];                                    // keys listed (those past VF_CAP are dropped)
    float thr[ROWS];                                  // T
    alignas(16) unsigned kmax[D];                     // largest element per channel, bf16 magnitude bits
};

template <int RB>
__global__ __launch_bounds__(VF_THREADS, RB == 4 ? 4 : 2) void voice_screen_kernel(
    int L, int Hq, int Hkv, int T, int Ta, int n_tok, int K, const uint16_t *__restrict__ k,
    const uint16_t *__restrict__ q, const int32_t *__restrict__ span, int32_t *__restrict__ hits)
{
    using SM = VfSmem<RB>;
    constexpr int KS = SM::KS, TILE = SM::TILE, ROWS = SM::ROWS, NBUF = SM::NBUF;
    constexpr int PF = TILE * 16 / VF_THREADS;        // 16-byte pieces per lane and tile
    static_assert(PF * VF_THREADS == TILE * 16, "whole pieces per thread");
    __shared__ SM sm;
    const int g = Hq / Hkv, R = n_tok * g, nrb = (R + ROWS - 1) / ROWS;
    const int wg = vh_xcd_order(blockIdx.x, gridDim.x), lk = wg / nrb, rblk = wg - lk * nrb;
    const int l = lk / Hkv, kv = lk - l * Hkv;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave % RB, ks = wave / RB;         // this wavefront's row block and key share
    const uint16_t *Kh = k + (size_t)lk * T * D;
    auto q_row = [&](int r) {                         // row = answer token * g + q-head of the group
        const int t = r / g, j = r - t * g;
        return q + (((size_t)t * L + l) * Hq + (size_t)kv * g + j) * D;
    };

    // B operand: column col = row rblk * ROWS + 32 rw + col; lane half h holds dimensions 16 s + 8 h .. + 8 of step s
    const int lrow = rw * 32 + col, row = rblk * ROWS + lrow;
    uint4 qf[8];
    float q1 = 0.f;
    {
        const uint4 *src = (const uint4 *)(row < R ? q_row(row) : q);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            qf[s] = row < R ? src[2 * s + half] : make_uint4(0, 0, 0, 0);
            const uint32_t d[4] = {qf[s].x, qf[s].y, qf[s].z, qf[s].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                q1 += fabsf(__uint_as_float(d[e] << 16)) + fabsf(__uint_as_float(d[e] & 0xffff0000u));
        }
        q1 += __shfl_xor(q1, 32);
    }
    if (tid < ROWS) sm.cnt[tid] = 0, sm.thr[tid] = -INFINITY;
    if (tid < D) sm.kmax[tid] = 0;

    float gm[8];                                      // maxima of this lane's groups
#pragma unroll
    for (int i = 0; i < 8; ++i) gm[i] = -INFINITY;
    u16x2_t km[4] = {};                               // maxima of channels 8 (lane % 16) .. + 8 over the keys this lane reads
    float lim = NAN;                                  // keys with a logit of at least this are listed (NaN: none)
    bool in_range = false;                            // the bound holds for this row

    const unsigned tile0 = lds_address(&sm.tile[0][0]);
    const FragOffsets fo(lane);
    // One sweep over the keys 0, step, 2 step ...; LIST (step 1): append the keys at or above the threshold.
    // The keys of a tile are looked at one iteration after their product, whose result is there by then.
    auto sweep = [&](auto list_c, int step) {
        constexpr bool LIST = decltype(list_c)::value;
        auto look = [&](const f32x16_t &x, int k0) {
            // x[i]: key k0 + step * (32 ks + 8 (i / 4) + 4 half + i % 4) against row lrow
            if constexpr (LIST) {
                float mx = x[0];
#pragma unroll
                for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[i]);
                if (__any(mx >= lim)) {
                    unsigned bits = 0;
#pragma unroll
                    for (int i = 0; i < 16; ++i) bits |= x[i] >= lim ? 1u << i : 0u;
                    while (__any(bits != 0)) {
                        if (bits) {
                            const int i = __ffs((int)bits) - 1;
                            bits &= bits - 1;
                            const int at = atomicAdd(&sm.cnt[lrow], 1);
                            if (at < VF_CAP) sm.list[lrow][at] = k0 + ks * 32 + 4 * half + 8 * (i >> 2) + (i & 3);
                        }
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) gm[i] = fmaxf(gm[i], fmaxf(x[2 * i], x[2 * i + 1]));
            }
        };
        const int dk = step * TILE, n = (Ta + dk - 1) / dk;
        const TileLoader<TILE, PF> ld(wave, lane, step);
        // past the audio the last key comes again (masked below)
        auto issue = [&](int t, int b) { ld.load(Kh, t * dk, Ta, tile0 + (unsigned)b * (TILE * D * 2)); };
        __syncthreads();                              // whatever shared the tiles' memory is done
#pragma unroll
        for (int b = 0; b < NBUF - 1; ++b) issue(b, b);
        f32x16_t x;
        const unsigned frag0 = tile0 + (unsigned)(ks * 32) * (D * 2);
        int buf = 0;
        for (int t = 0; t < n; ++t) {
            lds_loads_wait<(NBUF - 2) * PF>();        // this wavefront's part of tile t has landed
            lds_tile_barrier();                       // everyone's has, and tile t - 1 is read
            issue(t + NBUF - 1, buf == 0 ? NBUF - 1 : buf - 1);
            const int k0 = t * dk;
            if (t > 0) look(x, k0 - dk);
            // this wavefront's share of the tile's rows for the channels' maxima (two bf16 magnitudes a word)
#pragma unroll
            for (int j = 0; j < PF; ++j) {
                const int r = (wave * PF + j) * 4 + (lane >> 4);
                const uint4 a = sm.tile[buf][r * 16 + ((lane ^ r) & 15)];
                const uint32_t d[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) km[e] = __builtin_elementwise_max(km[e], __builtin_bit_cast(u16x2_t, d[e] & 0x7fff7fffu));
            }
            const unsigned fb = frag0 + (unsigned)buf * (TILE * D * 2);
            x = f32x16_t{};
#pragma unroll
            for (int s = 0; s < 8; ++s) x = mfma32(frag_read(fb + fo.o[s]), __builtin_bit_cast(bf16x8_t, qf[s]), x);
            if (k0 + dk > Ta) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + step * (ks * 32 + 4 * half + 8 * (i / 4) + i % 4) >= Ta) x[i] = -INFINITY;
            }
            buf = buf == NBUF - 1 ? 0 : buf + 1;
        }
        lds_loads_wait<0>();                          // the loads past the last tile
        __syncthreads();
        look(x, (n - 1) * dk);
    };
    // T: the K-th largest of the row's group maxima (-inf while fewer than K groups hold a key); then the limit
    // T - margin * m
    auto threshold = [&](float margin) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // the four lanes of a wavefront with these channels, then the wavefronts
            unsigned m = __builtin_bit_cast(unsigned, km[e]);
#pragma unroll
            for (int o = 16; o < 64; o <<= 1)
                m = __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, m), __builtin_bit_cast(u16x2_t, __shfl_xor(m, o))));
            if (lane < 16) {
                atomicMax(&sm.kmax[8 * lane + 2 * e], m & 0xffffu);
                atomicMax(&sm.kmax[8 * lane + 2 * e + 1], m >> 16);
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) sm.gmax[lrow][ks * SM::GRP + half * 8 + i] = gm[i];
        __syncthreads();
        // sixteen lanes a row: each ranks its share of the maxima among all
        for (int r = tid >> 4; r < ROWS; r += VF_THREADS / 16) {
            for (int a = tid & 15; a < KS * SM::GRP; a += 16) {
                const float v = sm.gmax[r][a];
                int gt = 0, ge = 0;
                for (int b = 0; b < KS * SM::GRP; ++b) {
                    const float w = sm.gmax[r][b];
                    gt += w > v;
                    ge += w >= v;
                }
                if (gt < K && ge >= K) sm.thr[r] = v;   // equal maxima write the same value
            }
        }
        __syncthreads();
        float S = 0.f, mx = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const uint32_t d[4] = {qf[s].x, qf[s].y, qf[s].z, qf[s].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float k0 = __uint_as_float(sm.kmax[16 * s + 8 * half + 2 * e] << 16);
                const float k1 = __uint_as_float(sm.kmax[16 * s + 8 * half + 2 * e + 1] << 16);
                S = fmaf(fabsf(__uint_as_float(d[e] << 16)), k0, S);
                S = fmaf(fabsf(__uint_as_float(d[e] & 0xffff0000u)), k1, S);
                mx = fmaxf(mx, fmaxf(k0, k1));
            }
        }
        S += __shfl_xor(S, 32);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        in_range = row < R && screen_in_range(S, q1, mx);
        // at least the lowest finite value: a masked key (-inf) is never listed
        lim = in_range ? fmaxf(sm.thr[lrow] - margin * VF_GAMMA * S, -FLT_MAX) : NAN;
    };
    // The sample's T lets about smp * K keys of a row pass, far under VF_CAP for nearly every row; an
    // overflow costs the work-group two more sweeps.  A short audio is its own sample.
    const int smp = Ta < 16 * TILE ? 1 : K <= 4 ? 3 : 2;
    if (__syncthreads_or(q1 > 0.f && q1 < INFINITY)) {
        sweep(std::false_type{}, smp);
        threshold(smp > 1 ? 3.f : 2.f);
        if (__syncthreads_or(in_range)) {
            sweep(std::true_type{}, 1);
            __syncthreads();
            if (smp > 1) {
                bool again = tid < ROWS && sm.cnt[tid] > VF_CAP;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // twice the sample's maximum, at most the largest finite value
                    const unsigned ch = 8 * (lane & 15) + 2 * e;
                    again |= km[e].x > min(sm.kmax[ch] + 0x80u, 0x7f7fu) || km[e].y > min(sm.kmax[ch + 1] + 0x80u, 0x7f7fu);
                }
                if (__syncthreads_or(again)) {
                    // other groups than the sample's: a key is in one group only
#pragma unroll
                    for (int i = 0; i < 8; ++i) gm[i] = -INFINITY;
                    sweep(std::false_type{}, 1);
                    threshold(2.f);
                    if (tid < ROWS) sm.cnt[tid] = 0;   // before the sweep's first barrier
                    sweep(std::true_type{}, 1);
                    __syncthreads();
                }
            }
        }
    }
    // rows outside the bound's range stay open, as those with too many keys
    if (ks == 0 && half == 0 && !in_range) sm.cnt[lrow] = VF_CAP + 1;
    __syncthreads();
    // Exact logits of the listed keys: sixteen lanes a row, four keys in flight; lane i keeps the
    // keys i, i + 16, ... and ranks them among all.
    const int l16 = tid & 15, base = lane & 48;
    for (int r = tid >> 4; r < ROWS; r += VF_THREADS / 16) {
        const int rg = rblk * ROWS + r;
        if (rg >= R) break;
        const int t = rg / g, j = rg - t * g, n = sm.cnt[r];
        int32_t *dst = hits + ((size_t)t * L + l) * Hq + (size_t)kv * g + j;
        if (n > VF_CAP) {
            if (l16 == 0) *dst = VH_OPEN;
            continue;
        }
        double qd[8];
        {
            const uint4 w = ((const uint4 *)q_row(rg))[l16];
            const uint32_t d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) bf16x2(d[e], qd[2 * e], qd[2 * e + 1]);
        }
        constexpr int NS = (VF_CAP + 15) / 16;
        double val[NS];
        int pos[NS], before[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            val[s] = -INFINITY, pos[s] = INT32_MAX, before[s] = 0;
            for (int u0 = 0; u0 < 16 && s * 16 + u0 < n; u0 += 4) {
                uint4 w[4];
                int p[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    p[u] = sm.list[r][min(s * 16 + u0 + u, n - 1)];
                    w[u] = ((const uint4 *)(Kh + (size_t)p[u] * D))[l16];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t d[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
                    double acc = 0.0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        double a, b;
                        bf16x2(d[e], a, b);
                        acc = fma(a, qd[2 * e], acc);
                        acc = fma(b, qd[2 * e + 1], acc);
                    }
                    acc = sum16d(acc);
                    if (l16 == u0 + u && s * 16 + u0 + u < n) val[s] = acc, pos[s] = p[u];
                }
            }
        }
#pragma unroll
        for (int s2 = 0; s2 < NS; ++s2)
            for (int o = 0; o < 16 && s2 * 16 + o < n; ++o) {
                const double w = __shfl(val[s2], base + o);
                const int pw = __shfl(pos[s2], base + o);
#pragma unroll
                for (int s = 0; s < NS; ++s) before[s] += w > val[s] || (w == val[s] && pw < pos[s]);
            }
        const int a = span[2 * t], b = span[2 * t + 1];
        int c = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) c += s * 16 + l16 < n && before[s] < K && pos[s] >= a && pos[s] < b;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) c += __shfl_xor(c, o);
        if (l16 == 0) *dst = c;
    }
}

// Voice hits in double throughout: for the rows that the screen left open (open_only; a work-group whose rows are
// all decided returns at once), or for all rows where there was no screen.
// Work-groups: ceil(n_tok * g / VH_ROWS) row blocks per KV-head (row = answer token * g + q-head
// of the group), in XCD order so that the row blocks of one KV-head read its keys through one L2.
// Wavefront w owns 16 rows of the block.  The logits run on v_mfma_f64_16x16x4f64 (lane
// l = i + 16k supplies A[i][k] and B[k][i]; D[i][j] lands in lane j + 16 (i % 4), element i / 4):
// A is a block of 16 keys from the staged tile, B the wavefront's 16 query rows (converted to
// double once and held in registers), and lane group k feeds dimension 32k + s at step s.  Every
// key element is read from shared memory once per wavefront.  A lane ends a key block holding
// four logits of its row (keys k + 4v) and keeps the best eight of the keys it sees (value
// descending; equal values keep the earlier, lower, position); the four lists of a row (one per
// lane group) are merged at the end.  Products of bf16 values are exact in double.
__global__ __launch_bounds__(NT, 4) void voice_hits_kernel(int L, int Hq, int Hkv, int T, int Ta, int n_tok, int K,
                                                       const uint16_t *__restrict__ k, const uint16_t *__restrict__ q,
                                                       const int32_t *__restrict__ span, int32_t *__restrict__ hits,
                                                       bool open_only)
{
    const int g = Hq / Hkv, R = n_tok * g, nrb = (R + VH_ROWS - 1) / VH_ROWS;
    const int v = vh_xcd_order(blockIdx.x, gridDim.x), lk = v / nrb, rblk = v - lk * nrb;
    const int l = lk / Hkv, kv = lk - l * Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kq = lane >> 4, li = lane & 15;
    const int r0 = rblk * VH_ROWS + wave * 16;
    if (open_only) {
        const int rg = rblk * VH_ROWS + tid;
        const int t = rg / g, j = rg - t * g;
        const bool open = tid < VH_ROWS && rg < R && hits[((size_t)t * L + l) * Hq + (size_t)kv * g + j] == VH_OPEN;
        if (!__syncthreads_or(open)) return;
    }
    // B operand: row r0 + li, dimensions 32 kq .. + 32
    double qd[32];
    {
        const int ra = r0 + li;
        const bool ok = ra < R;
        const int t = ok ? ra / g : 0, j = ok ? ra - t * g : 0;
        const uint4 *qrow = (const uint4 *)(q + (((size_t)t * L + l) * Hq + (size_t)kv * g + j) * D) + kq * 4;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint4 w = ok ? qrow[u] : make_uint4(0, 0, 0, 0);
            const uint32_t d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) bf16x2(d[e], qd[8 * u + 2 * e], qd[8 * u + 2 * e + 1]);
        }
    }
    double best[VH_KMAX];
    int bpos[VH_KMAX];
#pragma unroll
    for (int i = 0; i < VH_KMAX; ++i) {
        best[i] = -INFINITY;
        bpos[i] = INT32_MAX;
    }
    auto insert = [&](double val, int pos) {
        if (val > best[VH_KMAX - 1]) {
            // from the first entry it exceeds on, every entry moves down one (a displaced value may
            // equal the next: it stays the earlier of the two)
            bool move = false;
#pragma unroll
            for (int s = 0; s < VH_KMAX; ++s)
                if (move = move || val > best[s]; move) {
                    const double tv = best[s];
                    const int tp = bpos[s];
                    best[s] = val;
                    bpos[s] = pos;
                    val = tv;
                    pos = tp;
                }
        }
    };
    // key tile staged as doubles (each element converted once per work-group): key r, dimension
    // 32 kq + s at r * VH_KS + kq * 33 + s; the padding puts the 16 keys that one lane group reads
    // at a step on distinct banks.  After the loop the same memory holds the candidate lists.
    constexpr int VH_KS = 4 * 33 + 1;
    constexpr int TILE_DBL = VH_TILE * VH_KS, LIST_DBL = VH_ROWS * 4 * VH_KMAX * 3 / 2;   // lists: double + int
    __shared__ double ksd[TILE_DBL > LIST_DBL ? TILE_DBL : LIST_DBL];
    const uint16_t *Kh = k + (size_t)lk * T * D;
    // The next tile's keys are loaded into registers while the current tile is computed (each
    // thread holds VH_PF 16-byte pieces), then converted into the single shared buffer.
    constexpr int VH_PF = VH_TILE * (D / 8) / NT;
    uint4 pf[VH_PF];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int j = 0; j < VH_PF; ++j) {
            const int i = tid + j * NT, row = k0 + (i >> 4);
            pf[j] = row < Ta ? *(const uint4 *)(Kh + (size_t)row * D + (i & 15) * 8) : make_uint4(0, 0, 0, 0);
        }
    };
    fetch(0);
    for (int k0 = 0; k0 < Ta; k0 += VH_TILE) {
        __syncthreads();   // every wavefront is done with the previous tile
#pragma unroll
        for (int j = 0; j < VH_PF; ++j) {
            const int i = tid + j * NT, rr = i >> 4, c = i & 15;
            const uint32_t d[4] = {pf[j].x, pf[j].y, pf[j].z, pf[j].w};
            double *dst = ksd + rr * VH_KS + (c >> 2) * 33 + (c & 3) * 8;   // dimensions 8c .. 8c + 8
#pragma unroll
            for (int e = 0; e < 4; ++e) bf16x2(d[e], dst[2 * e], dst[2 * e + 1]);
        }
        __syncthreads();
        if (k0 + VH_TILE < Ta) fetch(k0 + VH_TILE);
        const int nk = min(VH_TILE, Ta - k0);
        for (int kb = 0; kb < nk; kb += 16) {
            // A: key k0 + kb + li, dimension 32 kq + s
            const double *ga = ksd + (kb + li) * VH_KS + kq * 33;
            v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s2 = 0; s2 < 32; ++s2) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[s2], qd[s2], acc, 0, 0, 0);
            // this lane: row r0 + li, keys k0 + kb + kq + 4 e
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = k0 + kb + kq + 4 * e;
                if (p < Ta) insert(acc[e], p);
            }
        }
    }
    __syncthreads();   // the tile's memory takes the candidate lists
    double (*sbest)[4 * VH_KMAX] = reinterpret_cast<double (*)[4 * VH_KMAX]>(ksd);
    int (*spos)[4 * VH_KMAX] = reinterpret_cast<int (*)[4 * VH_KMAX]>(ksd + VH_ROWS * 4 * VH_KMAX);
    const int rl = wave * 16 + li;   // this lane's row within the block
#pragma unroll
    for (int i = 0; i < VH_KMAX; ++i) {
        sbest[rl][kq * VH_KMAX + i] = best[i];
        spos[rl][kq * VH_KMAX + i] = bpos[i];
    }
    __syncthreads();
    const int rg = rblk * VH_ROWS + tid;
    if (tid < VH_ROWS && rg < R) {
        // top K of the row's candidates by (value descending, position ascending)
        const int t = rg / g, j = rg - t * g;
        const int a = span[2 * t], b = span[2 * t + 1];
        unsigned taken = 0;
        int c = 0;
        for (int n = 0; n < K; ++n) {
            int bi = -1;
            for (int i = 0; i < 4 * VH_KMAX; ++i) {
                if (taken >> i & 1u) continue;
                if (bi < 0 || sbest[tid][i] > sbest[tid][bi] ||
                    (sbest[tid][i] == sbest[tid][bi] && spos[tid][i] < spos[tid][bi]))
                    bi = i;
            }
            taken |= 1u << bi;
            const int pos = spos[tid][bi];
            c += pos >= a && pos < b;
        }
        hits[((size_t)t * L + l) * Hq + (size_t)kv * g + j] = c;
    }
}

// Rows of T_a gradient vectors, one per (answer token, KV-head); `parts` work-groups of KS_THREADS per row,
// each with `len` positions of it (a multiple of the round).  Sixteen lanes per position (eight floats
// each), KS_UNROLL positions per lane and round, the next round's loads in flight while this one is
// summed: the sixteen lanes sum their squares so that lane u of the row ends with round u's position,
// and one square root in double serves the round.  Norms are summed in double in a fixed order.
//
// What bounds it: HBM, once enough compute units stream; one alone takes about 30 GB/s whatever is in
// flight, so with few rows a row is split.  The parts' sums meet in a slot of the library (KsSlot), and
// the last work-group of a row to arrive adds them in order.  A launch takes a slot that its own stream used
// last or whose last user has ended, never one to wait for; with none it is not split.  72 rows of 7500
// positions (276 MB): 134 us with one work-group per row, 54.5 us split (5.1 TB/s); 8 rows of 15000 214 -> 19.6 us.
constexpr int KS_THREADS = 512, KS_SLOTS = KS_THREADS / 16, KS_UNROLL = 4;
typedef float f4v __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ inline float row_perm(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

constexpr int KS_STEP = KS_SLOTS * KS_UNROLL;   // positions of a work-group's round
constexpr int KS_PARTS = 768, KS_ROWS = 256;   // most parts of a split launch, most rows
struct KsSlot {
    double part[KS_PARTS];
    int arrived[KS_ROWS];                       // zero between launches
};
constexpr int KS_NSLOT = 8;
static __device__ KsSlot ks_slots[KS_NSLOT];

// SPLIT: `parts` > 1.
template <bool SPLIT>
__global__ __launch_bounds__(KS_THREADS) void key_sens_kernel(int Ta, int parts, int len, int slot_id,
                                                             const float *__restrict__ grad, float *__restrict__ sens)
{
    static_assert(KS_UNROLL == 4, "the sums below hand lane u the position of round u");
    constexpr int STEP = KS_STEP;
    const size_t row = blockIdx.x / (unsigned)parts;
    const int pt = (int)(blockIdx.x - row * parts), end = min(Ta, (pt + 1) * len);
    const int tid = threadIdx.x, l16 = tid & 15, slot = tid >> 4;
    const f4v *G4 = (const f4v *)(grad + row * (size_t)Ta * D) + 2 * l16;
    struct Round {
        f4v a[KS_UNROLL], b[KS_UNROLL];
    };
    // positions t0 + slot + 64 u; past the last one that comes again (not summed)
    auto load = [&](Round &r, int t0) {
#pragma unroll
        for (int u = 0; u < KS_UNROLL; ++u) {
            const f4v *p = G4 + (size_t)min(t0 + slot + u * KS_SLOTS, end - 1) * (D / 4);
            r.a[u] = __builtin_nontemporal_load(p);
            r.b[u] = __builtin_nontemporal_load(p + 1);
        }
    };
    double acc = 0.0;   // lanes 0..3 of a row of sixteen: positions of round 0..3
    auto add = [&](const Round &r, int t0) {
        float s2[KS_UNROLL];
#pragma unroll
        for (int u = 0; u < KS_UNROLL; ++u) {
            const f4v a = r.a[u], b = r.b[u];
            s2[u] = (a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w) + (b.x * b.x + b.y * b.y + b.z * b.z + b.w * b.w);
        }
        const bool odd = l16 & 1, up = l16 & 2;
        // with the neighbour (lane ^ 1), then with lane ^ 2: one position per lane of a quad
        const float p01 = (odd ? s2[1] : s2[0]) + row_perm<0xB1>(odd ? s2[0] : s2[1]);
        const float p23 = (odd ? s2[3] : s2[2]) + row_perm<0xB1>(odd ? s2[2] : s2[3]);
        float q = (up ? p23 : p01) + row_perm<0x4E>(up ? p01 : p23);
        q += row_perm<0x124>(q);   // the four quads of the row: rotations by four lanes, then by eight
        q += row_perm<0x128>(q);
        if (l16 < KS_UNROLL && t0 + slot + l16 * KS_SLOTS < end) acc += sqrt((double)q);
    };
    Round r0, r1;
    int t0 = pt * len;
    load(r0, t0);
    if constexpr (SPLIT) {
        // The rounds past the last position load it again.  Without those loads 72 rows of 7500 take 62 us
        // instead of 54.5; unsplit, with more rows than the chip holds at once, they cost: 600 rows of 300
        // positions 24.7 us with them, 19.1 without.
        for (; t0 < end; t0 += 2 * STEP) {
            load(r1, t0 + STEP);
            add(r0, t0);
            load(r0, t0 + 2 * STEP);
            add(r1, t0 + STEP);
        }
    } else {
        for (; t0 + 2 * STEP < end; t0 += 2 * STEP) {
            load(r1, t0 + STEP);
            add(r0, t0);
            load(r0, t0 + 2 * STEP);
            add(r1, t0 + STEP);
        }
        if (t0 + STEP < end) {
            load(r1, t0 + STEP);
            add(r0, t0);
            add(r1, t0 + STEP);
        } else
            add(r0, t0);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) acc += __shfl_xor(acc, o);
    __shared__ double red[KS_THREADS / 64];
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int i = 0; i < KS_THREADS / 64; ++i) s += red[i];
        if constexpr (SPLIT) {
            // agent-scope stores and loads around an agent-scope count: coherent across the dies' caches
            KsSlot &sl = ks_slots[slot_id];
            double *p = sl.part + row * parts;
            __hip_atomic_store(p + pt, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (atomicAdd(&sl.arrived[row], 1) != parts - 1) return;
            atomicExch(&sl.arrived[row], 0);
            s = 0.0;
            for (int i = 0; i < parts; ++i) s += __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        sens[row] = (float)(s / Ta);
    }
}

// The runtime's calls of the slot pool.  Other threads may be capturing: queries and event creation are not
// part of any capture, so this thread's calls are exempt from its check.
struct HipSlotRT {
    using Stream = hipStream_t;
    using Event = hipEvent_t;
    using Error = hipError_t;
    struct Uncaptured {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        Uncaptured() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
        ~Uncaptured() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    };
    // a failure that the caller goes round leaves no error behind for the next launch's check
    static Error handled(Error e)
    {
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
    }
    static bool ok(Error e) { return e == hipSuccess; }
    static Error create(Event &ev)
    {
        Uncaptured u;
        return handled(hipEventCreateWithFlags(&ev, hipEventDisableTiming | hipEventDisableSystemFence));
    }
    static Error query(Event ev, bool &ended)
    {
        Uncaptured u;
        const Error e = handled(hipEventQuery(ev));
        ended = e == hipSuccess;
        return e == hipErrorNotReady ? hipSuccess : e;
    }
    static Error wait(Stream st, Event ev) { return handled(hipStreamWaitEvent(st, ev, 0)); }
    static Error record(Event ev, Stream st) { return hipEventRecord(ev, st); }
    static bool shared_handle(Stream st) { return st == hipStreamPerThread; }
};
constexpr int KS_MAX_DEVICES = 64;
SlotPool<HipSlotRT, KS_NSLOT> ks_pool[KS_MAX_DEVICES];   // per device, for split launches

// Positions from which rows are split into `want` parts (0: never).  A split costs its slot 2 to 4 us.
// Measured unsplit and split: at 5 or fewer parts 144 rows of 1024 21.8 and 23.1 us, of 1300 26.9 and 24.3; at 4
// 191 rows of 2100 44.8 and 50.4, of 3000 62.8 and 53.6.  Few rows of few positions stream from the caches: 16
// rows of 1300 11.2 and 12.6, of 1500 14.1 and 12.6; 36 rows of 1024 10.8 and 12.8, of 1300 15.4 and 13.0.  72 rows
// of 1024 19.0 and 13.6; 240 rows unsplit stream at 5.6 TB/s.
int64_t ks_split_from(int64_t n, int64_t want)
{
    if (want < 4) return 0;
    if (want == 4) return 20 * KS_STEP;
    if (want == 5) return 9 * KS_STEP;
    return std::min<int64_t>(12 * KS_STEP, std::max<int64_t>(8 * KS_STEP, 45000 / n));
}

hipError_t launch_key_sens(int64_t n, int Ta, const float *grad, float *sens, hipStream_t st)
{
    int parts = 1, len = Ta, dev = 0;
    hipError_t e = hipSuccess;
    if (n <= KS_ROWS && Ta >= 8 * KS_STEP) {
        // parts for three work-groups a unit, of four rounds or more; none for a stream of another device than
        // the current one, where the slots' events belong
        int n_cu = 0;
        e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        hipDevice_t sdev = dev;
        if (st != nullptr && HipSlotRT::handled(hipStreamGetDevice(st, &sdev)) != hipSuccess) sdev = -1;
        const int64_t want = std::min<int64_t>(3 * n_cu, KS_PARTS) / n, from = ks_split_from(n, want);
        if (from > 0 && Ta >= from && dev < KS_MAX_DEVICES && sdev == dev) {
            len = (int)std::max<int64_t>(4 * KS_STEP, ((Ta + want - 1) / want + KS_STEP - 1) / KS_STEP * KS_STEP);
            parts = (int)((Ta + (int64_t)len - 1) / len);
        }
        // a captured launch may be replayed beside others: it keeps one work-group per row, and no slot
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (parts > 1 && (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone)) {
            (void)hipGetLastError();
            parts = 1;
        }
    }
    auto launch = [&](int np, int nl, int slot) {
        hipLaunchKernelGGL(np > 1 ? key_sens_kernel<true> : key_sens_kernel<false>, dim3((unsigned)(n * np)), dim3(KS_THREADS),
                           0, st, Ta, np, nl, slot, grad, sens);
        return hipGetLastError();
    };
    if (parts > 1 && ks_pool[dev].run(st, e, [&](int slot) { return launch(parts, len, slot); })) return e;
    return launch(1, Ta, 0);   // one work-group per row: no slot
}

// Rows per work-group of the screen: as many of 128, 64, 32 as there are and as leave every compute
// unit a work-group; fewer rows mean more shares of the keys.
template <int RB, typename... A>
hipError_t screen_rb(int64_t R, int64_t heads, hipStream_t st, A... args)
{
    using SM = VfSmem<RB>;
    hipLaunchKernelGGL(voice_screen_kernel<RB>, dim3((unsigned)((R + SM::ROWS - 1) / SM::ROWS * heads)), dim3(VF_THREADS), 0,
                       st, args...);
    return hipGetLastError();
}
template <typename... A>
hipError_t launch_voice_screen(int64_t R, int64_t heads, hipStream_t st, A... args)
{
    int dev = 0, n_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (R > 64 && (R + 127) / 128 * heads >= n_cu) return screen_rb<4>(R, heads, st, args...);
    if (R > 32 && (R + 63) / 64 * heads >= n_cu) return screen_rb<2>(R, heads, st, args...);
    return screen_rb<1>(R, heads, st, args...);
}

thread_local char t_msg[256] = "no error";

wnw_status triage_fail(wnw_status st, const char *msg)
{
    strncpy(t_msg, msg, sizeof t_msg - 1);
    return st;
}

}  // namespace

}  // namespace wnw

using namespace wnw;

extern "C" {

const char *wnw_triage_last_error(void)
{
    return t_msg;
}

wnw_status wnw_voice_hits(int32_t layers, int32_t q_heads, int32_t kv_heads, int32_t rows, int32_t audio_len,
                          int32_t n_tok, const void *k_dev, const void *q_dev, const int32_t *span_dev, int32_t top_k,
                          int32_t *hits_dev, void *hip_stream)
{
    if (layers < 1 || kv_heads < 1 || q_heads < kv_heads || q_heads % kv_heads || audio_len < 0 || rows < audio_len ||
        n_tok < 0 || (int64_t)layers * kv_heads > 65535)
        return triage_fail(WNW_ERR_INVALID, "bad sizes");
    const int g = q_heads / kv_heads;
    if ((int64_t)n_tok * g > INT32_MAX) return triage_fail(WNW_ERR_UNSUPPORTED, "too many answer-token rows");
    if (top_k < 1 || top_k > VH_KMAX || top_k > audio_len)
        return triage_fail(WNW_ERR_INVALID, "top_k must be in 1..8 and at most audio_len");
    if (n_tok == 0) return WNW_OK;
    if (!k_dev || !q_dev || !span_dev || !hits_dev) return triage_fail(WNW_ERR_INVALID, "NULL pointer");
    const int64_t R = (int64_t)n_tok * g, heads = (int64_t)layers * kv_heads;
    const int64_t nwg = (R + VH_ROWS - 1) / VH_ROWS * heads;
    if (nwg > INT32_MAX) return triage_fail(WNW_ERR_UNSUPPORTED, "too many answer tokens for one launch");
    // Short audio goes to the double kernel alone: the screen's fixed part (33 to 37 us) costs more than it
    // saves.  With few rows 27 us against 33 on 64 positions and 35 against 34 on 128; with 61440 rows (256 on 240
    // KV-heads) 43 against 45 us on 48 positions and 48 against 44 on 64.
    // Keys that are not aligned to the screen's loads (16 bytes, straight into shared memory) go there as well.
    const bool screen = audio_len >= (R * heads < 16384 ? 128 : 64) && (R + 31) / 32 * heads <= INT32_MAX &&
                        ((uintptr_t)k_dev & 15) == 0;
    if (screen) {
        const hipError_t es = launch_voice_screen(R, heads, (hipStream_t)hip_stream, layers, q_heads, kv_heads, rows, audio_len,
                                                  n_tok, top_k, (const uint16_t *)k_dev, (const uint16_t *)q_dev, span_dev,
                                                  hits_dev);
        if (es != hipSuccess) return triage_fail(WNW_ERR_HIP, hipGetErrorString(es));
    }
    hipLaunchKernelGGL(voice_hits_kernel, dim3((unsigned)nwg), dim3(NT), 0,
                       (hipStream_t)hip_stream, layers, q_heads, kv_heads, rows, audio_len, n_tok, top_k,
                       (const uint16_t *)k_dev, (const uint16_t *)q_dev, span_dev, hits_dev, screen);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? WNW_OK : triage_fail(WNW_ERR_HIP, hipGetErrorString(e));
}

wnw_status wnw_key_sensitivity(int32_t layers, int32_t kv_heads, int32_t audio_len, int32_t n_tok, const float *grad_dev,
                               float *sens_dev, void *hip_stream)
{
    if (layers < 1 || kv_heads < 1 || audio_len < 1 || n_tok < 0) return triage_fail(WNW_ERR_INVALID, "bad sizes");
    const int64_t n = (int64_t)n_tok * layers * kv_heads;
    if (n == 0) return WNW_OK;
    if (n > INT32_MAX) return triage_fail(WNW_ERR_UNSUPPORTED, "too many rows");
    if (!grad_dev || !sens_dev) return triage_fail(WNW_ERR_INVALID, "NULL pointer");
    const hipError_t e = launch_key_sens(n, audio_len, grad_dev, sens_dev, (hipStream_t)hip_stream);
    return e == hipSuccess ? WNW_OK : triage_fail(WNW_ERR_HIP, hipGetErrorString(e));
}

wnw_status wnw_triage(int32_t layers, int32_t kv_heads, int32_t group, int32_t n, const int32_t *sample,
                      const int32_t *hits, int32_t top_k, const float *sens, int32_t n_voice, int32_t n_anchor,
                      uint8_t *roles, float *importance, double *vs_out, double *hs_out)
{
    const int nh = layers * kv_heads, nq = nh * group;
    if (layers < 1 || kv_heads < 1 || group < 1 || n < 1 || top_k < 1 || n_voice < 0 || n_voice > nh || n_anchor < 0 ||
        n_anchor > n_voice)
        return triage_fail(WNW_ERR_INVALID, "bad sizes or counts");
    if (!sample || !hits || !sens || !roles || !importance) return triage_fail(WNW_ERR_INVALID, "NULL pointer");
    int ns = 0;
    for (int i = 0; i < n; ++i) {
        if (sample[i] < 0) return triage_fail(WNW_ERR_INVALID, "negative sample id");
        ns = std::max(ns, sample[i] + 1);
    }
    // per-sample means, then the mean over the samples present
    std::vector<double> hsum((size_t)ns * nq, 0.0), ssum((size_t)ns * nh, 0.0);
    std::vector<int> cnt(ns, 0);
    for (int i = 0; i < n; ++i) {
        const int s = sample[i];
        ++cnt[s];
        for (int m = 0; m < nq; ++m) hsum[(size_t)s * nq + m] += (double)hits[(size_t)i * nq + m] / top_k;
        for (int m = 0; m < nh; ++m) ssum[(size_t)s * nh + m] += (double)sens[(size_t)i * nh + m];
    }
    std::vector<double> hq(nq, 0.0), hs(nh, 0.0), vs(nh, 0.0), imp(nh);
    int used = 0;
    for (int s = 0; s < ns; ++s) {
        if (!cnt[s]) continue;
        ++used;
        for (int m = 0; m < nq; ++m) hq[m] += hsum[(size_t)s * nq + m] / cnt[s];
        for (int m = 0; m < nh; ++m) hs[m] += ssum[(size_t)s * nh + m] / cnt[s];
    }
    for (int m = 0; m < nq; ++m) hq[m] /= used;
    for (int m = 0; m < nh; ++m) hs[m] /= used;
    double mx = 0.0;
    for (int h = 0; h < nh; ++h) {
        double a = 0.0;
        for (int j = 0; j < group; ++j) a += hq[(size_t)h * group + j];
        vs[h] = a / group;
        imp[h] = vs[h] * hs[h];
        mx = std::max(mx, imp[h]);
    }
    std::vector<int> order(nh);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return imp[a] > imp[b]; });
    for (int r = 0; r < nh; ++r) roles[order[r]] = r < n_anchor ? WNW_ANCHOR : r < n_voice ? WNW_TIDAL : WNW_FIXED;
    for (int h = 0; h < nh; ++h) {
        importance[h] = mx > 0.0 ? (float)(imp[h] / mx) : 0.f;
        if (vs_out) vs_out[h] = vs[h];
        if (hs_out) hs_out[h] = hs[h];
    }
    return WNW_OK;
}

}  // extern "C"
