// Totals of a table of threshold columns (Alg. 3) from its sorted thresholds.
//
// A request runs on the device alone in the columns whose threshold lies above its length and races in the others, so
// it is found among the sorted thresholds once and added to the bucket behind it: what it amounts to in a race and on the
// device alone.  A column takes the device-only sums of the buckets up to its rank and the race sums of the
// buckets above it.  Where the device wins the race the two are the same but for the prompt, and go to sums in registers.
//
// Bound: LDS atomics.  A bucket has BK_COPIES copies, one for every 16th lane, side by side, so that a wave's updates
// meet four to a bank whatever the lengths are.  10^6 requests x 64 columns 13 us, every pair for
// itself 25 (4 10^6: 23 and 85).
#pragma once
#include "disco_pair.h"

namespace {

constexpr int BK_COPIES = 16;
constexpr int BK_MAX = 65;                     // buckets: columns + 1

struct Buckets {
    u64 race_l[BK_MAX * BK_COPIES];            // prompt tokens
    u64 lost_n[BK_MAX * BK_COPIES];            // output tokens of the races the server wins
    double lost_d[BK_MAX * BK_COPIES], lost_s[BK_MAX * BK_COPIES];     // their TTFTs on the device and on the server
    unsigned lost_c[BK_MAX * BK_COPIES];       // their number
    uint4 range[BK_MAX * BK_COPIES];           // smallest and largest bit pattern of the device's TTFTs, of the server's
    __align__(16) int th[64];                                // thresholds in order, the largest integer behind them
    int order[64];                             // column of a rank
    u64 base[7][DP_WAVES];
    u64 res[7][64];
};

__device__ __forceinline__ u64 pack_range(unsigned lo, unsigned hi) { return ((u64)hi << 32) | lo; }
__device__ __forceinline__ u64 fold_range(u64 a, u64 b)
{
    return pack_range(min((unsigned)a, (unsigned)b), max((unsigned)(a >> 32), (unsigned)(b >> 32)));
}
constexpr u64 NO_RANGE = 0x00000000FFFFFFFFull;
__device__ __forceinline__ u64 add_f64_bits(u64 a, u64 b)
{
    return (u64)__double_as_longlong(__longlong_as_double((long long)a) + __longlong_as_double((long long)b));
}
// KIND 0: integers, 1: doubles, 2: ranges
template <int KIND>
__device__ __forceinline__ u64 fold_kind(u64 a, u64 b) { return KIND == 0 ? a + b : (KIND == 1 ? add_f64_bits(a, b) : fold_range(a, b)); }

// Wave: x of bucket `lane`, x64 of bucket 64.  Returns to lane r the fold of the buckets 0 .. r (UP) or of those above r.
template <int KIND, bool UP>
__device__ __forceinline__ u64 fold_buckets(u64 x, u64 x64, int lane)
{
    const u64 none = KIND == 2 ? NO_RANGE : 0ull;          // (0 is also the bits of 0.0)
    if (!UP) {
        const u64 above = __shfl_down((unsigned long long)x, 1, 64);
        x = lane == 63 ? x64 : above;
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const u64 y = UP ? __shfl_up((unsigned long long)x, m, 64) : __shfl_down((unsigned long long)x, m, 64);
        const bool in = UP ? lane >= m : lane + m < 64;
        x = fold_kind<KIND>(x, in ? y : none);
    }
    return x;
}

template <class T, int KIND, bool UP, class Bits>
__device__ __forceinline__ void fold_word_of(const T* a, int nb, u64* res, int lane, Bits&& bits)
{
    const u64 none = KIND == 2 ? NO_RANGE : 0ull;
    u64 x = none, x64 = none;
#pragma unroll
    for (int k = 0; k < BK_COPIES; ++k) {
        const int at = (k + lane) & (BK_COPIES - 1);
        if (lane < nb) x = fold_kind<KIND>(x, bits(a[lane * BK_COPIES + at]));
        if (nb > 64) x64 = fold_kind<KIND>(x64, bits(a[64 * BK_COPIES + at]));
    }
    res[lane] = fold_buckets<KIND, UP>(x, x64, lane);
}

// Workgroup `bid` of `nblk`; G: columns rounded up to a power of two.  Words of DispPartial by column to out[f * 64 + c].
// Returns false if the workgroup has no requests.
template <int G>
__device__ __forceinline__ bool threshold_buckets(const TraceView& tr, const disco_policy* __restrict__ pol, int P, int need, int bid, int nblk,
                                                  Buckets& w, u64* out)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const i64 ngroups = (tr.n_req + 3) >> 2, first = (i64)bid * DP_BLOCK;
    if (first >= ngroups) return false;
    const bool vec = (((uintptr_t)tr.l | (uintptr_t)tr.n | (uintptr_t)tr.s | (tr.k ? (uintptr_t)tr.k : 0u)) & 15u) == 0;
    int l[4], n[4];
    float s[4], k[4];
    auto load = [&](i64 g4) {
        const i64 i0 = g4 * 4;
        if (vec && i0 + 3 < tr.n_req) {
            const int4 lv = *reinterpret_cast<const int4*>(tr.l + i0);
            const int4 nv = *reinterpret_cast<const int4*>(tr.n + i0);
            const float4 sv = *reinterpret_cast<const float4*>(tr.s + i0);
            l[0] = lv.x; l[1] = lv.y; l[2] = lv.z; l[3] = lv.w;
            n[0] = nv.x; n[1] = nv.y; n[2] = nv.z; n[3] = nv.w;
            s[0] = sv.x; s[1] = sv.y; s[2] = sv.z; s[3] = sv.w;
            if (tr.k) {
                const float4 kv = *reinterpret_cast<const float4*>(tr.k + i0);
                k[0] = kv.x; k[1] = kv.y; k[2] = kv.z; k[3] = kv.w;
            } else { k[0] = k[1] = k[2] = k[3] = tr.k_s; }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool v = i0 + q < tr.n_req;
                l[q] = v ? tr.l[i0 + q] : 0; n[q] = v ? tr.n[i0 + q] : 0; s[q] = v ? tr.s[i0 + q] : 0.0f;
                k[q] = tr.k ? (v ? tr.k[i0 + q] : 0.0f) : tr.k_s;
            }
        }
    };
    i64 g4 = first + t;
    load(g4);                                  // (in flight while the table is sorted)
    const int mine = t < P ? pol[t < P ? t : 0].l_th : 0x7FFFFFFF;
    if (t < 64) w.th[t] = mine;
    for (int i = t; i < BK_MAX * BK_COPIES; i += DP_BLOCK) {
        w.race_l[i] = 0ull; w.lost_n[i] = 0ull; w.lost_d[i] = 0.0; w.lost_s[i] = 0.0; w.lost_c[i] = 0u;
        w.range[i] = make_uint4(0xFFFFFFFFu, 0u, 0xFFFFFFFFu, 0u);
    }
    __syncthreads();
    int rank = 0;
    if (t < P)
#pragma unroll
        for (int j = 0; j < G; j += 4) {
            const int4 x = *reinterpret_cast<const int4*>(&w.th[j]);
            rank += (x.x < mine || (x.x == mine && j < t)) + (x.y < mine || (x.y == mine && j + 1 < t)) +
                    (x.z < mine || (x.z == mine && j + 2 < t)) + (x.w < mine || (x.w == mine && j + 3 < t));
        }
    __syncthreads();
    if (t < P) { w.th[rank] = mine; w.order[rank] = t; }
    __syncthreads();
    u64 tot_l = 0, tot_n = 0, won_n = 0;
    unsigned tot_c = 0, won_c = 0;
    double won_t = 0.0;
    unsigned won_min = 0xFFFFFFFFu, won_max = 0u;
    const int copy = lane & (BK_COPIES - 1);
#pragma unroll 1
    for (;;) {
        const i64 left = tr.n_req - g4 * 4;
        int at[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) at[q] = 0;
#pragma unroll
        for (int step = G / 2; step > 0; step >>= 1)
#pragma unroll
            for (int q = 0; q < 4; ++q) at[q] += w.th[at[q] + step - 1] <= l[q] ? step : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) at[q] += w.th[at[q]] <= l[q] ? 1 : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q >= left) break;
            const float d = __fmaf_rn((float)l[q], k[q], tr.c);
            const int cell = (at[q] < P ? at[q] : P) * BK_COPIES + copy;
            tot_l += (u64)l[q]; tot_n += (u64)n[q]; tot_c += 1u;
            atomicAdd((unsigned long long*)&w.race_l[cell], (unsigned long long)l[q]);
            if (need < 1) continue;
            if (d < s[q]) {                                  // ties go to the server
                won_n += (u64)n[q]; won_c += 1u;
                won_t += (double)d;
                won_min = min(won_min, f2u(d)); won_max = max(won_max, f2u(d));
                continue;
            }
            atomicAdd((unsigned long long*)&w.lost_n[cell], (unsigned long long)n[q]);
            atomicAdd(&w.lost_c[cell], 1u);
            if (need < 2) continue;
            unsafeAtomicAdd(&w.lost_d[cell], (double)d);
            unsafeAtomicAdd(&w.lost_s[cell], (double)s[q]);
            const uint4 r = w.range[cell];                   // (bounds only ever widen: a stale one costs an update too many)
            unsigned* at_r = reinterpret_cast<unsigned*>(&w.range[cell]);
            if (f2u(d) < r.x) atomicMin(at_r, f2u(d));
            if (f2u(d) > r.y) atomicMax(at_r + 1, f2u(d));
            if (f2u(s[q]) < r.z) atomicMin(at_r + 2, f2u(s[q]));
            if (f2u(s[q]) > r.w) atomicMax(at_r + 3, f2u(s[q]));
        }
        g4 += (i64)nblk * DP_BLOCK;
        if (g4 >= ngroups) break;
        load(g4);
    }
    const u64 base[7] = {wave_sum_u64(tot_l), wave_sum_u64(tot_n), wave_sum_u64((u64)tot_c), wave_sum_u64(won_n), wave_sum_u64((u64)won_c),
                         (u64)__double_as_longlong(wave_sum_f64(won_t)), pack_range(wave_min_u32(won_min), wave_max_u32(won_max))};
    if (lane == 0)
        for (int f = 0; f < 7; ++f) w.base[f][wave] = base[f];
    __syncthreads();
    const int nb = P + 1;
    auto ident = [](u64 x) { return x; };
    auto dbits = [](double x) { return (u64)__double_as_longlong(x); };
    if (wave == 0) fold_word_of<u64, 0, false>(w.race_l, nb, w.res[0], lane, ident);
    else if (wave == 1) fold_word_of<u64, 0, true>(w.lost_n, nb, w.res[1], lane, ident);
    else if (wave == 2) fold_word_of<unsigned, 0, true>(w.lost_c, nb, w.res[2], lane, [](unsigned x) { return (u64)x; });
    else if (wave == 3) fold_word_of<double, 1, true>(w.lost_d, nb, w.res[3], lane, dbits);
    else if (wave == 4) fold_word_of<double, 1, false>(w.lost_s, nb, w.res[4], lane, dbits);
    else if (wave == 5) fold_word_of<uint4, 2, true>(w.range, nb, w.res[5], lane, [](const uint4& x) { return pack_range(x.x, x.y); });
    else if (wave == 6) fold_word_of<uint4, 2, false>(w.range, nb, w.res[6], lane, [](const uint4& x) { return pack_range(x.z, x.w); });
    else if (wave < 14 && lane == 0) {
        const int f = wave - 7;
        u64 x = w.base[f][0];
        for (int v = 1; v < DP_WAVES; ++v)
            x = f == 5 ? add_f64_bits(x, w.base[f][v]) : (f == 6 ? fold_range(x, w.base[f][v]) : x + w.base[f][v]);
        w.base[f][0] = x;
    }
    __syncthreads();
    if (wave < 8 && lane < P) {
        u64 x = 0ull;
        switch (wave) {
        case 0: x = w.res[0][lane]; break;
        case 1: x = w.base[0][0]; break;
        case 2: x = w.base[3][0] + w.res[1][lane]; break;
        case 3: x = w.base[1][0]; break;
        case 4: x = w.base[2][0]; break;
        case 5: x = w.base[4][0] + w.res[2][lane]; break;
        case 6: x = add_f64_bits(w.base[5][0], add_f64_bits(w.res[3][lane], w.res[4][lane])); break;
        default: x = fold_range(w.base[6][0], fold_range(w.res[5][lane], w.res[6][lane]));
        }
        out[wave * 64 + w.order[lane]] = x;
    }
    __syncthreads();
    return true;
}

}  // namespace
