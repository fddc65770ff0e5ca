// Traces of a few thousand requests: a workgroup per policy column, which
// takes every request of the trace, so that nothing has to be handed from
// launch to launch.  A call on such a trace is a chain of dependent launches
// of 3 - 15 us each whose work is a fraction of that (first reads of device
// memory, barriers, tickets): what counts is how few of them there are.
#pragma once
#include "disco_launch.h"
#include "disco_len.h"
#include "disco_pair.h"

namespace {

constexpr int SM_BLOCK = 1024;
constexpr int SM_WAVES = SM_BLOCK / 64;

// ------------------------------------------------------- order statistics --

// Ranks among up to SMALL_REQ keys in LDS: most-significant-digit-first radix selection by one workgroup, up to 10 bits
// at a time, one histogram per wanted rank once their prefixes may differ.
constexpr int SR_BITS = 10;
struct RankLds {
    unsigned key[SMALL_REQ];
    unsigned hist[DISCO_MAX_Q << SR_BITS];
    unsigned wsum[SM_WAVES], digit[DISCO_MAX_Q], rem[DISCO_MAX_Q];
};

// Inclusive prefix sums over the 64 lanes (as wave_incl_max_dpp).
__device__ __forceinline__ unsigned wave_incl_sum_u32(unsigned v, int lane)
{
    v += dpp_u32<0x111>(0u, v); v += dpp_u32<0x112>(0u, v); v += dpp_u32<0x114>(0u, v); v += dpp_u32<0x118>(0u, v);
    const unsigned t0 = (unsigned)bcast_i((int)v, 15), t1 = (unsigned)bcast_i((int)v, 31), t2 = (unsigned)bcast_i((int)v, 47);
    const int row = lane >> 4;
    return v + (row > 0 ? t0 : 0u) + (row > 1 ? t1 : 0u) + (row > 2 ? t2 : 0u);
}

// All threads; s.key[0 .. n) written (no barrier needed in between).  k: ranks from 1 (0: none, its prefix means
// nothing); on return prefix[z] = the key of rank k[z], if all keys have at most nbits bits (other keys are counted
// nowhere they could be chosen from, and nothing is read out of bounds).
__device__ __forceinline__ void wg_select(RankLds& s, int n, int nbits, int nq, unsigned k[DISCO_MAX_Q], unsigned prefix[DISCO_MAX_Q])
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int z = t >> 8, tt = t & 255;                      // a quarter of the workgroup scans a rank's histogram
    static_assert(DISCO_MAX_Q == 4 && SM_BLOCK == 1024, "a quarter of the workgroup per rank");
#pragma unroll
    for (int q = 0; q < DISCO_MAX_Q; ++q) prefix[q] = 0u;
    bool first = true;
    int left = nbits;
#pragma unroll 1
    while (left > 0) {
        const int passes = (left + SR_BITS - 1) / SR_BITS, w = (left + passes - 1) / passes, sh = left - w;
        const int bins = 1 << w, dm = bins - 1;
        for (int i = t; i < (first ? bins : nq * bins); i += SM_BLOCK) s.hist[i] = 0u;
        if (t < DISCO_MAX_Q) { s.digit[t] = (unsigned)dm; s.rem[t] = 1u; }
        __syncthreads();
        if (first) {
#pragma unroll 4
            for (int i = t; i < n; i += SM_BLOCK) atomicAdd(&s.hist[(s.key[i] >> sh) & (unsigned)dm], 1u);
        } else {
#pragma unroll 2
            for (int i = t; i < n; i += SM_BLOCK) {
                const unsigned key = s.key[i], hi = key >> left, d = (key >> sh) & (unsigned)dm;
#pragma unroll
                for (int q = 0; q < DISCO_MAX_Q; ++q)
                    if (q < nq && hi == prefix[q]) atomicAdd(&s.hist[(q << w) + (int)d], 1u);
            }
        }
        __syncthreads();
        const int per = bins >= 256 ? bins >> 8 : 1;
        const unsigned* row = s.hist + ((first ? 0 : z) << w);
        const bool on = z < nq && tt * per < bins;
        unsigned mine = 0u;
        if (on) for (int b = 0; b < per; ++b) mine += row[tt * per + b];
        const unsigned incl = wave_incl_sum_u32(mine, lane);
        if (lane == 63) s.wsum[wave] = incl;
        __syncthreads();
        unsigned below = incl - mine;
        for (int v = wave & ~3; v < wave; ++v) below += s.wsum[v];
        const unsigned kz = z == 0 ? k[0] : (z == 1 ? k[1] : (z == 2 ? k[2] : k[3]));
        if (on && below < kz && below + mine >= kz) {        // at most one thread of the quarter
            int b = 0;
            for (; b < per - 1; ++b) {
                const unsigned c = row[tt * per + b];
                if (below + c >= kz) break;
                below += c;
            }
            s.digit[z] = (unsigned)(tt * per + b); s.rem[z] = kz - below;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < DISCO_MAX_Q; ++q) { prefix[q] = (prefix[q] << w) | s.digit[q]; k[q] = s.rem[q]; }
        left = sh;
        first = false;
        __syncthreads();
    }
}

// The requests of the trace, SM_BATCH strides of the workgroup at a time: all loads of a batch are issued before the first
// is used (the trace lies in the caches; one load after the other is what such a kernel would wait for).
// f(i, l, n, s, d); OUT: output lengths wanted.
constexpr int SM_BATCH = 8;
template <bool OUT, class F>
__device__ __forceinline__ void for_requests(const TraceView& tr, F&& f)
{
    const int n = (int)tr.n_req;
#pragma unroll 1
    for (int base = (int)threadIdx.x; base < n; base += SM_BATCH * SM_BLOCK) {
        int l[SM_BATCH], nn[SM_BATCH];
        float s[SM_BATCH], k[SM_BATCH];
#pragma unroll
        for (int q = 0; q < SM_BATCH; ++q) {
            const int i = base + q * SM_BLOCK, at = i < n ? i : base;
            l[q] = tr.l[at];
            nn[q] = OUT ? tr.n[at] : 0;
            s[q] = tr.s[at];
            k[q] = tr.k ? tr.k[at] : tr.k_s;
        }
#pragma unroll
        for (int q = 0; q < SM_BATCH; ++q) {
            const int i = base + q * SM_BLOCK;
            if (i < n) f(i, l[q], nn[q], s[q], __fmaf_rn((float)l[q], k[q], tr.c));
        }
    }
}
// The same one request at a time, for outcomes that take a draw of their own.
template <bool OUT, class F>
__device__ __forceinline__ void for_requests_narrow(const TraceView& tr, F&& f)
{
    const int n = (int)tr.n_req;
#pragma unroll 1
    for (int i = (int)threadIdx.x; i < n; i += SM_BLOCK) {
        const int l = tr.l[i];
        f(i, l, OUT ? tr.n[i] : 0, tr.s[i], __fmaf_rn((float)l, tr.k ? tr.k[i] : tr.k_s, tr.c));
    }
}
// f(i, l, n, outcome) for a column; the kind of the column is the same for the whole workgroup.
template <bool OUT, class F>
__device__ __forceinline__ void for_outcomes(const TraceView& tr, const disco_policy& p, F&& f)
{
    if (p.mode == DISCO_MODE_SERVER_CONSTRAINED)
        for_requests<OUT>(tr, [&](int i, int l, int n, float s, float d) { f(i, l, n, pair_eval<0>(p, l, s, d, i)); });
    else if (p.mode == DISCO_MODE_DEVICE_CONSTRAINED)
        for_requests<OUT>(tr, [&](int i, int l, int n, float s, float d) { f(i, l, n, pair_eval<1>(p, l, s, d, i)); });
    else
        for_requests_narrow<OUT>(tr, [&](int i, int l, int n, float s, float d) { f(i, l, n, pair_eval<2>(p, l, s, d, i)); });
}

// ---------------------------------------------------------- column totals --

// Totals of one column over all requests (all threads); the first wave returns with them.
struct ColumnLds { u64 w[8][SM_WAVES]; };

struct ColumnSums {
    u64 s_pre = 0, d_pre = 0, d_dec = 0, n_tot = 0, started = 0, won = 0;
    double ts = 0.0;
    unsigned mn = 0xFFFFFFFFu, mx = 0u;
    __device__ __forceinline__ void add(int l, int n, const PairResult& e)
    {
        s_pre += e.srv_started ? (u64)l : 0ull;
        d_pre += e.dev_started ? (u64)l : 0ull;
        started += e.dev_started ? 1ull : 0ull;
        d_dec += e.dev_win ? (u64)n : 0ull;
        won += e.dev_win ? 1ull : 0ull;
        n_tot += (u64)n;
        ts += (double)e.ttft;
        mn = min(mn, f2u(e.ttft)); mx = max(mx, f2u(e.ttft));
    }
};

__device__ __forceinline__ disco_accum wg_fold(const ColumnSums& c, ColumnLds& s)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u64 v[8] = {wave_sum_u64(c.s_pre), wave_sum_u64(c.d_pre), wave_sum_u64(c.d_dec), wave_sum_u64(c.n_tot), wave_sum_u64(c.started),
                      wave_sum_u64(c.won), (u64)__double_as_longlong(wave_sum_f64(c.ts)),
                      (u64)wave_min_u32(c.mn) | ((u64)wave_max_u32(c.mx) << 32)};
    if (lane == 0)
#pragma unroll
        for (int f = 0; f < 8; ++f) s.w[f][wave] = v[f];
    __syncthreads();
    disco_accum a;
    memset(&a, 0, sizeof(a));
    if (wave != 0) return a;
    // lane = wave whose part it holds; the order of the additions is fixed
    u64 x[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) x[f] = wave_sum_u64(lane < SM_WAVES ? s.w[f][lane] : 0ull);
    a.s_pre = (i64)x[0]; a.d_pre = (i64)x[1]; a.d_dec = (i64)x[2]; a.s_dec = (i64)(x[3] - x[2]);
    a.n_dev_started = (i64)x[4]; a.n_dev_win = (i64)x[5];
    a.ttft_sum = wave_sum_f64(lane < SM_WAVES ? __longlong_as_double((long long)s.w[6][lane]) : 0.0);
    a.ttft_min_bits = wave_min_u32(lane < SM_WAVES ? (unsigned)s.w[7][lane] : 0xFFFFFFFFu);
    a.ttft_max_bits = wave_max_u32(lane < SM_WAVES ? (unsigned)(s.w[7][lane] >> 32) : 0u);
    return a;
}

// Leaves the dispatch part of an accumulator (its timeline part is another call's).
__device__ __forceinline__ void store_dispatch_accum(disco_accum* o, const disco_accum& a)
{
    o->s_pre = a.s_pre; o->s_dec = a.s_dec; o->d_pre = a.d_pre; o->d_dec = a.d_dec;
    o->n_dev_started = a.n_dev_started; o->n_dev_win = a.n_dev_win; o->ttft_sum = a.ttft_sum;
    o->ttft_min_bits = a.ttft_min_bits; o->ttft_max_bits = a.ttft_max_bits;
}

// ---------------------------------------------------- prompt-token sums ----

// A(L) = prompt tokens of the requests of length >= L, for lengths 0 .. nbins - 1 in LDS (and `beyond`, those of longer
// prompts): SMALL_REQ requests of less than 2^15 tokens add up to less than 2^32.
constexpr int SL_BINS = LEN_MAX_BINS, SL_PER = (SL_BINS + SM_BLOCK - 1) / SM_BLOCK;
static_assert((u64)SMALL_REQ * SL_BINS < (1ull << 32), "sums of 32 bits");
struct SmallLenLds { unsigned a[SL_PER * SM_BLOCK]; unsigned wsum[SM_WAVES]; u64 beyond[SM_WAVES]; };

struct SmallLenSums {
    const unsigned* a;
    u64 beyond;
    int nbins;
    __device__ __forceinline__ u64 operator()(int L) const
    {
        if (L < 0) L = 0;
        return L < nbins ? (u64)a[L] + beyond : beyond;
    }
};

// All threads; nbins <= SL_BINS.
__device__ __forceinline__ SmallLenSums wg_len_sums(const TraceView& tr, int nbins, SmallLenLds& s)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, n = (int)tr.n_req;
    for (int i = t; i < nbins; i += SM_BLOCK) s.a[i] = 0u;
    __syncthreads();
    u64 out = 0;
#pragma unroll 1
    for (int base = t; base < n; base += SM_BATCH * SM_BLOCK) {
        int l[SM_BATCH];
#pragma unroll
        for (int q = 0; q < SM_BATCH; ++q) l[q] = base + q * SM_BLOCK < n ? tr.l[base + q * SM_BLOCK] : -1;
#pragma unroll
        for (int q = 0; q < SM_BATCH; ++q) {
            if (l[q] >= 0 && l[q] < nbins) atomicAdd(&s.a[l[q]], 1u);
            else if (l[q] > 0) out += (u64)l[q];
        }
    }
    out = wave_sum_u64(out);
    if (lane == 0) s.beyond[wave] = out;
    __syncthreads();
    // consecutive lengths per thread, an odd number of them: no bank conflicts
    const int per = ((nbins + SM_BLOCK - 1) / SM_BLOCK) | 1, v0 = t * per, v1 = min(v0 + per, nbins);
    unsigned mine = 0u;
    for (int v = v0; v < v1; ++v) mine += s.a[v] * (unsigned)v;
    const unsigned incl = wave_incl_sum_u32(mine, lane);
    if (lane == 63) s.wsum[wave] = incl;
    __syncthreads();
    unsigned upto = incl, all = 0u;
    u64 beyond = 0ull;
    for (int w = 0; w < SM_WAVES; ++w) { all += s.wsum[w]; upto += w < wave ? s.wsum[w] : 0u; beyond += s.beyond[w]; }
    unsigned above = all - upto;                             // tokens of the lengths behind this thread's
    for (int v = v1 - 1; v >= v0; --v) { above += s.a[v] * (unsigned)v; s.a[v] = above; }
    __syncthreads();
    return SmallLenSums{s.a, beyond, nbins};
}

}  // namespace
