// Budget search over the wait map of device-constrained columns (Alg. 2's tail wait w_tail, Eq. 1's ramp slope beta),
// ten bisection steps per pass over the trace.
//
// Whether the device of a request is started, and whether it wins, are step functions of the searched parameter x:
// the wait w(l; x) is monotone in x (a minimum of monotone terms, every operation rounded monotonically), started =
// s > w and won = started and w + d < s change at most once as w grows.  The 2^D - 1 midpoints that the next D
// bisection steps can reach are sorted by construction (the in-order walk of the bisection tree), so a request's
// share of all of them is: its share of the first one, plus one change at the candidate where it starts to differ.
// A request that is the same at the first and the last candidate (nearly all of them from the second pass on: the
// bracket is down to 1/1024) is added to two sums in registers; another one finds its two candidates (a guess from their
// spacing, corrected by bisection where it is not the answer or next to it), with the operations of the dispatch pass
// itself, and adds its tokens to their LDS bins.  Prefix sums over the bins
// give every candidate's totals, exact integers, and the walk down the tree records the steps of the plain bisection.
//
//   k_bins_init     states, templates, candidates of the first pass; clears the device-wide bins; stages the table
//   k_search_bins   one pass (grid.y = search)
//   k_search_walk   bins -> totals, D recorded steps, candidates of the next pass (workgroup = search)
// The second pass also lists the requests whose outcome changes inside its bracket (one in 2^SB_DEPTH where the server TTFTs
// are spread out): the workgroup that walks its bins takes all remaining steps from that list, which its first
// round brings down to a few requests in LDS.  Small traces take all of it in one launch (k_small_wait_search).
//
// Bound: the first pass by its reads and LDS atomics, the others by latency.  4 10^6 requests, 32 steps: first pass 31 us (0.064 GB,
// 2.1 TB/s), second 23, its walk with 20 steps more 23, two empty passes 18, the evaluation 20; 115 us in all.  Four passes of
// eight steps: 40, 24, 22, 21 and 5 for each walk, 136 us; 100 000 requests 68 against 80 us, 2000: 38 against 76.
// (Candidates found by bisection alone: first pass 40 us.)
#include <math.h>
#include <string.h>

#include "disco_launch.h"
#include "disco_search_plan.h"
#include "disco_small.h"
#include "disco_stage.h"
#include "disco_state.h"

namespace {

constexpr int SB_CAND = 1 << SB_DEPTH;            // (2^SB_DEPTH - 1 candidates)
constexpr int SB_BLOCK = 1024;
constexpr int SB_MAX_BLOCKS = 512;                // two workgroups per CU
// Device-wide bins of a search, SB_COPIES copies: prompt tokens, output tokens, device prompt tokens and device
// output tokens at the first candidate, then the changes of the latter two by candidate.
constexpr int SB_HEAD = 4, SB_WORDS = SB_HEAD + 2 * SB_CAND, SB_COPIES = 4;
constexpr unsigned LIST_LDS = 2048;               // entries that a workgroup can add (one with more of them ends the list)
// Requests of one interval that the walk holds in LDS; with more of them its rounds go over the whole list.
constexpr unsigned WALK_LDS = 8192;

struct BinSpec { double target; float lo, hi; int which_param, which_acc; };
struct BinSpecs { BinSpec s[DISCO_MAX_COLS]; };

// Middle candidate in sorted order and the walk from it: a step to the left or right halves `step`.
struct TreePos { int idx, step; };
__device__ __forceinline__ TreePos tree_root(int depth) { return TreePos{(1 << (depth - 1)) - 1, 1 << (depth - 1) >> 1}; }
__device__ __forceinline__ void tree_down(TreePos& t, bool right) { t.idx += right ? t.step : -t.step; t.step >>= 1; }

// Sorted candidates of the next `depth` steps below the bracket of `st` (a thread each).
__device__ __forceinline__ void write_candidates(const SearchState& st, disco_policy p, float* cand, int depth)
{
    const int c = threadIdx.x;
    if (c >= (1 << depth) - 1) return;
    double lo = st.lo, hi = st.hi;
    TreePos t = tree_root(depth);
    for (;;) {
        search_set_mid(st.which_param, lo, hi, p);
        if (t.idx == c) break;
        const bool right = c > t.idx;
        search_halve(st.which_param, lo, hi, search_param(st.which_param, p), right);
        tree_down(t, right);
    }
    cand[c] = (float)search_param(st.which_param, p);
}

__device__ __forceinline__ SearchState bin_state(const BinSpec& b, int n_steps)
{
    SearchState s;
    s.lo = (double)b.lo; s.hi = (double)b.hi; s.target = b.target;
    s.which_param = b.which_param; s.which_acc = b.which_acc; s.step = 0; s.n_steps = n_steps;
    return s;
}

// Workgroup 0 stages the table (totals at their identity for the evaluation at the answers), the others start a search each.
__global__ __launch_bounds__(SB_BLOCK) void k_bins_init(PolTable host, BinSpecs specs, int n, int n_steps, SearchState* st, disco_policy* templ,
                                                        u64* __restrict__ bins, float* __restrict__ cand, unsigned* __restrict__ listed,
                                                        int depth, disco_policy* staged, unsigned* tickets, u64* totals)
{
    if (blockIdx.x == 0) {
        SelInit none;
        memset(&none, 0, sizeof(none));
        stage_table(host.p, n, staged, tickets, totals, none, 0, 1);
        return;
    }
    const int j = (int)blockIdx.x - 1;
    const SearchState s = bin_state(specs.s[j], n_steps);
    const disco_policy p = host.p[j];
    if (threadIdx.x == 0) { st[j] = s; templ[j] = p; listed[j] = 0u; }
    write_candidates(s, p, cand + j * SB_CAND, depth);
    u64* mine = bins + (size_t)j * SB_COPIES * SB_WORDS;
    for (int i = threadIdx.x; i < SB_COPIES * SB_WORDS; i += SB_BLOCK) mine[i] = 0ull;
}

// Started and won at one candidate (the operations of pair_eval<1>).
struct WaitOutcome { bool started, won; };
__device__ __forceinline__ WaitOutcome wait_outcome(const disco_policy& p, bool slope, float x, int l, float s, float d)
{
    const float beta = slope ? x : p.beta, tail = slope ? p.w_tail : x;
    const float ramp = beta * (float)l;
    float w = (ramp < tail) ? ramp : tail;            // a NaN ramp falls through to w_tail
    w = (l == p.l_mid) ? p.w_mid : w;
    w = (l <= p.l_th) ? 0.0f : w;
    const float at = w + d;
    WaitOutcome o;
    o.started = s > w;
    o.won = o.started && at < s;
    return o;
}

// The candidates in LDS, and their (all but) even spacing.
struct Candidates { const float* x; int M; float first, per; };
__device__ __forceinline__ Candidates candidates(const float* sc, int M)
{
    const float a = sc[0], z = sc[M - 1];
    return Candidates{sc, M, a, z > a ? (float)(M - 1) / (z - a) : 0.0f};
}

// First candidate at which `like_last` holds; it does not at the first one and does at the last.  `near`: where the wait
// crosses the value that decides -- the candidates are even up to rounding, so that one or its neighbour is the answer nearly
// always; bisection otherwise.  (Bisection alone: ten dependent reads of LDS per request in the first pass.)
template <class F>
__device__ __forceinline__ int first_like_last(const Candidates& c, float near, F&& like_last)
{
    int lo = 0, hi = c.M - 1;
    const int g = (int)fminf(fmaxf(ceilf((near - c.first) * c.per), 1.0f), (float)hi);       // (a NaN goes to 1)
    if (g < hi) { if (like_last(c.x[g])) hi = g; else lo = g; }
    if (hi == g) { if (g - 1 > lo) { if (like_last(c.x[g - 1])) hi = g - 1; else lo = g - 1; } }
    else if (g + 1 < hi) { if (like_last(c.x[g + 1])) hi = g + 1; else lo = g + 1; }
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (like_last(c.x[mid])) hi = mid; else lo = mid;
    }
    return hi;
}

// The interval between candidates in which a request's outcomes change: k between candidate k - 1 and candidate k, 0 below the
// first one, M behind the last one, NONE outside the bracket; started in the low half, won in the high one.
constexpr unsigned NONE = 0xFFFFu;

// A request's changes between the candidates into the bins; with the ends of the bracket also where they lie.
template <bool WHERE>
__device__ __forceinline__ unsigned add_changes(const disco_policy& p, bool slope, const Candidates& c, float lo, float hi, int l, int n, float s,
                                                float d, const WaitOutcome& a, u64* changes)
{
    const WaitOutcome z = wait_outcome(p, slope, c.x[c.M - 1], l, s, d);
    const float per_l = slope ? 1.0f / (float)l : 1.0f;
    unsigned ks = NONE, kw = NONE;
    if (a.started != z.started) {
        ks = (unsigned)first_like_last(c, s * per_l, [&](float x) { return wait_outcome(p, slope, x, l, s, d).started == z.started; });
        atomicAdd((unsigned long long*)&changes[ks], (unsigned long long)(z.started ? (u64)l : 0ull - (u64)l));
    }
    if (a.won != z.won) {
        kw = (unsigned)first_like_last(c, (s - d) * per_l, [&](float x) { return wait_outcome(p, slope, x, l, s, d).won == z.won; });
        atomicAdd((unsigned long long*)&changes[SB_CAND + kw], (unsigned long long)(z.won ? (u64)n : 0ull - (u64)n));
    }
    if (WHERE) {                                     // (an outcome changes once at most)
        const WaitOutcome at_lo = wait_outcome(p, slope, lo, l, s, d), at_hi = wait_outcome(p, slope, hi, l, s, d);
        ks = at_lo.started != a.started ? 0u : (at_hi.started != z.started ? (unsigned)c.M : ks);
        kw = at_lo.won != a.won ? 0u : (at_hi.won != z.won ? (unsigned)c.M : kw);
    }
    return ks | (kw << 16);
}

// list, listed: nullable; `from`: the step the pass starts at (a search that is further is done).
template <bool VEC>
__global__ __launch_bounds__(SB_BLOCK) void k_search_bins(TraceView tr, const SearchState* __restrict__ st,
                                                          const disco_policy* __restrict__ templ, const float* __restrict__ cand,
                                                          u64* __restrict__ bins, int M, int from, uint2* __restrict__ list, unsigned cap,
                                                          unsigned* __restrict__ listed)
{
    __shared__ float sc[SB_CAND];
    __shared__ u64 sb[SB_WORDS];
    __shared__ uint2 kept[LIST_LDS];
    __shared__ unsigned nkept, base;
    const int j = blockIdx.y;
    if (st[j].step != from) return;
    for (int i = threadIdx.x; i < SB_WORDS; i += SB_BLOCK) sb[i] = 0ull;
    if ((int)threadIdx.x < M) sc[threadIdx.x] = cand[j * SB_CAND + threadIdx.x];
    if (threadIdx.x == 0) nkept = 0u;
    const disco_policy p = templ[j];
    const bool slope = st[j].which_param == DISCO_PARAM_BETA;
    uint2* mylist = list ? list + (size_t)j * cap : nullptr;
    const float lo = (float)st[j].lo, hi = (float)st[j].hi;              // the bracket, which the candidates divide
    __syncthreads();
    const Candidates cd = candidates(sc, M);
    u64 tot_l = 0, tot_n = 0, base_pre = 0, base_dec = 0;
    const i64 ngroups = (tr.n_req + 3) >> 2;
    for (i64 g4 = (i64)blockIdx.x * SB_BLOCK + threadIdx.x; g4 < ngroups; g4 += (i64)gridDim.x * SB_BLOCK) {
        int l[4], n[4];
        float s[4], k[4];
        const i64 i0 = g4 * 4;
        if (VEC && i0 + 3 < tr.n_req) {
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
            for (int q = 0; q < 4; ++q) {            // requests past the end have no tokens: they add nothing
                const bool v = i0 + q < tr.n_req;
                l[q] = v ? tr.l[i0 + q] : 0; n[q] = v ? tr.n[i0 + q] : 0; s[q] = v ? tr.s[i0 + q] : 0.0f;
                k[q] = tr.k ? (v ? tr.k[i0 + q] : 0.0f) : tr.k_s;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float d = __fmaf_rn((float)l[q], k[q], tr.c);
            const WaitOutcome a = wait_outcome(p, slope, cd.first, l[q], s[q], d);
            tot_l += (u64)l[q]; tot_n += (u64)n[q];
            base_pre += a.started ? (u64)l[q] : 0ull;
            base_dec += a.won ? (u64)n[q] : 0ull;
            if (mylist == nullptr) {
                add_changes<false>(p, slope, cd, lo, hi, l[q], n[q], s[q], d, a, sb + SB_HEAD);
                continue;
            }
            const unsigned where = add_changes<true>(p, slope, cd, lo, hi, l[q], n[q], s[q], d, a, sb + SB_HEAD);
            if (where != (NONE | (NONE << 16)) && i0 + q < tr.n_req) {
                const uint2 entry = make_uint2((unsigned)(i0 + q), where);
                const unsigned at = atomicAdd(&nkept, 1u);
                if (at < LIST_LDS) kept[at] = entry;
            }
        }
    }
    const u64 head[SB_HEAD] = {wave_sum_u64(tot_l), wave_sum_u64(tot_n), wave_sum_u64(base_pre), wave_sum_u64(base_dec)};
    if ((threadIdx.x & 63) == 0)
        for (int f = 0; f < SB_HEAD; ++f) atomicAdd((unsigned long long*)&sb[f], (unsigned long long)head[f]);
    __syncthreads();
    u64* dst = bins + ((size_t)j * SB_COPIES + blockIdx.x % SB_COPIES) * SB_WORDS;
    for (int i = threadIdx.x; i < SB_WORDS; i += SB_BLOCK)
        if (sb[i]) atomicAdd((unsigned long long*)&dst[i], (unsigned long long)sb[i]);
    if (mylist == nullptr) return;
    const unsigned mine = nkept <= LIST_LDS ? nkept : 0u;
    if (threadIdx.x == 0) base = nkept ? atomicAdd(&listed[j], mine ? mine : cap + 1u) : 0u;
    __syncthreads();
    for (unsigned i = threadIdx.x; i < mine; i += SB_BLOCK)
        if (base + i < cap) mylist[base + i] = kept[i];
}

// What the workgroup that walks a search's bins holds in LDS.
struct WalkLds {
    u64 tot[2 * SB_CAND];          // changes by candidate, then the totals at every candidate
    u64 head[SB_HEAD], wsum[SB_BLOCK / 64], wave[4][SB_BLOCK / 64];
    float sc[SB_CAND];
    SearchState st;
    unsigned kept[WALK_LDS], nkept;
    int chosen;                    // interval between candidates that the steps have led to
};

// Changes in w.tot -> totals at every candidate: those at the first one (w.head[2], w.head[3]) plus the changes up to it.
__device__ __forceinline__ void changes_to_totals(WalkLds& w)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    constexpr int HALF = SB_BLOCK / 64 / 2;                  // waves per kind
    const u64 x0 = w.tot[2 * t], x1 = w.tot[2 * t + 1];
    u64 incl = x0 + x1;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned lo = (unsigned)__shfl_up((int)(unsigned)incl, d, 64), hi = (unsigned)__shfl_up((int)(unsigned)(incl >> 32), d, 64);
        if (lane >= d) incl += ((u64)hi << 32) | lo;
    }
    if (lane == 63) w.wsum[wave] = incl;
    __syncthreads();
    u64 below = incl - x0 - x1 + w.head[wave < HALF ? 2 : 3];
    for (int v = wave & ~(HALF - 1); v < wave; ++v) below += w.wsum[v];
    w.tot[2 * t] = below + x0; w.tot[2 * t + 1] = below + x0 + x1;
    __syncthreads();
}

// `depth` recorded steps from the totals (thread 0; all threads meet the barrier).
__device__ __forceinline__ void take_steps(WalkLds& w, int depth, const disco_cost_params& cost, disco_search_out* o)
{
    if (threadIdx.x == 0) {
        SearchState st = w.st;
        TreePos pos = tree_root(depth);
        int chosen = 0;
        for (int d = 0; d < depth; ++d) {
            const u64 d_pre = w.tot[pos.idx], d_dec = w.tot[SB_CAND + pos.idx];
            const double A = acc_value(st.which_acc, cost, (i64)w.head[0], (i64)(w.head[1] - d_dec), (i64)d_pre, (i64)d_dec);
            const double mid = (double)w.sc[pos.idx];
            const bool above = A > st.target;
            o->hist_param[st.step] = mid;
            o->hist_acc[st.step] = A;
            search_halve(st.which_param, st.lo, st.hi, mid, above);
            st.step += 1;
            chosen = pos.idx + (above ? 1 : 0);
            tree_down(pos, above);
        }
        w.st = st;
        w.chosen = chosen;
        w.nkept = 0u;
    }
    __syncthreads();
}

// After take_steps: the requests whose outcome changes in the chosen interval are the only ones that still matter.  Entry e is
// request of(e), its intervals where(e); w.kept, w.nkept on return (all threads).
template <class Of, class Where>
__device__ __forceinline__ void keep_open(WalkLds& w, unsigned count, Of&& of, Where&& where)
{
    const unsigned k = (unsigned)w.chosen;
    for (unsigned e = threadIdx.x; e < count; e += SB_BLOCK) {
        const unsigned x = where(e);
        if ((x & 0xFFFFu) == k || (x >> 16) == k) {
            const unsigned at = atomicAdd(&w.nkept, 1u);
            if (at < WALK_LDS) w.kept[at] = of(e);
        }
    }
    __syncthreads();
}
// A candidate at an end of the chosen interval, where the totals are known.
__device__ __forceinline__ int known_end(const WalkLds& w) { return w.chosen > 0 ? w.chosen - 1 : 0; }

// All remaining steps by one workgroup, SB_DEPTH of them per round over its requests: all of the trace (ALL), of a list in
// device memory, or (from_lds) those in w.kept.  Of a list w.head holds the totals of all requests at x_base, with these
// ones' outcomes there.  ALL: `where` takes a word per request, and the rounds behind the first go on with those whose outcome
// changes in the chosen interval.
template <bool ALL>
__device__ __forceinline__ void rounds(const TraceView& tr, const uint2* __restrict__ list, unsigned count, bool from_lds, const disco_policy& p,
                                       float x_base, const disco_cost_params& cost, WalkLds& w, unsigned* where, disco_search_out* o)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const bool slope = w.st.which_param == DISCO_PARAM_BETA;
    u64 all_pre = w.head[2], all_dec = w.head[3];
    __syncthreads();
#pragma unroll 1
    while (w.st.step < w.st.n_steps) {
        const int left = w.st.n_steps - w.st.step, depth = left < SB_DEPTH ? left : SB_DEPTH;
        const bool listed = !ALL || from_lds;
        for (int i = t; i < 2 * SB_CAND; i += SB_BLOCK) w.tot[i] = 0ull;
        write_candidates(w.st, p, w.sc, depth);
        const float lo = (float)w.st.lo, hi = (float)w.st.hi;
        __syncthreads();
        const Candidates cd = candidates(w.sc, (1 << depth) - 1);
        u64 sum[4] = {0, 0, 0, 0};                           // prompt and output tokens, device prompt and output tokens at the first candidate
        constexpr int U = 4;
#pragma unroll 1
        for (unsigned e0 = (unsigned)t; e0 < count; e0 += U * SB_BLOCK) {
            int l[U], n[U];
            float s[U], k[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const unsigned e = e0 + q * SB_BLOCK < count ? e0 + q * SB_BLOCK : e0;
                const i64 i = from_lds ? (i64)w.kept[e] : (ALL ? (i64)e : (i64)list[e].x);
                l[q] = tr.l[i]; n[q] = tr.n[i]; s[q] = tr.s[i]; k[q] = tr.k ? tr.k[i] : tr.k_s;
            }
#pragma unroll 1
            for (int q = 0; q < U; ++q) {
                const unsigned e = e0 + q * SB_BLOCK;
                if (e >= count) break;
                const int lq = q == 0 ? l[0] : (q == 1 ? l[1] : (q == 2 ? l[2] : l[3])), nq = q == 0 ? n[0] : (q == 1 ? n[1] : (q == 2 ? n[2] : n[3]));
                const float sq = q == 0 ? s[0] : (q == 1 ? s[1] : (q == 2 ? s[2] : s[3])), kq = q == 0 ? k[0] : (q == 1 ? k[1] : (q == 2 ? k[2] : k[3]));
                const float d = __fmaf_rn((float)lq, kq, tr.c);
                const WaitOutcome a = wait_outcome(p, slope, cd.first, lq, sq, d);
                sum[0] += (u64)lq; sum[1] += (u64)nq;
                sum[2] += a.started ? (u64)lq : 0ull; sum[3] += a.won ? (u64)nq : 0ull;
                if (listed) {
                    const WaitOutcome b = wait_outcome(p, slope, x_base, lq, sq, d);
                    sum[2] -= b.started ? (u64)lq : 0ull; sum[3] -= b.won ? (u64)nq : 0ull;
                }
                const unsigned x = add_changes<ALL>(p, slope, cd, lo, hi, lq, nq, sq, d, a, w.tot);
                if (ALL && !from_lds) where[e] = x;
            }
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) { const u64 x = wave_sum_u64(sum[f]); if (lane == 0) w.wave[f][wave] = x; }
        __syncthreads();
        if (t < 4) {
            u64 x = 0ull;
            for (int v = 0; v < SB_BLOCK / 64; ++v) x += w.wave[t][v];
            if (t >= 2) w.head[t] = x + (listed ? (t == 2 ? all_pre : all_dec) : 0ull);
            else if (!listed) w.head[t] = x;
        }
        __syncthreads();
        changes_to_totals(w);
        take_steps(w, depth, cost, o);
        if (ALL && !from_lds) {
            keep_open(w, count, [&](unsigned e) { return e; }, [&](unsigned e) { return where[e]; });
            static_assert(WAIT_SMALL_REQ <= WALK_LDS, "all of the trace fits w.kept");
            from_lds = true;
            count = w.nkept;
            const int at = known_end(w);
            x_base = w.sc[at];
            all_pre = w.tot[at]; all_dec = w.tot[SB_CAND + at];
            __syncthreads();
        }
    }
}

// depth: steps of the pass that has run; next: those of the pass to come, 0 after the last one.  list: the requests whose
// outcome changes inside the bracket of this pass (nullable: none listed); up to
// `cap` of them, all remaining steps are taken here.
__global__ __launch_bounds__(SB_BLOCK) void k_search_walk(TraceView tr, SearchState* st_, const disco_policy* __restrict__ templ, disco_policy* pol,
                                                          float* __restrict__ cand, u64* __restrict__ bins, disco_search_out* sout,
                                                          disco_cost_params cost, int depth, int next, int from,
                                                          const uint2* __restrict__ list, unsigned cap, const unsigned* __restrict__ listed)
{
    __shared__ WalkLds w;
    const int j = blockIdx.x, t = threadIdx.x;
    u64* mine = bins + (size_t)j * SB_COPIES * SB_WORDS;
    float* cj = cand + j * SB_CAND;
    // (everything is fetched side by side, before the first of it is looked at)
    const SearchState was = st_[j];
    const disco_policy p = templ[j];
    const unsigned count = list ? listed[j] : 0u;
    const float c_t = cj[t];
    u64 x[2] = {0ull, 0ull}, h = 0ull;
#pragma unroll
    for (int k = 0; k < SB_COPIES; ++k) {
        x[0] += mine[k * SB_WORDS + SB_HEAD + t];
        x[1] += mine[k * SB_WORDS + SB_HEAD + SB_CAND + t];
        if (t < SB_HEAD) h += mine[k * SB_WORDS + t];
    }
    if (was.step != from) return;
    static_assert(SB_CAND == SB_BLOCK, "a thread per candidate");
    w.sc[t] = t < (1 << depth) - 1 ? c_t : 0.0f;
    w.tot[t] = x[0]; w.tot[SB_CAND + t] = x[1];
    if (t < SB_HEAD) w.head[t] = h;
    if (t == 0) w.st = was;
    __syncthreads();
    changes_to_totals(w);
    take_steps(w, depth, cost, &sout[j]);
    const bool rest = list != nullptr && count <= cap;
    if (rest) {
        const uint2* mylist = list + (size_t)j * cap;
        keep_open(w, count, [&](unsigned e) { return mylist[e].x; }, [&](unsigned e) { return mylist[e].y; });
        const bool few = w.nkept <= WALK_LDS;                // (else all of the list, against the first candidate)
        const int at = few ? known_end(w) : 0;
        const float x_base = w.sc[at];
        if (t == 0) { w.head[2] = w.tot[at]; w.head[3] = w.tot[SB_CAND + at]; }
        __syncthreads();
        rounds<false>(tr, mylist, few ? w.nkept : count, few, p, x_base, cost, w, nullptr, &sout[j]);
    } else if (next > 0) {
        for (int i = t; i < SB_COPIES * SB_WORDS; i += SB_BLOCK) mine[i] = 0ull;      // (for the next pass)
    }
    const SearchState st = w.st;
    if (t == 0) st_[j] = st;
    if (next > 0 && !rest) write_candidates(st, p, cj, next);
    else if (t == 0) { disco_policy a = p; search_set_answer(st.which_param, st.hi, a); pol[j] = a; }
}

// Small traces, workgroup = search: every step from all requests, then the evaluation at the answer.
__global__ __launch_bounds__(SB_BLOCK) void k_small_wait_search(TraceView tr, PolTable host, BinSpecs specs, int n_steps, disco_cost_params cost,
                                                                disco_search_out* __restrict__ sout, disco_policy* __restrict__ pol_out,
                                                                disco_accum* __restrict__ acc)
{
    __shared__ WalkLds w;
    __shared__ ColumnLds col;
    __shared__ unsigned where[WAIT_SMALL_REQ];
    const int j = blockIdx.x;
    disco_policy p = host.p[j];
    if (threadIdx.x == 0) w.st = bin_state(specs.s[j], n_steps);
    if (threadIdx.x < SB_HEAD) w.head[threadIdx.x] = 0ull;
    __syncthreads();
    disco_search_out* o = &sout[j];
    rounds<true>(tr, nullptr, (unsigned)tr.n_req, false, p, 0.0f, cost, w, where, o);
    const SearchState st = w.st;
    search_set_answer(st.which_param, st.hi, p);
    ColumnSums sums;
    for_requests<true>(tr, [&](int i, int l, int n, float s, float d) { sums.add(l, n, pair_eval<1>(p, l, s, d, i)); });
    const disco_accum tot = wg_fold(sums, col);
    if (threadIdx.x != 0) return;
    o->param = st.hi;
    o->acc_at_param = acc_value(st.which_acc, cost, tot.s_pre, tot.s_dec, tot.d_pre, tot.d_dec);
    o->lo = st.lo;
    o->hi = st.hi;
    o->at_param = tot;
    if (pol_out) pol_out[j] = p;
    if (acc) store_dispatch_accum(&acc[j], tot);
}

BinSpecs bin_specs(const SpecTable& t, int n)
{
    BinSpecs b;
    memset(&b, 0, sizeof(b));
    for (int j = 0; j < n; ++j)
        b.s[j] = BinSpec{t.s[j].target, (float)t.s[j].lo, (float)t.s[j].hi, t.s[j].which_param, t.s[j].which_acc};
    return b;
}

}  // namespace

// Whether these passes beat the fused ones, which evaluate the next one to three levels of all searches as policy columns
// of one pass: these cost a read of the trace and two outcomes per request for every search and take ten steps, the cost
// of a fused pass grows with its columns alone.  One and two searches: these passes (never slower, 1 to 64 steps on 10 000
// to 10^6 requests, and 4 10^6 from 10 steps or with one search).  Beyond that the smaller of two estimates in microseconds,
// fitted to whole calls; where it errs, the calls differ by a tenth at most.  These passes against the fused ones, device
// prompt tokens, 10^6 requests:
//    4 searches  1 step  40 against 45 us,   4 steps  52 / 67,   16 steps  82 / 155,  32 steps 117 / 267
//   16 searches  1 step  66 / 59,            4 steps 110 / 87,   16 steps 184 / 265,  32 steps 215 / 499
//   64 searches  1 step 165 / 83,            4 steps 339 / 171,  16 steps 580 / 514,  32 steps 697 / 981
// and 64 searches at 4 10^6 requests 555 / 257 us (one step), 2859 / 3028 (32); at 10 000 requests 37 / 41 and 83 / 502.
// `decode`: some search's accumulator takes the output tokens too, which the fused passes then add up.
bool disco_search_bins_pays(i64 n_req, int n_search, int n_steps, bool decode)
{
    if (n_search <= 2) return true;
    const int depth = disco_search_depth(n_search);
    int cols = 1;
    while (cols < n_search * ((1 << depth) - 1)) cols <<= 1;
    const double n = 1e-6 * (double)n_req;
    const double fused = (n_steps + depth - 1) / depth * (12.0 + (decode ? 0.45 : 0.30) * n * cols);
    // (steps in the first two passes; an outcome that changes costs the more the fewer steps narrowed the bracket)
    double fixed = 6.0 + 0.5 * n_steps, per_search = n_steps == 1 ? 2.2 : (n_steps == 2 ? 3.7 : 4.8);
    if (n_steps > SB_DEPTH) { fixed = 26.0; per_search = n_steps >= 2 * SB_DEPTH - 2 ? 7.5 : 8.5; }
    if (n_steps > 2 * SB_DEPTH) { fixed += 12.0 + 0.95 * (n_steps - 2 * SB_DEPTH); per_search += 1.8 + 0.1 * (n_steps - 2 * SB_DEPTH); }
    return fixed + per_search * n * n_search < fused;
}

size_t disco_search_bins_bytes(int n_search)
{
    // (the list behind them starts at a multiple of 8)
    return (size_t)n_search * (SB_COPIES * SB_WORDS * sizeof(u64) + SB_CAND * sizeof(float) + 2 * sizeof(unsigned));
}

void disco_launch_small_wait_search(const TraceView& v, const PolTable& host, int n_search, int n_steps, const SpecTable& spec,
                                    const disco_cost_params& cost, disco_search_out* sout, disco_policy* pol_out, disco_accum* acc,
                                    hipStream_t stream)
{
    hipLaunchKernelGGL(k_small_wait_search, dim3((unsigned)n_search), dim3(SB_BLOCK), 0, stream, v, host, bin_specs(spec, n_search), n_steps, cost,
                       sout, pol_out, acc);
}

void disco_launch_search_bins(const TraceView& v, const PolTable& host, int n_search, int n_steps, const SpecTable& spec,
                              const disco_cost_params& cost, void* scratch, size_t scratch_bytes, SearchState* st, disco_policy* pol,
                              disco_policy* templ, unsigned* tickets, u64* totals, disco_search_out* sout, hipStream_t stream)
{
    u64* bins = (u64*)scratch;
    float* cand = (float*)(bins + (size_t)n_search * SB_COPIES * SB_WORDS);
    unsigned* listed = (unsigned*)(cand + (size_t)n_search * SB_CAND);
    uint2* list = (uint2*)((char*)scratch + disco_search_bins_bytes(n_search));
    const size_t room = (scratch_bytes - disco_search_bins_bytes(n_search)) / sizeof(uint2) / (size_t)n_search;
    const SearchPlan s = search_plan(v.n_req, n_search, n_steps, room);
    i64 b = (v.n_req + 4 * SB_BLOCK - 1) / (4 * SB_BLOCK);
    const i64 most = SB_MAX_BLOCKS / n_search > 8 ? SB_MAX_BLOCKS / n_search : 8;      // (every workgroup adds up to 2048 bins)
    if (b > most) b = most;
    b /= disco_grid_divisor();
    if (b < 1) b = 1;
    auto a16 = [](const void* q) { return ((uintptr_t)q & 15u) == 0; };
    const bool vec = a16(v.l) && a16(v.n) && a16(v.s) && (!v.k || a16(v.k));
    hipLaunchKernelGGL(k_bins_init, dim3((unsigned)n_search + 1u), dim3(SB_BLOCK), 0, stream, host, bin_specs(spec, n_search), n_search, n_steps, st,
                       templ, bins, cand, listed, s.depth[0], pol, tickets, totals);
    int from = 0;
    for (int pass = 0; pass < s.npass; ++pass) {
        const int M = (1 << s.depth[pass]) - 1;
        uint2* mylist = s.list && pass == 1 ? list : nullptr;
        if (vec) hipLaunchKernelGGL(k_search_bins<true>, dim3((unsigned)b, (unsigned)n_search), dim3(SB_BLOCK), 0, stream, v, st, templ, cand, bins, M, from, mylist, s.cap, listed);
        else hipLaunchKernelGGL(k_search_bins<false>, dim3((unsigned)b, (unsigned)n_search), dim3(SB_BLOCK), 0, stream, v, st, templ, cand, bins, M, from, mylist, s.cap, listed);
        hipLaunchKernelGGL(k_search_walk, dim3((unsigned)n_search), dim3(SB_BLOCK), 0, stream, v, st, templ, pol, cand, bins, sout, cost,
                           s.depth[pass], s.depth[pass + 1], from, mylist, s.cap, listed);
        from += s.depth[pass];
    }
}
