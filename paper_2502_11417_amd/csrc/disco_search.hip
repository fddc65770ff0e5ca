// Budget search over the wait map of device-constrained columns (Alg. 2's tail wait w_tail, Eq. 1's ramp slope beta),
// eight bisection steps per pass over the trace.
//
// Whether the device of a request is started, and whether it wins, are step functions of the searched parameter x:
// the wait w(l; x) is monotone in x (a minimum of monotone terms, every operation rounded monotonically), started =
// s > w and won = started and w + d < s change at most once as w grows.  The 2^D - 1 midpoints that the next D
// bisection steps can reach are sorted by construction (the in-order walk of the bisection tree), so a request's
// share of all of them is: its share of the first one, plus one change at the candidate where it starts to differ.
// A request that is the same at the first and the last candidate (nearly all of them from the second pass on: the
// bracket is down to 1/256) is added to two sums in registers; another one finds its two candidates by bisection,
// with the operations of the dispatch pass itself, and adds its tokens to their LDS bins.  Prefix sums over the bins
// give every candidate's totals, exact integers, and the walk down the tree records the steps of the plain bisection.
//
//   k_bins_init     states, templates, candidates of the first pass; clears the device-wide bins
//   k_search_bins   one pass (grid.y = search)
//   k_search_walk   bins -> totals, D recorded steps, candidates of the next pass (workgroup = search)
//
// Bound: the first pass by its bisections and LDS atomics (42 us for 4 10^6 requests, 1.1 TB/s), the others by the
// latency of one read of 12-16 bytes per request (13-18 us, 2.7-3.7 TB/s out of the caches), the walks by latency
// (6-9 us).  32 steps over 4 10^6 requests: 138 us with the evaluation at the answer; 427 us in eleven passes of three
// steps each with seven policy columns (k_dispatch_acc<8>, 32 us a pass), which templates of other kinds still take, and
// many searches at once where those passes are the faster ones (disco_search_bins_pays).
#include <math.h>

#include "disco_launch.h"
#include "disco_state.h"

namespace {

constexpr int SB_DEPTH = 8;                       // bisection steps per pass, at most
constexpr int SB_CAND = 256;                      // 2^SB_DEPTH - 1 candidates
constexpr int SB_BLOCK = 1024;
constexpr int SB_MAX_BLOCKS = 512;                // two workgroups per CU
// Device-wide bins of a search, DISCO_NCOPY copies: prompt tokens, output tokens, device prompt tokens and device
// output tokens at the first candidate, then the changes of the latter two by candidate.
constexpr int SB_HEAD = 4, SB_WORDS = SB_HEAD + 2 * SB_CAND;

// Middle candidate in sorted order and the walk from it: a step to the left or right halves `step`.
struct TreePos { int idx, step; };
__device__ __forceinline__ TreePos tree_root(int depth) { return TreePos{(1 << (depth - 1)) - 1, 1 << (depth - 1) >> 1}; }
__device__ __forceinline__ void tree_down(TreePos& t, bool right) { t.idx += right ? t.step : -t.step; t.step >>= 1; }

// Sorted candidates of the next `depth` steps below the bracket of `st`.
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

__global__ __launch_bounds__(SB_CAND) void k_bins_init(SpecTable t, SearchState* st, const disco_policy* __restrict__ pol,
                                                       disco_policy* templ, u64* __restrict__ bins, float* __restrict__ cand, int depth)
{
    const int j = blockIdx.x;
    SearchState s = t.s[j];
    s.lo = (double)(float)s.lo; s.hi = (double)(float)s.hi;
    s.step = 0;
    const disco_policy p = pol[j];
    if (threadIdx.x == 0) { st[j] = s; templ[j] = p; }
    write_candidates(s, p, cand + j * SB_CAND, depth);
    u64* mine = bins + (size_t)j * DISCO_NCOPY * SB_WORDS;
    for (int i = threadIdx.x; i < DISCO_NCOPY * SB_WORDS; i += SB_CAND) mine[i] = 0ull;
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

template <bool VEC>
__global__ __launch_bounds__(SB_BLOCK) void k_search_bins(TraceView tr, const SearchState* __restrict__ st,
                                                          const disco_policy* __restrict__ templ, const float* __restrict__ cand,
                                                          u64* __restrict__ bins, int M)
{
    __shared__ float sc[SB_CAND];
    __shared__ u64 sb[SB_WORDS];
    const int j = blockIdx.y;
    for (int i = threadIdx.x; i < SB_WORDS; i += SB_BLOCK) sb[i] = 0ull;
    if ((int)threadIdx.x < M) sc[threadIdx.x] = cand[j * SB_CAND + threadIdx.x];
    const disco_policy p = templ[j];
    const bool slope = st[j].which_param == DISCO_PARAM_BETA;
    __syncthreads();
    const float x0 = sc[0], x1 = sc[M - 1];
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
            const WaitOutcome a = wait_outcome(p, slope, x0, l[q], s[q], d), z = wait_outcome(p, slope, x1, l[q], s[q], d);
            tot_l += (u64)l[q]; tot_n += (u64)n[q];
            base_pre += a.started ? (u64)l[q] : 0ull;
            base_dec += a.won ? (u64)n[q] : 0ull;
            if (a.started != z.started) {            // the first candidate that is like the last one
                int lo = 0, hi = M - 1;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (wait_outcome(p, slope, sc[mid], l[q], s[q], d).started == z.started) hi = mid; else lo = mid;
                }
                atomicAdd((unsigned long long*)&sb[SB_HEAD + hi], (unsigned long long)(z.started ? (u64)l[q] : 0ull - (u64)l[q]));
            }
            if (a.won != z.won) {
                int lo = 0, hi = M - 1;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (wait_outcome(p, slope, sc[mid], l[q], s[q], d).won == z.won) hi = mid; else lo = mid;
                }
                atomicAdd((unsigned long long*)&sb[SB_HEAD + SB_CAND + hi], (unsigned long long)(z.won ? (u64)n[q] : 0ull - (u64)n[q]));
            }
        }
    }
    const u64 head[SB_HEAD] = {wave_sum_u64(tot_l), wave_sum_u64(tot_n), wave_sum_u64(base_pre), wave_sum_u64(base_dec)};
    if ((threadIdx.x & 63) == 0)
        for (int f = 0; f < SB_HEAD; ++f) atomicAdd((unsigned long long*)&sb[f], (unsigned long long)head[f]);
    __syncthreads();
    u64* dst = bins + ((size_t)j * DISCO_NCOPY + blockIdx.x % DISCO_NCOPY) * SB_WORDS;
    for (int i = threadIdx.x; i < SB_WORDS; i += SB_BLOCK)
        if (sb[i]) atomicAdd((unsigned long long*)&dst[i], (unsigned long long)sb[i]);
}

// depth: steps of the pass that has run; next: those of the pass to come, 0 after the last one.
__global__ __launch_bounds__(2 * SB_CAND) void k_search_walk(SearchState* st_, const disco_policy* __restrict__ templ, disco_policy* pol,
                                                             float* __restrict__ cand, u64* __restrict__ bins, disco_search_out* sout,
                                                             disco_cost_params cost, int depth, int next)
{
    __shared__ u64 tot[2 * SB_CAND], head[SB_HEAD], wsum[2 * SB_CAND / 64];
    __shared__ float sc[SB_CAND];
    __shared__ SearchState sst;
    const int j = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    u64* mine = bins + (size_t)j * DISCO_NCOPY * SB_WORDS;
    float* cj = cand + j * SB_CAND;
    if (t < SB_CAND) sc[t] = t < (1 << depth) - 1 ? cj[t] : 0.0f;
    u64 x = 0ull;
#pragma unroll
    for (int k = 0; k < DISCO_NCOPY; ++k) x += mine[k * SB_WORDS + SB_HEAD + t];
    if (t < SB_HEAD) {
        u64 h = 0ull;
        for (int k = 0; k < DISCO_NCOPY; ++k) h += mine[k * SB_WORDS + t];
        head[t] = h;
    }
    // totals at candidate c: those at the first one plus the changes up to c
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned lo = (unsigned)__shfl_up((int)(unsigned)x, d, 64), hi = (unsigned)__shfl_up((int)(unsigned)(x >> 32), d, 64);
        if (lane >= d) x += ((u64)hi << 32) | lo;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    x += head[t < SB_CAND ? 2 : 3];
    for (int w = wave & ~(SB_CAND / 64 - 1); w < wave; ++w) x += wsum[w];
    tot[t] = x;
    for (int i = t; i < DISCO_NCOPY * SB_WORDS; i += 2 * SB_CAND) mine[i] = 0ull;      // (read above: for the next pass)
    __syncthreads();
    if (t == 0) {
        SearchState st = st_[j];
        disco_search_out* o = &sout[j];
        TreePos pos = tree_root(depth);
        for (int d = 0; d < depth; ++d) {
            const u64 d_pre = tot[pos.idx], d_dec = tot[SB_CAND + pos.idx];
            const double A = acc_value(st.which_acc, cost, (i64)head[0], (i64)(head[1] - d_dec), (i64)d_pre, (i64)d_dec);
            const double mid = (double)sc[pos.idx];
            const bool above = A > st.target;
            o->hist_param[st.step] = mid;
            o->hist_acc[st.step] = A;
            search_halve(st.which_param, st.lo, st.hi, mid, above);
            st.step += 1;
            tree_down(pos, above);
        }
        st_[j] = st;
        sst = st;
    }
    __syncthreads();
    disco_policy p = templ[j];
    if (next > 0) write_candidates(sst, p, cj, next);
    else if (t == 0) { search_set_answer(sst.which_param, sst.hi, p); pol[j] = p; }
}

}  // namespace

// Whether these passes beat the fused ones, which evaluate the next one to three levels of all searches as policy columns
// of one pass: these cost a read of the trace and two outcomes per request for every search and take eight steps, the cost
// of a fused pass grows with its columns alone.  One and two searches: these passes (never slower by more than 8 %, 1 to 64
// steps on 20 000 to 4 10^6 requests).  Beyond that the smaller of two estimates in microseconds, fitted to whole calls; where
// it errs, the calls differ by a tenth at most.  These passes against the fused ones, device prompt tokens, 10^6 requests:
//   16 searches  4 steps 120 against 87 us,  16 steps 268 / 264,  32 steps  366 / 495
//   32 searches  4 steps 203 / 117,          16 steps 474 / 360,  32 steps  642 / 684
//   64 searches  4 steps 372 / 169,          32 steps 1192 / 972, 64 steps 1786 / 1886
// and 64 searches at 4 10^6 requests 747 / 256 us (one step), 4339 / 2989 (32); at 20 000 requests 41 / 42 and 112 / 498.
// `decode`: some search's accumulator takes the output tokens too, which the fused passes then add up.
bool disco_search_bins_pays(i64 n_req, int n_search, int n_steps, bool decode)
{
    if (n_search <= 2) return true;
    const int depth = disco_search_depth(n_search);
    int cols = 1;
    while (cols < n_search * ((1 << depth) - 1)) cols <<= 1;
    const double n = 1e-6 * (double)n_req;
    const double fused = (n_steps + depth - 1) / depth * (12.0 + (decode ? 0.45 : 0.30) * n * cols);
    const int npass = (n_steps + SB_DEPTH - 1) / SB_DEPTH, first = (n_steps + npass - 1) / npass;
    double per_search = first <= 2 ? 2.6 : 2.0 + 0.65 * first;       // the first pass bisects, the later ones hardly
    if (npass > 1) per_search += 5.1 + 2.3 * (npass - 2);
    return 4.0 + 0.08 * n_search + 1.6 * first + 14.0 * (npass - 1) + per_search * n * n_search < fused;
}

size_t disco_search_bins_bytes(int n_search)
{
    return (size_t)n_search * (DISCO_NCOPY * SB_WORDS * sizeof(u64) + SB_CAND * sizeof(float));
}

void disco_launch_search_bins(const TraceView& v, int n_search, int n_steps, const SpecTable& spec, const disco_cost_params& cost,
                              void* scratch, SearchState* st, disco_policy* pol, disco_policy* templ, disco_search_out* sout,
                              hipStream_t stream)
{
    u64* bins = (u64*)scratch;
    float* cand = (float*)(bins + (size_t)n_search * DISCO_NCOPY * SB_WORDS);
    // the steps are shared out evenly over the passes they take
    const int npass = (n_steps + SB_DEPTH - 1) / SB_DEPTH;
    auto depth_of = [&](int pass) { return pass < npass ? n_steps / npass + (pass < n_steps % npass ? 1 : 0) : 0; };
    i64 b = (v.n_req + 4 * SB_BLOCK - 1) / (4 * SB_BLOCK);
    if (b > SB_MAX_BLOCKS) b = SB_MAX_BLOCKS;
    b /= disco_grid_divisor();
    if (b < 1) b = 1;
    auto a16 = [](const void* q) { return ((uintptr_t)q & 15u) == 0; };
    const bool vec = a16(v.l) && a16(v.n) && a16(v.s) && (!v.k || a16(v.k));
    hipLaunchKernelGGL(k_bins_init, dim3((unsigned)n_search), dim3(SB_CAND), 0, stream, spec, st, pol, templ, bins, cand, depth_of(0));
    for (int pass = 0; pass < npass; ++pass) {
        const int M = (1 << depth_of(pass)) - 1;
        if (vec) hipLaunchKernelGGL(k_search_bins<true>, dim3((unsigned)b, (unsigned)n_search), dim3(SB_BLOCK), 0, stream, v, st, templ, cand, bins, M);
        else hipLaunchKernelGGL(k_search_bins<false>, dim3((unsigned)b, (unsigned)n_search), dim3(SB_BLOCK), 0, stream, v, st, templ, cand, bins, M);
        hipLaunchKernelGGL(k_search_walk, dim3((unsigned)n_search), dim3(2 * SB_CAND), 0, stream, st, templ, pol, cand, bins, sout, cost,
                           depth_of(pass), depth_of(pass + 1));
    }
}
