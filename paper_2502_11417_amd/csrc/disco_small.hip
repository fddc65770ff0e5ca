// Dispatch totals, tabulated threshold search and TTFT order statistics of
// small traces (disco_small.h): one launch each, workgroup = policy column.
#include <math.h>
#include <string.h>

#include "disco_final.h"
#include "disco_small.h"
#include "disco_stage.h"

namespace {

// Bound by latency, like all of this file: 6 us for 2000 requests, 13 for 32 000 (11 and 14 in the two kernels of the
// general pass).
__global__ __launch_bounds__(SM_BLOCK) void k_small_dispatch(TraceView tr, PolTable host, const disco_policy* __restrict__ device,
                                                             int P, disco_accum* __restrict__ acc, PairOut out)
{
    __shared__ ColumnLds lds;
    const int c = blockIdx.x;
    if (c >= P) {                                            // the workgroups behind the columns write the per-pair outputs
        mat_body(tr, device ? device : host.p, P, out, c - P, (int)gridDim.x - P);
        return;
    }
    const disco_policy p = device ? device[c] : host.p[c];
    ColumnSums sums;
    for_outcomes<true>(tr, p, [&](int, int l, int n, const PairResult& e) { sums.add(l, n, e); });
    const disco_accum a = wg_fold(sums, lds);
    if (threadIdx.x == 0) store_dispatch_accum(&acc[c], a);
}

// Threshold searches of server-constrained columns (workgroup = search): the prompt-token sums by length in LDS, the steps of
// the plain bisection, the evaluation at the answer.  12 us for 2000 requests x 4 searches, 21 - 25 for 32 000 (six
// launches of 3 - 8 us each in the general search).
__global__ __launch_bounds__(SM_BLOCK) void k_small_search(TraceView tr, PolTable templ, SmallSearches sp, int n_steps, int nbins,
                                                           disco_cost_params cost, disco_search_out* __restrict__ sout,
                                                           disco_policy* __restrict__ pol_out, disco_accum* __restrict__ acc)
{
    __shared__ SmallLenLds lds;
    __shared__ ColumnLds col;
    const int c = blockIdx.x;
    const SmallSearch st = sp.s[c];
    const SmallLenSums A = wg_len_sums(tr, nbins, lds);
    disco_search_out* o = &sout[c];
    const u64 all = A(0);
    int lo = st.lo, hi = st.hi;
    for (int step = 0; step < n_steps; ++step) {
        const int mid = lo + (hi - lo) / 2;
        const double a = (double)(i64)(st.which_acc == DISCO_ACC_SERVER_PREFILL_TOK ? A(mid) : all);
        if (threadIdx.x == 0) { o->hist_param[step] = (double)mid; o->hist_acc[step] = a; }
        if (lo < hi) { if (a > st.target) lo = mid + 1; else hi = mid; }
    }
    disco_policy p = templ.p[c];
    p.l_th = hi;                                             // the feasible end of the bracket
    ColumnSums sums;
    for_requests<true>(tr, [&](int i, int l, int n, float s, float d) { sums.add(l, n, pair_eval<0>(p, l, s, d, i)); });
    const disco_accum tot = wg_fold(sums, col);
    if (threadIdx.x != 0) return;
    o->param = (double)hi;
    o->acc_at_param = acc_value(st.which_acc, cost, tot.s_pre, tot.s_dec, tot.d_pre, tot.d_dec);
    o->lo = (double)lo;
    o->hi = (double)hi;
    o->at_param = tot;
    if (pol_out) pol_out[c] = p;
    if (acc) store_dispatch_accum(&acc[c], tot);
}

// The column's TTFTs as keys in LDS, then its quantiles.  (The general selection is nine launches: one for each digit's
// histograms, their sums and choices, and the passes that only the device can rule out: 45 - 60 us; here 6 us for 500
// requests, 15 for 16 000, 24 for 32 000.)  Without timelines the column's record follows at once (with_tl = 0); with
// them the workgroups behind the columns stage the table and start the TBT selection.
struct SmallBeginLds { RankLds rank; FinalLds fin; TtftFound found; };

__global__ __launch_bounds__(SM_BLOCK) void k_small_begin(TraceView tr, PolTable host, const disco_policy* __restrict__ device, int P,
                                                          disco_policy* __restrict__ staged, unsigned* __restrict__ tickets, SelInit si,
                                                          FinalArgs fin)
{
    __shared__ SmallBeginLds lds;
    const int c = blockIdx.x, n = (int)tr.n_req, nq = si.nq;
    SelState* S = si.S;
    if (c >= P) {
        // 0 the table, 1 start of the TBT selection, the others clear; no start of the TTFT selection
        static_assert(STAGE_THREADS == SM_BLOCK, "the kinds of workgroup share a launch");
        const int bid = c - P;
        stage_table(device ? device : host.p, P, staged, tickets, nullptr, si, bid > 0 ? bid + 1 : 0, (int)gridDim.x - P + 1);
        return;
    }
    const disco_policy p = device ? device[c] : host.p[c];
    const unsigned lo = si.acc[c].ttft_min_bits, hi = si.acc[c].ttft_max_bits;
    unsigned k[DISCO_MAX_Q] = {0u, 0u, 0u, 0u}, prefix[DISCO_MAX_Q] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < DISCO_MAX_Q; ++q)
        if (q < nq) k[q] = (unsigned)nearest_rank(si.q[q], tr.n_req);
    unsigned rank[DISCO_MAX_Q] = {k[0], k[1], k[2], k[3]};
    if (n > 0) {
        for_outcomes<false>(tr, p, [&](int i, int, int, const PairResult& e) { lds.rank.key[i] = f2u(e.ttft) - lo; });
        wg_select(lds.rank, n, hi > lo ? 32 - __clz(hi - lo) : 0, nq, k, prefix);
    }
    if (threadIdx.x == 0) {
        if (c == 0) { S->g[0].minb = 0u; S->g[0].gather_error = 0; }
#pragma unroll
        for (int q = 0; q < DISCO_MAX_Q; ++q)
            if (q < nq) {
                lds.found.rank[q] = (i64)rank[q];
                lds.found.q[q] = n > 0 ? u2f(prefix[q] + lo) : NAN;
                if (fin.with_tl) S->slot[0][c * nq + q] = SelSlot{prefix[q] + lo, n <= 0, 1, (i64)rank[q], tr.n_req};
            }
    }
    if (fin.with_tl) return;
    __syncthreads();
    stats_final(c, fin, lds.fin, nullptr, &lds.found);
}

}  // namespace

void disco_launch_small_dispatch(const TraceView& v, const PolTable& host, const disco_policy* device, int P, disco_accum* acc,
                                 uint8_t* decision, float* ttft, hipStream_t stream)
{
    const PairOut out{decision, ttft};
    const i64 tasks = decision || ttft ? (v.n_req + 4 * DP_BLOCK - 1) / (4 * DP_BLOCK) * ((P + MAT_COLS - 1) / MAT_COLS) : 0;
    hipLaunchKernelGGL(k_small_dispatch, dim3((unsigned)(P + tasks)), dim3(SM_BLOCK), 0, stream, v, host, device, P, acc, out);
}

void disco_launch_small_search(const TraceView& v, const PolTable& templ, const SmallSearches& sp, int n_search, int n_steps, int nbins,
                               const disco_cost_params& cost, disco_search_out* sout, disco_policy* pol_out, disco_accum* acc,
                               hipStream_t stream)
{
    hipLaunchKernelGGL(k_small_search, dim3((unsigned)n_search), dim3(SM_BLOCK), 0, stream, v, templ, sp, n_steps, nbins, cost, sout,
                       pol_out, acc);
}

void disco_launch_small_begin(const TraceView& v, const PolTable& host, const disco_policy* device, int P, disco_policy* staged,
                              unsigned* tickets, const SelInit& si, const FinalArgs& fin, hipStream_t stream)
{
    const unsigned others = fin.with_tl ? 2u + STAGE_CLEAR : 0u;
    hipLaunchKernelGGL(k_small_begin, dim3((unsigned)P + others), dim3(SM_BLOCK), 0, stream, v, host, device, P, staged, tickets, si, fin);
}
