// Staging of a call's policy table in its workspace and the start of the
// order-statistic selections, by one launch (workgroups by kind).
#pragma once
#include "disco_launch.h"
#include "disco_state.h"

namespace {

// The timeline totals follow the dispatch totals in the same workspace region.
__host__ __device__ inline MigPartial* tl_totals(u64* totals)
{
    return reinterpret_cast<MigPartial*>(totals + DISCO_NCOPY * 64 * 8);
}

// Start of a selection (all threads of one workgroup): one thread per slot: rank from (num, den, M), empty
// prefix; plan of the passes.
constexpr int STAGE_CLEAR = 61;    // workgroups that clear them

// Nearest rank of a quantile among M values, 0 if there are none.
__device__ __forceinline__ i64 nearest_rank(const disco_quantile& q, i64 M)
{
    i64 k = M > 0 ? ((i64)q.num * M + q.den - 1) / q.den : 0;
    if (M > 0 && k < 1) k = 1;
    return k > M ? M : k;
}

__device__ void select_init(const SelInit& si, int which, int P, const disco_policy* pol)
{
    SelState* S = si.S;
    const int nq = si.nq;
    const disco_accum* acc = si.acc;
    const i64 n_req = si.n_req;
    const disco_quantile qs[4] = {si.q[0], si.q[1], si.q[2], si.q[3]};
    __shared__ unsigned smin, smax;
    __shared__ int all_thresholds;
    if (threadIdx.x == 0) { smin = 0xFFFFFFFFu; smax = 0u; all_thresholds = 1; }
    if (which == 0) {
        // a table of length-threshold columns (Alg. 3) is selected by classes: thresholds in ascending order
        const int t = threadIdx.x;
        __shared__ __align__(16) int lth_s[DISCO_MAX_COLS];
        unsigned lo = 0u, hi = 0u;
        int mode = 0, lth = 0;
        if (t < P) { mode = pol[t].mode; lth = pol[t].l_th; lo = acc[t].ttft_min_bits; hi = acc[t].ttft_max_bits; }
        if (t < DISCO_MAX_COLS) lth_s[t] = t < P ? lth : 0x7FFFFFFF;
        __syncthreads();
        if (t < P) {
            if (mode != DISCO_MODE_SERVER_CONSTRAINED) all_thresholds = 0;
            atomicMin(&smin, lo);
            atomicMax(&smax, hi);
            int rank = 0;
#pragma unroll
            for (int k = 0; k < DISCO_MAX_COLS; k += 4) {          // (the ones behind the table are never in front)
                const int4 x = *reinterpret_cast<const int4*>(&lth_s[k]);
                rank += (x.x < lth || (x.x == lth && k < t)) + (x.y < lth || (x.y == lth && k + 1 < t)) +
                        (x.z < lth || (x.z == lth && k + 2 < t)) + (x.w < lth || (x.w == lth && k + 3 < t));
            }
            S->tc.sorted_lth[rank] = lth;
            S->tc.col_of_pos[rank] = (unsigned char)t;
            S->tc.pos_of_col[t] = (unsigned char)rank;
        }
        __syncthreads();
        if (t == 0) { S->tc.on = all_thresholds; S->tb.on = 0; S->tb.pad = 0; }
        if (t < DISCO_MAX_SLOTS) { S->tb.fill[t] = 0u; S->tb.of_slot[t] = -1; }
    }
    __syncthreads();
    if (which == 0 && threadIdx.x < DISCO_MAX_PASS) {
        // digits of 8 bits from the top of the range's bits down
        const unsigned lo = smin <= smax ? smin : 0u, hi = smin <= smax ? smax : 0u;
        const int i = threadIdx.x, bits = hi != lo ? 32 - __clz(hi - lo) : 0, left = bits - 8 * i;
        SelGlobal& g = S->g[0];
        g.plan.width[i] = left <= 0 ? 0 : (left < 8 ? left : 8);
        g.plan.shift[i] = left <= 8 ? 0 : left - 8;
        if (i == 0) {
            g.minb = lo; g.maxb = hi;
            g.plan.npass = (bits + 7) / 8; g.plan.pad = 0;
            g.gather_bound = 0ull; g.n_list = 0u; g.gather_error = 0;
        }
    }
    if (which == 1 && threadIdx.x == 0) {
        SelGlobal g;
        {
            // TBT: raw keys; the passes are planned on the device (TlSel)
            g.minb = 0u; g.maxb = 0x7FFFFFFFu;
            g.gather_bound = 0ull; g.n_list = 0u; g.gather_error = 0;
            g.plan.npass = 0; g.plan.pad = 0;
            for (int i = 0; i < DISCO_MAX_PASS; ++i) { g.plan.shift[i] = 0; g.plan.width[i] = 0; }
            TlSel& tl = S->tl;
            tl.ncls = 0; tl.nwalk = 0; tl.walk_mask = 0ull; tl.error = 0; tl.nlist = 0u; tl.nlist_back = 0u; tl.left_fast = 0u; tl.left_buf = 0u;
            TlPlan& start = tl.plan[0];
            start.left = 31; start.shift = 0; start.width = 0; start.G = 0; start.window = 0; start.key_lo = 0u; start.fallback = 0; start.reset = 0;
            for (int i = 0; i < DISCO_TBT_MAX_PASS; ++i) tl.restart[i] = 0;
        }
        S->g[which] = g;
    }
    if (which == 1) {
        for (int i = threadIdx.x; i < DISCO_MAX_CLS; i += blockDim.x) S->tl.cls_mask[i] = 0ull;
        for (int i = threadIdx.x; i < DISCO_CLS_SLOTS; i += blockDim.x) { S->tl.gslot[i] = 0ull; S->tl.gwalk[i] = 0u; }
        if (threadIdx.x == 0) S->tl.goverflow = 0;
    }
    for (int s = threadIdx.x; s < P * nq; s += blockDim.x) {
        int c = s / nq, qi = s % nq;
        i64 M = which ? acc[c].tbt_count : n_req;
        SelSlot sl;
        sl.M = M;
        const i64 k = nearest_rank(qs[qi], M);
        sl.rank = k; sl.k_rem = k; sl.prefix = 0u; sl.done = (M <= 0);
        S->slot[which][s] = sl;
    }
}


// Staging of the policy table (wave 0); all 1024 threads also put the tickets and the per-column totals that
// the workgroups of a pass add into at their identity: the dispatch totals (8 words per column and copy,
// word-major; word 7 = {min bits, max bits}) and, behind them, the timeline totals (all zero).
constexpr int STAGE_THREADS = 1024;
__device__ inline void reset_totals(u64* totals)
{
    constexpr int DISP_WORDS = 8 * DISCO_NCOPY * 64, TL_WORDS = DISCO_NCOPY * 64 * (int)(sizeof(MigPartial) / 8);
    for (int w = threadIdx.x; w < DISP_WORDS + TL_WORDS; w += STAGE_THREADS)
        totals[w] = (w >= 7 * DISCO_NCOPY * 64 && w < DISP_WORDS) ? 0x00000000FFFFFFFFull : 0ull;
}

// With a selection state (si.S), the TTFT selection of the statistics (and, if asked, the TBT selection) is started
// in the same launch by a workgroup of its own (one after the other in one workgroup: 10 us for 8 columns and
// 12.5 us for 64, now 6 with the clearing and 10).
// Workgroup `bid` of `nblk`: 0 the table, 1 and 2 the starts of the two selections, the others clear what the second one counts in.
// totals nullable.
__device__ __forceinline__ void stage_table(const disco_policy* src, int P, disco_policy* dst, unsigned* tickets, u64* totals,
                                            const SelInit& si, int bid, int nblk)
{
    if (bid > 2) {                 // (1 MB and 32 KB per column)
        const int first = (bid - 3) * STAGE_THREADS + (int)threadIdx.x, step = (nblk - 3) * STAGE_THREADS;
        for (int w = first; w < DISCO_MAX_CLS * (DISCO_PP_NMAX + 1); w += step) si.ppcnt[w] = 0u;
        for (int w = first; w < P * DISCO_DELAY_BINS; w += step) si.dhist[w] = 0u;
        if (si.ghist)
            for (int w = first; w < DISCO_GHIST_WORDS / 4; w += step) reinterpret_cast<uint4*>(si.ghist)[w] = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    if (bid > 0) {
        select_init(si, bid - 1, P, src);
        return;
    }
    const int i = threadIdx.x;
    if (i < 64) {
        if (i < P) dst[i] = src[i];
        const bool any_buffer = __ballot(i < P && src[i < P ? i : 0].mig_mode == DISCO_MIG_BUFFER) != 0ull;
        tickets[i] = (i == DISCO_FLAG_BUFFER && any_buffer) ? 1u : 0u;
    }
    if (totals != nullptr) reset_totals(totals);
}

}  // namespace
