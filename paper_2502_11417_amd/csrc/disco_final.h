// The result record of a column, from its accumulators and the selections.
#pragma once
#include <math.h>

#include "disco_launch.h"
#include "disco_state.h"

namespace {

constexpr int FINAL_THREADS = 256;

// The record of a column from its accumulators and the selections' results (workgroup = column).
//
// Order statistics of the delayed tokens per migrated request: the counts by number of delayed tokens come from the
// first histogram pass of the timelines with a buffer hand-off; migrations of the lag trigger have none and count as
// zeros.  Nearest rank, like the other order statistics; NaN for a column without migrations.
//
// Bound by latency: the counts, the accumulators and the slots are fetched side by side by different waves, the record is
// put together in LDS (9 us with one thread for all but the counts, now 4 - 6).
struct FinalLds {
    u64 wtot[4];
    i64 drank[DISCO_MAX_Q];
    float dq[DISCO_MAX_Q];
    disco_stats st;
};

// TTFT order statistics of a column, where the workgroup that makes its record has them itself.
struct TtftFound { i64 rank[DISCO_MAX_Q]; float q[DISCO_MAX_Q]; };

// All threads of a workgroup of at least FINAL_THREADS.  last: plan of the last TBT pass (nullable without timelines);
// found: nullable, in LDS.
__device__ __forceinline__ void stats_final(int c, const FinalArgs& f, FinalLds& lds, const TlPlan* last, const TtftFound* found = nullptr)
{
    constexpr int PER = DISCO_DELAY_BINS / 256;
    u64* wtot = lds.wtot;
    i64* drank = lds.drank;
    float* dq = lds.dq;
    disco_stats& st = lds.st;
    const int nq = f.nq, with_tl = f.with_tl;
    const i64 n_req = f.n_req;
    const disco_accum* acc = f.acc;
    const SelState* S = f.S;
    const int t = threadIdx.x < FINAL_THREADS ? (int)threadIdx.x : FINAL_THREADS, lane = t & 63, wave = t >> 6;      // (the other threads only meet the barriers)
    const i64 migrated = with_tl ? acc[c].n_migrated : 0;
    const bool delays = with_tl && nq > 0 && migrated > 0;
    unsigned v[PER];
    u64 mine = 0;
    if (delays && t < FINAL_THREADS) {
        const unsigned* row = f.dhist + (size_t)c * DISCO_DELAY_BINS;
#pragma unroll
        for (int k = 0; k < PER; ++k) { v[k] = row[t * PER + k]; mine += v[k]; }
    }
    if (t < (int)(sizeof(st) / 8)) reinterpret_cast<u64*>(&st)[t] = 0ull;
    if (t < DISCO_MAX_Q) dq[t] = NAN;
    __syncthreads();
    if (t == 0) {
        const disco_accum a = acc[c];
        st.n_req = n_req;
        st.s_pre = a.s_pre + (with_tl ? a.m_s_repre : 0);
        st.d_pre = a.d_pre + (with_tl ? a.m_d_repre : 0);
        st.s_dec = with_tl ? a.m_s_dec : a.s_dec;
        st.d_dec = with_tl ? a.m_d_dec : a.d_dec;
        st.n_dev_started = a.n_dev_started;
        st.n_dev_win = a.n_dev_win;
        st.n_migrated = migrated;
        st.tbt_count = with_tl ? a.tbt_count : 0;
        st.mean_ttft = a.ttft_sum / (double)n_req;                       // 0/0 = NaN for an empty batch
        st.mean_tbt = with_tl ? a.tlast_sum / (double)a.tbt_count : NAN;  // telescoped sum of gaps
        st.mean_delay_num = (with_tl && a.n_migrated > 0) ? (double)a.delay_sum / (double)a.n_migrated : NAN;
        st.server_cost = server_cost_of(f.cost, st.s_pre, st.s_dec);
        st.device_energy = device_energy_of(f.cost, st.d_pre, st.d_dec);
        st.device_cost = f.cost.lambda * st.device_energy;
        st.total_cost = st.server_cost + st.device_cost;
    }
    if (t >= 64 && t < 64 + DISCO_MAX_Q) {
        const int qi = t - 64;
        float tq = NAN, bq = NAN;
        if (qi < nq) {
            const disco_quantile q = qi == 0 ? f.q[0] : (qi == 1 ? f.q[1] : (qi == 2 ? f.q[2] : f.q[3]));
            if (found != nullptr) {
                st.ttft_rank[qi] = found->rank[qi];
                tq = found->q[qi];
            } else {
                const SelSlot s0 = S->slot[0][c * nq + qi];
                st.ttft_rank[qi] = s0.rank;
                if (s0.M > 0 && !S->g[0].gather_error) tq = u2f(S->g[0].minb + s0.prefix);
            }
            if (with_tl) {
                const SelSlot s1 = S->slot[1][c * nq + qi];
                st.tbt_rank[qi] = s1.rank;
                // (all digits decided: after the last pass, or by the one before it)
                const bool whole = last->left == last->width && !(last->window != 0 && S->tl.restart[DISCO_TBT_MAX_PASS - 1] != 0);
                if (s1.M > 0 && !S->tl.error && whole) bq = u2f(s1.prefix + last->key_lo);
            }
            i64 k = ((i64)q.num * migrated + q.den - 1) / q.den;
            if (k < 1) k = 1;
            drank[qi] = k < migrated ? k : migrated;
        }
        st.ttft_q[qi] = tq; st.tbt_q[qi] = bq;
    }
    // inclusive prefix sums of the per-thread counts
    u64 incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned lo = (unsigned)__shfl_up((int)(unsigned)incl, d, 64), hi = (unsigned)__shfl_up((int)(unsigned)(incl >> 32), d, 64);
        if (lane >= d) incl += ((u64)hi << 32) | lo;
    }
    if (lane == 63 && t < FINAL_THREADS) wtot[wave] = incl;
    __syncthreads();
    if (delays && t < FINAL_THREADS) {
        u64 counted = 0;
        for (int w = 0; w < 4; ++w) { counted += wtot[w]; incl += w < wave ? wtot[w] : 0ull; }
        const u64 zeros = (u64)migrated > counted ? (u64)migrated - counted : 0;      // hand-offs without a count: no delayed token
        if (t == 0) v[0] += (unsigned)zeros;
        const u64 below = t > 0 ? incl - mine + zeros : 0;               // migrated requests with fewer delayed tokens than t * PER
        for (int qi = 0; qi < nq; ++qi) {
            const u64 k = (u64)drank[qi];
            u64 cum = below;
#pragma unroll
            for (int b = 0; b < PER; ++b) {
                if (cum < k && cum + v[b] >= k) dq[qi] = (float)(t * PER + b);
                cum += v[b];
            }
        }
    }
    __syncthreads();
    if (t < DISCO_MAX_Q) st.delay_q[t] = dq[t];
    __syncthreads();
    if (t < (int)(sizeof(st) / 8)) reinterpret_cast<u64*>(&f.out[c])[t] = reinterpret_cast<const u64*>(&st)[t];
}

}  // namespace
