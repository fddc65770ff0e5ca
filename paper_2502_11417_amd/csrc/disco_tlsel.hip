// TBT order statistics over token timelines (Sec. 5.1 metrics on the
// timelines of Sec. 4.3): classes of timelines, analytic histogram of
// pure-pacing timelines, digit selection between the histogram passes.
//
// A timeline is histogrammed once per class = set of policy columns that use
// it, not once per column.  For threshold- or wait-ordered tables the sets
// are nested, so there are at most P + 1 of them per source.  Classes whose
// members are all short pure-pacing timelines (constant source gap below the
// pacing interval) need no token walk at all: the gap in front of token t is
// round(t tau) - round((t-1) tau) for every one of them, so counting the
// timelines per class and length gives their histogram.
//
// Launches of a selection: classification, assignment and the gap pools
// (other file); per regular pass k_tbt_pass (plan, analytic bins, pools,
// timelines left to be walked: workgroups by kind) and k_tbt_select (one
// workgroup per slot); per spare pass k_tbt_pass alone.  A launch that finds the selection finished returns at once, which
// still costs about 2 us on the device: hence few launches.
#include <string.h>

#include "disco_final.h"
#include "disco_tl_general_kernel.h"
#include "disco_tl_hist_buf.h"
#include "disco_tl_hist_fast.h"

namespace {

// Distinct column sets of a workgroup's requests: an open-addressing hash table in LDS (CL_SLOTS slots, far more
// than the DISCO_MAX_CLS sets a class-mode selection can hold).  A lane looks its set up with one LDS read in the
// common case (lanes with the same set read the same slot); a new set is claimed with a compare-and-swap.
constexpr int CL_BLOCK = 1024;              // classification: 16 waves share one table
constexpr int CL_SLOTS = DISCO_CLS_SLOTS;

struct ClassTable {
    u64 slot[CL_SLOTS];            // 0 = free
    unsigned walk[CL_SLOTS];       // a member of the set needs a token walk
    u64 dense[DISCO_MAX_CLS];      // the sets, compacted (table_compact)
    unsigned long long dense_walk;
    unsigned wave_cnt[CL_BLOCK / 64];
    int overflow;
};

__device__ __forceinline__ void table_clear(ClassTable& T)
{
    for (int i = threadIdx.x; i < CL_SLOTS; i += CL_BLOCK) { T.slot[i] = 0ull; T.walk[i] = 0u; }
    if (threadIdx.x < DISCO_MAX_CLS) T.dense[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) { T.dense_walk = 0ull; T.overflow = 0; }
}

__device__ __forceinline__ void table_insert(ClassTable& T, u64 m, bool walked)
{
    if (m == 0ull) return;
    unsigned h = (unsigned)((m * 0x9E3779B97F4A7C15ull) >> 56) & (CL_SLOTS - 1);
    volatile u64* vs = T.slot;
    for (int probe = 0; probe < CL_SLOTS; ++probe) {
        u64 cur = vs[h];
        if (cur == 0ull) cur = (u64)atomicCAS((unsigned long long*)&T.slot[h], 0ull, (unsigned long long)m);
        if (cur == 0ull || cur == m) {           // claimed now, or already there
            if (walked && ((volatile unsigned*)T.walk)[h] == 0u) ((volatile unsigned*)T.walk)[h] = 1u;
            return;
        }
        h = (h + 1) & (CL_SLOTS - 1);
    }
    T.overflow = 1;                              // (more than CL_SLOTS distinct sets)
}

// All threads: the occupied slots in slot order -> dense[0 .. count), dense_walk; more than DISCO_MAX_CLS -> overflow.
__device__ __forceinline__ int table_compact(ClassTable& T)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    const u64 v = threadIdx.x < CL_SLOTS ? T.slot[threadIdx.x] : 0ull;
    const u64 occ = __ballot(v != 0ull);
    if (lane == 0) T.wave_cnt[wave] = (unsigned)__popcll(occ);
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < CL_SLOTS / 64; ++w) { const int c = (int)T.wave_cnt[w]; before += w < wave ? c : 0; total += c; }
    if (v != 0ull) {
        const int pos = before + __popcll(occ & ((1ull << lane) - 1ull));
        if (pos < DISCO_MAX_CLS) {
            T.dense[pos] = v;
            if (T.walk[threadIdx.x]) atomicOr(&T.dense_walk, 1ull << pos);
        }
    }
    if (threadIdx.x == 0 && total > DISCO_MAX_CLS) T.overflow = 1;
    __syncthreads();
    return total < DISCO_MAX_CLS ? total : DISCO_MAX_CLS;
}

// Column sets of every request.  Every workgroup collects its distinct sets in an LDS hash table and enters them
// (a few dozen) into a device-wide table of the same kind, from which every workgroup of the assignment numbers them as
// classes (a last workgroup that did so behind a ticket took half of this launch).  The device-wide table was zeroed when the
// selection started (select_init, in the launch that stages the policy table).
// Summaries of buffer hand-offs that were found with other prices (reuse_walk) say neither which timelines are paced nor
// where the others hand off: with any of them the general kernel walks all timelines with the prices of this call.
__global__ __launch_bounds__(CL_BLOCK) void k_tl_classify(TraceView tr, const disco_policy* __restrict__ pol, int P,
                                                     const TlSummary* __restrict__ summary,
                                                     const BufSummary* __restrict__ bufsum, u64 tag, SelState* S)
{
    __shared__ disco_policy sp[DISCO_MAX_COLS];
    __shared__ ClassTable T;
    if ((int)threadIdx.x < P) sp[threadIdx.x] = pol[threadIdx.x];
    table_clear(T);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const i64 nround = (tr.n_req + CL_BLOCK - 1) / CL_BLOCK;
    bool stale = false;
    for (i64 rnd = blockIdx.x; rnd < nround; rnd += gridDim.x) {
        const i64 i = rnd * CL_BLOCK + threadIdx.x;
        if (i >= tr.n_req) continue;
        const int l = tr.l[i], n = tr.n[i];
        const float s = tr.s[i];
        const float k = tr.k ? tr.k[i] : tr.k_s;
        u64 m[TL_KINDS];
        request_sets(sp, P, l, s, __fmaf_rn((float)l, k, tr.c), i, m);
        const TlSummary sm = summary[i];
        table_insert(T, m[TL_DEV], !timeline_is_analytic(TL_DEV, n, sm));
        table_insert(T, m[TL_SRV], !timeline_is_analytic(TL_SRV, n, sm));
        table_insert(T, m[TL_SRV_LAG], !timeline_is_analytic(TL_SRV_LAG, n, sm));
        if ((m[TL_SRV_BUF] | m[TL_DEV_BUF]) != 0ull) {
            const BufSummary bs = bufsum[i];
            // (a hand-off leaves the target a token: another one is no summary of this trace and must not index its tokens)
            stale = stale || bs.tag != tag || summary_m(bs.m_s) > n - 2 || summary_m(bs.m_d) > n - 2;
            table_insert(T, m[TL_SRV_BUF], !buf_timeline_is_analytic(TL_SRV_BUF, n, bs));
            table_insert(T, m[TL_DEV_BUF], !buf_timeline_is_analytic(TL_DEV_BUF, n, bs));
        }
    }
    {
        // this workgroup's distinct sets into the device-wide table (same probing; entries are never changed once
        // claimed, so a stale read can only cost an extra compare-and-swap)
        const int mine_n = table_compact(T);
        TlSel& g = S->tl;
        if ((int)threadIdx.x < mine_n) {
            const u64 m = T.dense[threadIdx.x];
            const bool walked = (T.dense_walk >> threadIdx.x) & 1ull;
            unsigned h = (unsigned)((m * 0x9E3779B97F4A7C15ull) >> 56) & (CL_SLOTS - 1);
            volatile u64* vs = g.gslot;
            bool placed = false;
            for (int probe = 0; probe < CL_SLOTS && !placed; ++probe) {
                u64 cur = vs[h];
                if (cur == 0ull) cur = (u64)atomicCAS((unsigned long long*)&g.gslot[h], 0ull, (unsigned long long)m);
                if (cur == 0ull || cur == m) {
                    if (walked && ((volatile unsigned*)g.gwalk)[h] == 0u) atomicOr(&g.gwalk[h], 1u);
                    placed = true;
                } else {
                    h = (h + 1) & (CL_SLOTS - 1);
                }
            }
            if (!placed) atomicOr(&g.goverflow, 1);
        }
        if (threadIdx.x == 0 && T.overflow) atomicOr(&g.goverflow, 1);
        if (__ballot(stale) != 0ull && lane == 0) atomicOr(&g.goverflow, 2);
    }
}

// Of one class: counts by length -> number of timelines longer than t, in place (all threads; `part`: 1024 words of LDS).
__device__ void longer_than(unsigned* row, unsigned* part)
{
    constexpr int PER = (DISCO_PP_NMAX + 1 + 1023) / 1024;
    const int t0 = threadIdx.x * PER;
    unsigned v[PER];
    unsigned sum = 0;
    for (int q = 0; q < PER; ++q) { v[q] = (t0 + q <= DISCO_PP_NMAX) ? row[t0 + q] : 0u; sum += v[q]; }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {            // inclusive suffix sums of the per-thread totals
        const unsigned o = (threadIdx.x + d < 1024) ? part[threadIdx.x + d] : 0u;
        __syncthreads();
        part[threadIdx.x] += o;
        __syncthreads();
    }
    unsigned above = (threadIdx.x + 1 < 1024) ? part[threadIdx.x + 1] : 0u;       // lengths beyond this thread's slice
    for (int q = PER - 1; q >= 0; --q) {
        if (t0 + q <= DISCO_PP_NMAX) row[t0 + q] = above;                         // timelines with n > t0 + q
        above += v[q];
    }
    __threadfence_block();                          // (the workgroup reads the row it has written)
    __syncthreads();
}

// Step 1 of a TBT pass (all threads of a workgroup, class c; beside the
// workgroups that walk tokens, hence atomic adds): add the analytic bins of
// the class's pure-pacing timelines to its device-wide rows.  ppcnt[c][t] timelines of class c have a token t (the first
// pass makes that of the counts by length), and the gap in front of it is the same number for all of them.
__device__ void analytic_class(const TlPlan& pl, int ncls, int pass, unsigned* ghist, unsigned* ppcnt, float tau, int c, unsigned* lds)
{
    const int width = pl.width;
    unsigned* row = ppcnt + (size_t)c * (DISCO_PP_NMAX + 1);
    if (pass == 0) longer_than(row, lds);
    if (row[0] == 0u) return;                             // no pure-pacing timeline in this class (uniform)
    const int Gused = pl.G < DISCO_MAX_GRP ? pl.G : DISCO_MAX_GRP;
    const unsigned dmask = (1u << width) - 1u;
    const int words = Gused << width;
    const int shift = pl.shift, up = pl.shift + width;
    const unsigned key_cap = pl.window ? (1u << pl.window) : 0xFFFFFFFFu;
    __syncthreads();
    for (int i = threadIdx.x; i < words; i += blockDim.x) lds[i] = 0u;
    __syncthreads();
    for (int t = 1 + (int)threadIdx.x; t < DISCO_PP_NMAX; t += blockDim.x) {
        const unsigned cnt = row[t];
        if (!cnt) continue;
        const unsigned key = tbt_key(f2u((float)t * tau - (float)(t - 1) * tau), pl.key_lo, key_cap);
        const unsigned hi = key >> up;                     // clamped keys match no prefix
        int g = -1;
        for (int k = 0; k < Gused; ++k) g = (hi == pl.grp_prefix[k] && g < 0) ? k : g;
        if (g >= 0) atomicAdd(&lds[((unsigned)g << width) | ((key >> shift) & dmask)], cnt);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < words; i += blockDim.x) {
        const unsigned v = lds[i];
        if (v) atomicAdd(&ghist[((size_t)((i >> width) * ncls + c) << width) | (i & dmask)], v);
    }
}

// Step 2 (all threads of a workgroup, (column, quantile) slot s): add up the
// class histograms of the classes that contain the slot's column (or take the
// slot's own histogram in the fallback), walk to the digit that holds the
// remaining rank, extend the prefix.
//   binsum: LDS scratch of binsum_cap words: the bin counts of a slot with more than two bins per thread are summed over
//   its classes there with coalesced reads of the class rows (a thread then scans consecutive bins from LDS); wider digits
//   and the fallback read the rows directly.
__device__ void select_slot(SelState* S, const TlPlan& pl, int pass, int nq, const unsigned* ghist, int s, u64* wsum /* LDS, 64 */,
                            int* s_digit, u64* s_rem, u64* binsum, int binsum_cap)
{
    const TlSel& tl = S->tl;
    const int width = pl.width, ncls = tl.ncls, fallback = pl.fallback;
    SelSlot sl = S->slot[1][s];
    const int g = pl.slot_grp[s];
    if (sl.done || g < 0) return;                         // uniform
    if (pl.reset) { sl.prefix = 0u; sl.k_rem = sl.rank; }
    const int col = s / nq;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nbins = 1 << width;
    const int per = (nbins + (int)blockDim.x - 1) / (int)blockDim.x;      // consecutive bins per thread
    const int b0 = threadIdx.x * per;
    // up to two bins per thread are summed over the classes in registers, wider digits in LDS
    const bool direct = !fallback && per <= 2;
    const bool staged = !fallback && !direct && nbins <= binsum_cap;
    u64 own[2] = {0ull, 0ull};
    if (direct || staged) {
        // the classes that contain the column (the first wave lists them in wsum[0 .. nk), nk in *s_digit), then
        // every bin is the sum over their rows: all loads independent and coalesced
        __syncthreads();
        if (wave == 0) {
            const bool in = lane < ncls && ((tl.cls_mask[lane] >> col) & 1ull);
            const u64 inb = __ballot(in);
            if (in) wsum[__popcll(inb & ((1ull << lane) - 1ull))] = (u64)lane;
            if (lane == 0) *s_digit = __popcll(inb);
        }
        __syncthreads();
        const int nk = *s_digit;
        if (direct) {
            if (b0 < nbins) {
                const unsigned* base = ghist + ((size_t)(g * ncls) << width) + b0;
                if (per == 2) {
#pragma unroll 8
                    for (int j = 0; j < nk; ++j) {
                        const uint2 v = *reinterpret_cast<const uint2*>(base + ((size_t)wsum[j] << width));
                        own[0] += v.x; own[1] += v.y;
                    }
                } else {
#pragma unroll 8
                    for (int j = 0; j < nk; ++j) own[0] += base[(size_t)wsum[j] << width];
                }
            }
        } else {
            for (int b = threadIdx.x; b < nbins; b += (int)blockDim.x) {
                u64 c = 0;
#pragma unroll 4
                for (int j = 0; j < nk; ++j) c += ghist[((size_t)(g * ncls + (int)wsum[j]) << width) | b];
                binsum[b] = c;
            }
        }
        __syncthreads();
    }
    auto bin_count = [&](int b) -> u64 {
        if (direct) return b == b0 ? own[0] : own[1];
        if (staged) return binsum[b];
        if (fallback) return ghist[((size_t)s << width) | b];
        u64 c = 0;
        for (int k = 0; k < ncls; ++k)
            if ((tl.cls_mask[k] >> col) & 1ull) c += ghist[((size_t)(g * ncls + k) << width) | b];
        return c;
    };
    u64 mine = 0;
    for (int b = b0; b < b0 + per && b < nbins; ++b) mine += bin_count(b);
    u64 incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        unsigned lo = (unsigned)__shfl_up((int)(unsigned)incl, d, 64);
        unsigned hi = (unsigned)__shfl_up((int)(unsigned)(incl >> 32), d, 64);
        if (lane >= d) incl += ((u64)hi << 32) | lo;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = incl;
    if (threadIdx.x == 0) *s_digit = -1;
    __syncthreads();
    u64 before = 0;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    incl += before;
    const u64 k = (u64)sl.k_rem;
    if (incl >= k && incl - mine < k) {                   // at most one thread: the rank falls into its bins
        u64 rem = k - (incl - mine);
        int dsel = b0;
        for (int b = b0; b < b0 + per && b < nbins; ++b) {
            const u64 c = bin_count(b);
            dsel = b;
            if (rem <= c) break;
            rem -= c;
        }
        *s_digit = dsel;
        *s_rem = rem;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int dsel = *s_digit;
        u64 rem = *s_rem;
        // window mode: a rank beyond the counted keys, or in the bottom bin (which also holds the keys below the
        // window), is not decided here -> start over on raw keys.  Raw keys: the rank is always found.
        if (pl.window && (dsel < 0 || (dsel == 0 && pl.left == pl.window))) S->tl.restart[pass] = 1;
        if (dsel < 0) { dsel = nbins - 1; rem = 1; }
        sl.k_rem = (i64)rem;
        sl.prefix = (sl.prefix << width) | (unsigned)dsel;
        S->slot[1][s] = sl;
    }
}

// The same for a digit of at most SEL_NARROW_BITS bits in class mode, by one wave (lane = class): many slots side by side
// in one workgroup.
constexpr int SEL_NARROW_BITS = 4;

__device__ void select_slot_narrow(SelState* S, const TlPlan& pl, int pass, int nq, const unsigned* ghist, int s)
{
    const TlSel& tl = S->tl;
    const int width = pl.width, ncls = tl.ncls, lane = threadIdx.x & 63;
    SelSlot sl = S->slot[1][s];
    const int g = pl.slot_grp[s];
    if (sl.done || g < 0) return;                         // uniform
    if (pl.reset) { sl.prefix = 0u; sl.k_rem = sl.rank; }
    const int col = s / nq, nbins = 1 << width;
    static_assert(DISCO_MAX_CLS <= 64, "a lane per class");
    const bool in = lane < ncls && ((tl.cls_mask[lane] >> col) & 1ull);
    u64 rem = (u64)sl.k_rem;
    int dsel = -1;
    for (int b = 0; b < nbins && dsel < 0; ++b) {
        const u64 c = wave_sum_u64(in ? (u64)ghist[((size_t)(g * ncls + lane) << width) | (unsigned)b] : 0ull);
        if (rem <= c) dsel = b; else rem -= c;
    }
    if (lane == 0) {
        // as in select_slot: what the window does not decide starts over on raw keys
        if (pl.window && (dsel < 0 || (dsel == 0 && pl.left == pl.window))) S->tl.restart[pass] = 1;
        if (dsel < 0) { dsel = nbins - 1; rem = 1; }
        sl.k_rem = (i64)rem;
        sl.prefix = (sl.prefix << width) | (unsigned)dsel;
        S->slot[1][s] = sl;
    }
}

// Words of the device-wide bins a pass uses.
__device__ __forceinline__ int bins_used(const TlPlan& pl, int ncls, int ns)
{
    const int Gused = pl.G < DISCO_MAX_GRP ? pl.G : DISCO_MAX_GRP;
    return pl.width <= 0 ? 0 : (pl.fallback ? ns : Gused * ncls) << pl.width;
}
// The bins of the next pass back to zero (thread t of nt): what the pass before this one used, all of them before the second.
__device__ __forceinline__ void clear_next_bins(const SelState* S, int pass, int ns, unsigned* bins, int t, int nt)
{
    const int words = pass > 0 ? bins_used(S->tl.plan[pass], S->tl.ncls, ns) : DISCO_GHIST_WORDS;
    for (int i = t; i < (words + 3) / 4; i += nt) reinterpret_cast<uint4*>(bins)[i] = make_uint4(0u, 0u, 0u, 0u);
}

__device__ __forceinline__ BufHistArgs buf_hist_args(const TimelineArgs& a)
{
    BufHistArgs h;
    h.h.tau = a.tau; h.h.kt = a.kt; h.h.P = a.P; h.h.nq = a.nq; h.h.pass = a.pass;
    h.h.S = a.S; h.h.ghist = a.ghist; h.h.desc = a.desc; h.h.list = a.list; h.h.runs = a.runs;
    h.bufsum = (const BufSummary*)a.bufsum;
    h.buffer_flag = a.buffer_flag;
    return h;
}

static_assert(TH_BLOCK == 1024 && TBH_BLOCK == 1024 && TL_BLOCK == 1024, "the kinds of workgroup share launches");

// Workgroup = slot: the digit of the slot; SEL_CLEAR workgroups behind them clear the bins of the next pass.
constexpr int SEL_CLEAR = DISCO_GHIST_WORDS / 4 / 1024;
__global__ __launch_bounds__(1024) void k_tbt_select(SelState* S, int pass, int P, int nq, const unsigned* __restrict__ ghist,
                                                     unsigned* __restrict__ next)
{
    __shared__ u64 wsum[DISCO_MAX_CLS];
    __shared__ int s_digit;
    __shared__ u64 s_rem;
    const TlPlan& pl = S->tl.plan[pass + 1];
    if (pl.width <= 0) return;
    const int ns = P * nq;
    if ((int)blockIdx.x < ns) select_slot(S, pl, pass, nq, ghist, blockIdx.x, wsum, &s_digit, &s_rem, nullptr, 0);
    else clear_next_bins(S, pass, ns, next, ((int)blockIdx.x - ns) * 1024 + (int)threadIdx.x, SEL_CLEAR * 1024);
}

// A pass: its plan, the analytic bins (a class per workgroup), the pools and what is left of the walk list, or the per-slot
// histograms of a table whose column sets do not fit the class scheme (then every workgroup walks).
//   PASS_REGULAR  its digits are taken by k_tbt_select behind it
//   PASS_DENSE    the same from DENSE_REQ requests on: two workgroups per CU, for the timelines that no pool holds (those of a
//                 source slower than the reader; a wave's walk waits for its LDS atomics and loads).  In 64 registers it
//                 spills, which costs the other passes 0.6 us each, more than it gains on fewer requests.  Statistics of
//                 threshold columns with such sources, PASS_DENSE against PASS_REGULAR: 10^6 requests x 8 columns 3452 / 3551 us
//                 (lag), 5598 / 5762 (buffer), x 1 column 3259 / 3452; 10^5 requests 713 / 713, 998 / 995, 551 / 562
//   PASS_SPARE    a pass after those that normally decide every slot (the window was missed, or the digits are narrow): the
//                 workgroup that finishes last takes every slot's digit and clears the next pass's bins; one launch
//                 matters more here than speed, as normally all workgroups return at once
//   PASS_LAST     the last spare pass, which also makes the columns' records
enum { PASS_REGULAR, PASS_DENSE, PASS_SPARE, PASS_LAST };
constexpr i64 DENSE_REQ = 1 << 18;
constexpr unsigned TP_ANALYTIC = DISCO_MAX_CLS;

template <int KIND>
__global__ __launch_bounds__(1024, KIND == PASS_DENSE ? 8 : 4) void k_tbt_pass(TraceView tr, i64 n_tok, int align,
                                                                               const disco_policy* __restrict__ pol,
                                                                               TimelineArgs a, FinalArgs fin)
{
    __shared__ __align__(16) unsigned smem[DISCO_TL_HIST_WORDS];
    __shared__ TimelineLds lds;
    __shared__ TlPlan pl;
    SelState* S = a.S;
    const TlSel& tl = S->tl;
    const unsigned bid = blockIdx.x;
    tbt_open_pass(S, a.pass, a.P, a.nq, pl);
    if (pl.width <= 0) {                                // selection finished (the same answer in every workgroup)
        if (KIND == PASS_LAST && (int)bid < a.P) stats_final((int)bid, fin, *reinterpret_cast<FinalLds*>(smem), &pl);
        return;
    }
    if (pl.fallback) {
        timeline_body<true>(smem, lds, tr, n_tok, align, pol, a, &pl, bid, gridDim.x);
    } else {
        // with timelines left to walk the workgroups of the classes take a share of them too (192 of 256 workgroups walking, 1.3
        // times the time); the last one, as the long requests are dealt first
        const bool walks = pl.walks != 0;
        if (bid < TP_ANALYTIC && (int)bid < tl.ncls) {
            analytic_class(pl, tl.ncls, a.pass, a.ghist, a.ppcnt, a.tau, (int)bid, smem);
            __syncthreads();                            // the bins are used again
        }
        if (walks || bid >= TP_ANALYTIC) {
            const unsigned others = gridDim.x - TP_ANALYTIC, at = bid >= TP_ANALYTIC ? bid - TP_ANALYTIC : bid + others;
            const unsigned of = walks ? gridDim.x : others;
            HistArgs h;
            h.tau = a.tau; h.kt = a.kt; h.P = a.P; h.nq = a.nq; h.pass = a.pass; h.S = a.S; h.ghist = a.ghist; h.desc = a.desc; h.list = a.list; h.runs = a.runs;
            tl_hist_fast_body(smem, tr, n_tok, align, h, pl, at, of);
            __syncthreads();
            tl_hist_buf_body(smem, tr, n_tok, align, buf_hist_args(a), pl, at, of);
        }
    }
    if (KIND == PASS_REGULAR || KIND == PASS_DENSE) return;
    if (!take_last_ticket(a.ticket)) return;
    __shared__ u64 wsum[DISCO_MAX_CLS];
    __shared__ int s_digit;
    __shared__ u64 s_rem;
    __syncthreads();
    if (!pl.fallback && pl.width <= SEL_NARROW_BITS) {
        for (int s = threadIdx.x >> 6; s < a.P * a.nq; s += (int)blockDim.x >> 6) select_slot_narrow(S, pl, a.pass, a.nq, a.ghist, s);
    } else {
        for (int s = 0; s < a.P * a.nq; ++s) {
            select_slot(S, pl, a.pass, a.nq, a.ghist, s, wsum, &s_digit, &s_rem, reinterpret_cast<u64*>(smem), DISCO_TL_HIST_WORDS / 2);
            __syncthreads();
        }
    }
    if (threadIdx.x == 0) *a.ticket = 0u;
    if (KIND == PASS_SPARE) {
        clear_next_bins(S, a.pass, a.P * a.nq, a.gclear, (int)threadIdx.x, (int)blockDim.x);
    } else {
        __threadfence_block();                          // (the slots' digits are read back)
        __syncthreads();
        for (int c = 0; c < a.P; ++c) {
            stats_final(c, fin, *reinterpret_cast<FinalLds*>(smem), &pl);
            __syncthreads();
        }
    }
}

}  // namespace

void disco_launch_tl_classify(const TraceView& v, const disco_policy* pol, int P, const void* summary, const void* bufsum,
                              const BufCostArgs& bc, SelState* S, hipStream_t stream)
{
    i64 b = (v.n_req + CL_BLOCK - 1) / CL_BLOCK;
    if (b < 1) b = 1;
    if (b > 256) b = 256;                          // (more workgroups cost more in the merge than they save in the scan)
    b /= disco_grid_divisor();
    if (b < 1) b = 1;
    hipLaunchKernelGGL(k_tl_classify, dim3((unsigned)b), dim3(CL_BLOCK), 0, stream, v, pol, P, (const TlSummary*)summary,
                       (const BufSummary*)bufsum, price_tag(bc), S);
}

// One pass of the TBT selection and the step to the next one.
void disco_launch_tbt_pass(const TraceView& v, i64 n_tok, const disco_policy* pol, const TimelineArgs& a, const FinalArgs& fin,
                           hipStream_t stream)
{
    const int align = (int)(((uintptr_t)v.arr >> 2) & 3);
    // all workgroups resident at once: more of them make an empty launch dearer
    const i64 per_wave = (v.n_req + 15) / 16;                    // workgroups if every wave took one request
    const bool dense = a.pass < DISCO_TBT_REGULAR_PASS && v.n_req >= DENSE_REQ;
    const i64 most = (dense ? 512 : 256) - (i64)TP_ANALYTIC;
    i64 walkers = per_wave < 1 ? 1 : (per_wave > most ? most : per_wave);
    walkers /= disco_grid_divisor();
    const dim3 grid(TP_ANALYTIC + (unsigned)(walkers < 1 ? 1 : walkers));
    if (a.pass < DISCO_TBT_REGULAR_PASS) {
        if (dense) hipLaunchKernelGGL(k_tbt_pass<PASS_DENSE>, grid, dim3(1024), 0, stream, v, n_tok, align, pol, a, fin);
        else hipLaunchKernelGGL(k_tbt_pass<PASS_REGULAR>, grid, dim3(1024), 0, stream, v, n_tok, align, pol, a, fin);
        hipLaunchKernelGGL(k_tbt_select, dim3((unsigned)(a.P * a.nq + SEL_CLEAR)), dim3(1024), 0, stream, a.S, a.pass, a.P, a.nq, a.ghist,
                           a.gclear);
    } else if (a.pass + 1 < DISCO_TBT_MAX_PASS) {
        hipLaunchKernelGGL(k_tbt_pass<PASS_SPARE>, grid, dim3(1024), 0, stream, v, n_tok, align, pol, a, fin);
    } else {
        hipLaunchKernelGGL(k_tbt_pass<PASS_LAST>, grid, dim3(1024), 0, stream, v, n_tok, align, pol, a, fin);
    }
}
