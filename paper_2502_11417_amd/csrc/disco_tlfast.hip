// Token timelines (Sec. 4.3): the class-mode TBT histogram passes of
// disco_reduce_stats and what prepares them once per selection.
//
//   k_tl_assign  lane = request: timelines that the token walk's summaries
//                prove analytic (running maximum never left 0, so
//                delta_t = round(t tau)) are counted per class and length;
//                the others get their histogram row into the request's
//                descriptor and the request into the walk list
//   k_pp_reduce  per-workgroup count slices -> counts per class and length
//   k_tl_runs    the listed timelines' gaps, counted per value once
//                (disco_tl_runs.h)
//
// A pass over these and what is left of the walk list is k_tbt_pass (the
// selection's own file; workgroup body and walker in disco_tl_hist_fast.h): a
// wave walks one request at a time in chunks of 256 tokens, four consecutive
// tokens per lane (one 16-byte load per lane and chunk, the next chunk's
// load issued before the current one is used).
//
// The delivery recurrence delta_t = max(r_t, delta_{t-1} + tau) is evaluated
// in the shifted domain u_t = r_t - t tau, where it is a running maximum M_t
// and delta_t = fma(t, tau, M_t).  `max` is exact and associative, so any
// evaluation order gives the sequential definition bit for bit.  The
// histogram walk needs M_t per token: a 4-element scan in registers and a DPP
// scan across the wave; the gaps delta_t - delta_{t-1} go to the LDS
// histogram of the timeline's class.
//
// Lag trigger (token t is overdue by more than kappa tau): evaluated exactly,
// one IEEE fp32 operation at a time in the order of the definition (slot =
// delta_{t-1} + tau, lag = r_t - slot), in every chunk that passes a cheap necessary
// condition (see walk_hist); the other chunks provably cannot trigger.
//
// A timeline is computed once per request and source, never per policy
// column: the recurrence does not depend on the pair's TTFT, so every column
// only picks the timeline of its dispatch winner.
#include <string.h>

#include "disco_tl_runs.h"

namespace {


// Analytic timelines per class and length, counted per workgroup in LDS (two 16-bit counts per word, a workgroup
// sees at most 65535 requests) for the first PP_LDS_CLS classes and stored as one slice per workgroup; classes
// beyond that (tables of many columns) are counted in device memory directly.
constexpr int PP_LDS_CLS = 16;
constexpr int PP_WORDS = DISCO_PP_NMAX / 2 + 1;              // words per class: lengths 0 .. DISCO_PP_NMAX
constexpr int AS_BLOCK = 1024;
constexpr int DH_LDS_BINS = 64;              // delayed-token counts below this are counted in LDS: [column][count], 16 KB

// The classes from the device-wide table of column sets, in ascending order (so that their numbers do not depend on
// timing), and the rows of those with tokens to walk in the workgroups' LDS histograms, in class order.
struct ClassList {
    u64 mask[DISCO_MAX_CLS];                   // 0: none
    u64 found[DISCO_MAX_CLS];
    unsigned char walk[DISCO_MAX_CLS], found_walk[DISCO_MAX_CLS];
    signed char slot[DISCO_MAX_CLS];           // LDS row of a walked class, -1 otherwise
    unsigned cnt[DISCO_CLS_SLOTS / 64];
    int total;
};

// All threads.
__device__ __forceinline__ void list_classes(const TlSel& tl, ClassList& L)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    u64 v = 0ull;
    unsigned w = 0u;
    if (t < DISCO_CLS_SLOTS) { v = tl.gslot[t]; w = tl.gwalk[t]; }
    const u64 occ = __ballot(v != 0ull);
    if (t < DISCO_CLS_SLOTS && lane == 0) L.cnt[wave] = (unsigned)__popcll(occ);
    if (t < DISCO_MAX_CLS) { L.mask[t] = 0ull; L.walk[t] = 0; }
    __syncthreads();
    int before = 0, total = 0;
    for (int k = 0; k < DISCO_CLS_SLOTS / 64; ++k) { const int c = (int)L.cnt[k]; before += k < wave ? c : 0; total += c; }
    if (v != 0ull) {
        const int at = before + __popcll(occ & ((1ull << lane) - 1ull));
        if (at < DISCO_MAX_CLS) { L.found[at] = v; L.found_walk[at] = w != 0u; }
    }
    if (t == 0) L.total = total;
    __syncthreads();
    const int n = total < DISCO_MAX_CLS ? total : DISCO_MAX_CLS;
    if (t < n) {
        const u64 mine = L.found[t];
        int rank = 0;
#pragma unroll 8
        for (int k = 0; k < n; ++k) rank += L.found[k] < mine ? 1 : 0;
        L.mask[rank] = mine; L.walk[rank] = L.found_walk[t];
    }
    __syncthreads();
    if (wave == 0) {
        const u64 wm = __ballot(L.walk[lane] != 0);
        L.slot[lane] = L.walk[lane] ? (signed char)__popcll(wm & ((1ull << lane) - 1ull)) : (signed char)-1;
    }
    __syncthreads();
}

// The counter `idx` (-1: none) of every lane plus one; the one of the first lane that has any is added to once for all
// lanes that share it (requests of one length).
__device__ __forceinline__ void count_shared(unsigned* __restrict__ counters, int idx, int lane)
{
    const u64 any = __ballot(idx >= 0);
    if (!any) return;
    const int leader = __ffsll((long long)any) - 1;
    const int i0 = bcast_i(idx, leader);
    const u64 same = __ballot(idx == i0);
    if (lane == leader) atomicAdd(&counters[i0], (unsigned)__popcll(same));
    if (idx >= 0 && idx != i0) atomicAdd(&counters[idx], 1u);
}

// use_lds = 0: counts in device memory (small traces: a slice per workgroup and their sum cost more than the few atomics).
__global__ __launch_bounds__(AS_BLOCK) void k_tl_assign(TraceView tr, const disco_policy* __restrict__ pol, int P, float tau,
                                                        const TlSummary* __restrict__ summary,
                                                        const BufSummary* __restrict__ bufsum, SelState* S,
                                                        u64* __restrict__ desc_out, unsigned* __restrict__ list,
                                                        unsigned* __restrict__ slices, unsigned* __restrict__ ppcnt,
                                                        unsigned* __restrict__ dhist, int use_lds)
{
    __shared__ __align__(16) unsigned cnt[PP_LDS_CLS * PP_WORDS];          // 128 KB
    __shared__ unsigned dh[DISCO_MAX_COLS * DH_LDS_BINS];
    __shared__ unsigned s_nw[2], s_base[2];                  // [0] long requests (front of the list), [1] the others (back)
    __shared__ ClassList cl;
    __shared__ disco_policy spol[DISCO_MAX_COLS];
    if ((int)threadIdx.x < P) spol[threadIdx.x] = pol[threadIdx.x];
    list_classes(S->tl, cl);
    const int over = S->tl.goverflow;                        // bit 0: too many sets, bit 1: summaries found at other prices
    const bool fallback = cl.total > DISCO_MAX_CLS || over != 0;
    const int ncls = fallback ? DISCO_MAX_CLS : (cl.total > 0 ? cl.total : 1);
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        // for the passes; gaps sit just above the pacing interval (down to a few thousand ulps below it after rounding): a
        // window of keys is tried first (not at other prices: the passes of 128 slots would not suffice for a second start), 21
        // bits or as many as two digits have if the LDS rows of the walked classes leave room for digits of less than 11 bits.
        // (A third walk for the last bit of 12 wait columns: 49 us of 570 with 10^5 requests, 64 of 400 with 30 000; a rank
        // beyond the shorter window costs a pass more than one beyond the longer.)
        const int lane = threadIdx.x;
        TlSel& g = S->tl;
        const u64 wm = __ballot(cl.walk[lane] != 0);
        g.cls_mask[lane] = cl.mask[lane];
        g.cls_slot[lane] = cl.slot[lane];
        if (cl.walk[lane]) g.slot_cls[cl.slot[lane]] = (unsigned char)lane;
        if (lane == 0) {
            const unsigned tb = f2u(tau);
            const int nwalk = __popcll(wm);
            const int wl = fit_width(nwalk > 0 ? nwalk : 1, DISCO_TL_HIST_WORDS), wg = fit_width(ncls, DISCO_GHIST_WORDS);
            const int two = 2 * (wl < wg ? wl : wg), window = tb < 8192u || (over & 2) != 0 ? 0 : (two < 21 ? two : 21);
            g.ncls = ncls; g.walk_mask = wm; g.nwalk = nwalk;
            TlPlan& start = g.plan[0];
            start.window = window; start.left = window ? window : 31; start.key_lo = window ? tb - 8192u : 0u;
            start.fallback = fallback ? 1 : 0;
        }
    }
    if (fallback) return;                                    // per-slot histograms: the general kernel walks everything
    const int nlds = use_lds ? (ncls < PP_LDS_CLS ? ncls : PP_LDS_CLS) : 0;
    for (int i = threadIdx.x; i < nlds * PP_WORDS; i += AS_BLOCK) cnt[i] = 0u;
    for (int i = threadIdx.x; i < P * DH_LDS_BINS; i += AS_BLOCK) dh[i] = 0u;
    if (threadIdx.x < 2) s_nw[threadIdx.x] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    // a contiguous share of the requests per workgroup (at most 65535, see the launch)
    const i64 per = (tr.n_req + gridDim.x - 1) / gridDim.x;
    const i64 lo = (i64)blockIdx.x * per;
    const i64 hi = lo + per < tr.n_req ? lo + per : tr.n_req;
    u64 wmask = 0ull, lmask = 0ull;                          // bit r: this thread's request of round r has tokens to walk / is long
    int round = 0;
    for (i64 i = lo + threadIdx.x; i < hi; i += AS_BLOCK, ++round) {
        const int l = tr.l[i], n = tr.n[i];
        const float s = tr.s[i];
        const float k = tr.k ? tr.k[i] : tr.k_s;
        const TlSummary sm = summary[i];
        u64 m[TL_KINDS];
        request_sets(spol, P, l, s, __fmaf_rn((float)l, k, tr.c), i, m);
        u64 desc = DESC_NONE5;
        BufSummary bs{0.0f, -1, 0, 0, 0.0f, -1, 0ull};
        if ((m[TL_SRV_BUF] | m[TL_DEV_BUF]) != 0ull) {
            bs = bufsum[i];
            // migrated requests by number of delayed tokens, per column (those without one are implied by the
            // migration count)
#pragma unroll
            for (int kind = TL_SRV_BUF; kind <= TL_DEV_BUF; ++kind) {
                const int me = kind == TL_SRV_BUF ? bs.m_s : bs.m_d;
                const int dl = kind == TL_SRV_BUF ? bs.delay_s : bs.delay_d;
                if (m[kind] == 0ull || summary_m(me) < 0 || dl <= 0) continue;
                const int bin = dl < DISCO_DELAY_BINS - 1 ? dl : DISCO_DELAY_BINS - 1;
                for (u64 left = m[kind]; left != 0ull; left &= left - 1ull) {
                    const int c = __ffsll((long long)left) - 1;
                    if (bin < DH_LDS_BINS) atomicAdd(&dh[c * DH_LDS_BINS + bin], 1u);
                    else atomicAdd(&dhist[(size_t)c * DISCO_DELAY_BINS + bin], 1u);
                }
            }
        }
#pragma unroll
        for (int kind = 0; kind < TL_KINDS; ++kind) {
            int direct = -1;                                 // counter in device memory
            if (m[kind] != 0ull) {
                const int c = cls_find(cl.mask, ncls, m[kind]);
                const int sl = c >= 0 ? cl.slot[c] : -1;
                if (c < 0) {
                    S->tl.error = 1;                         // a set the classification did not see: never expected
                } else if (kind < TL_SRV_BUF ? timeline_is_analytic(kind, n, sm) : buf_timeline_is_analytic(kind, n, bs)) {
                    if (c < nlds) atomicAdd(&cnt[c * PP_WORDS + (n >> 1)], 1u << (16 * (n & 1)));
                    else direct = c * (DISCO_PP_NMAX + 1) + n;
                } else if (sl < 0) {
                    S->tl.error = 1;
                } else {
                    desc = (desc & ~(0xFFull << (8 * kind))) | ((u64)(unsigned)sl << (8 * kind));
                }
            }
            if (nlds < ncls) count_shared(ppcnt, direct, lane);
        }
        desc_out[i] = desc;
        const bool walk = desc != DESC_NONE5, lng = n >= WALK_LONG_TOKENS;
        if (walk) wmask |= 1ull << round;
        if (walk && lng) lmask |= 1ull << round;
        const u64 wb = __ballot(walk);
        if (wb) {
            const u64 lb = __ballot(walk && lng);
            if (lane == __ffsll((long long)wb) - 1) {
                if (lb) atomicAdd(&s_nw[0], (unsigned)__popcll(lb));
                if (wb & ~lb) atomicAdd(&s_nw[1], (unsigned)__popcll(wb & ~lb));
            }
        }
    }
    __syncthreads();
    // the requests with tokens to walk go to a device-wide list (any order: the histograms are sums), a range of it
    // per workgroup
    const unsigned nw0 = s_nw[0], nw1 = s_nw[1];
    __syncthreads();
    if (threadIdx.x == 0) {
        s_base[0] = nw0 ? atomicAdd(&S->tl.nlist, nw0) : 0u;
        s_base[1] = nw1 ? atomicAdd(&S->tl.nlist_back, nw1) : 0u;
        s_nw[0] = 0u; s_nw[1] = 0u;
    }
    __syncthreads();
    if (nw0 | nw1) {
        round = 0;
        for (i64 i = lo + threadIdx.x; i < hi; i += AS_BLOCK, ++round) {
            const bool w = (wmask >> round) & 1ull, lng = (lmask >> round) & 1ull;
            const u64 wb = __ballot(w);
            if (!wb) continue;
            const u64 lb = __ballot(w && lng), sb = wb & ~lb;
            const int leader = __ffsll((long long)wb) - 1;
            unsigned at0 = 0u, at1 = 0u;
            if (lane == leader) {
                if (lb) at0 = atomicAdd(&s_nw[0], (unsigned)__popcll(lb));
                if (sb) at1 = atomicAdd(&s_nw[1], (unsigned)__popcll(sb));
            }
            at0 = (unsigned)bcast_i((int)at0, leader);
            at1 = (unsigned)bcast_i((int)at1, leader);
            const u64 below = (1ull << lane) - 1ull;
            if (w && lng) list[s_base[0] + at0 + (unsigned)__popcll(lb & below)] = (unsigned)i;
            if (w && !lng) list[(size_t)tr.n_req - 1 - (s_base[1] + at1 + (unsigned)__popcll(sb & below))] = (unsigned)i;
        }
    }
    for (int i = threadIdx.x; i < P * DH_LDS_BINS; i += AS_BLOCK)
        if (dh[i]) atomicAdd(&dhist[(size_t)(i / DH_LDS_BINS) * DISCO_DELAY_BINS + i % DH_LDS_BINS], dh[i]);
    // (whole vectors: the words behind the last class belong to rows that are not read)
    static_assert(PP_LDS_CLS * PP_WORDS % 4 == 0, "slices of whole vectors");
    uint4* mine = reinterpret_cast<uint4*>(slices) + (size_t)blockIdx.x * (PP_LDS_CLS * PP_WORDS / 4);
    for (int i = threadIdx.x; 4 * i < nlds * PP_WORDS; i += AS_BLOCK) mine[i] = reinterpret_cast<const uint4*>(cnt)[i];
}

// ppcnt[c][n] += sum over the workgroup slices.  Workgroup = (class, 256 words of two lengths each); four groups
// of threads share the slices and meet in LDS.  The launch also clears the device-wide bins of the histogram passes (1 MB;
// the TTFT selection has used them before).
__global__ __launch_bounds__(1024) void k_pp_reduce(const SelState* S, int nslices, const unsigned* __restrict__ slices,
                                                    unsigned* __restrict__ ppcnt, unsigned* __restrict__ ghist, int use_lds)
{
    __shared__ unsigned part[2][1024];
    static_assert(DISCO_GHIST_WORDS % 4 == 0, "bins of whole vectors");
    for (unsigned i = (blockIdx.y * gridDim.x + blockIdx.x) * 1024u + threadIdx.x; i < DISCO_GHIST_WORDS / 4; i += gridDim.x * gridDim.y * 1024u)
        reinterpret_cast<uint4*>(ghist)[i] = make_uint4(0u, 0u, 0u, 0u);
    const TlSel* tl = &S->tl;
    const int c = blockIdx.x;
    if (tl->plan[0].fallback || !use_lds || c >= tl->ncls || c >= PP_LDS_CLS) return;
    const int w = blockIdx.y * 256 + (threadIdx.x & 255), grp = threadIdx.x >> 8;
    unsigned even = 0u, odd = 0u;
    if (w < PP_WORDS) {
#pragma unroll 8
        for (int b = grp; b < nslices; b += 4) {
            const unsigned v = slices[((size_t)b * PP_LDS_CLS + c) * PP_WORDS + w];
            even += v & 0xFFFFu; odd += v >> 16;
        }
    }
    part[0][threadIdx.x] = even; part[1][threadIdx.x] = odd;
    __syncthreads();
    if (grp == 0 && w < PP_WORDS) {
        for (int g = 1; g < 4; ++g) { even += part[0][threadIdx.x + 256 * g]; odd += part[1][threadIdx.x + 256 * g]; }
        unsigned* row = ppcnt + (size_t)c * (DISCO_PP_NMAX + 1);
        if (even) row[2 * w] += even;
        if (odd && 2 * w + 1 <= DISCO_PP_NMAX) row[2 * w + 1] += odd;
    }
}

// The gaps of the listed timelines, per value, into the workgroup's pool; the descriptors then name those alone that are left to
// the passes.  List entries are dealt as in the passes.  Bound by vector issue (some 800 instructions per request): 56 us for the
// 17 M tokens of 35 000 requests with lag hand-offs (10^6 requests x 8 columns), 43 with buffer hand-offs, after which a pass
// takes 13 us; walked token by token a pass took 59 and 69 us.  10^5 requests x 12 wait columns: 26 us, and 18 instead of 45 a pass.
constexpr int TR_BLOCK = 512, TR_WAVES = TR_BLOCK / 64;
constexpr int TR_MAX_BLOCKS = 768;           // what the chip holds at once (six waves per SIMD)
// An attempt at a timeline of too many moves, or at a full pool, is made in vain; one that succeeds spares every pass a walk.  A
// wave stops trying when its pool is full, and after RUNS_VAIN attempts in vain one behind the other (where fewer than one in eight
// succeeds): sources slower than the reader, 10^6 requests x 1 column 3.05 ms of order statistics, 3.37 without the rule; gaps
// of many stalls, which fill the pools, 0.87 and 1.20.
constexpr int RUNS_VAIN = 12;

__global__ __launch_bounds__(TR_BLOCK, 6) void k_tl_runs(TraceView tr, i64 n_tok, int align, float tau, float kt, SelState* S,
                                                      u64* __restrict__ desc_rw, const unsigned* __restrict__ list,
                                                      const TlSummary* __restrict__ summary, const BufSummary* __restrict__ bufsum, RunPool runs)
{
    __shared__ __align__(16) RunLds rl[TR_WAVES];
    __shared__ unsigned used;
    TlSel& tl = S->tl;
    uint2* pool = runs.pool + (size_t)blockIdx.x * runs.cap;
    if (threadIdx.x == 0) used = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int vain = 0;                                            // the wave's last attempts that were in vain
    bool some_fast = false, some_buf = false;
    const i64 nfront = (i64)tl.nlist, nlist = tl.plan[0].fallback ? 0 : nfront + (i64)tl.nlist_back;
    const i64 nwaves = (i64)gridDim.x * (TR_WAVES);
    i64 rb = (nlist + nwaves - 1) / nwaves;
    rb = rb < 1 ? 1 : (rb > 64 ? 64 : rb);
    const i64 nround = (nlist + rb * nwaves - 1) / (rb * nwaves);
    for (i64 rnd = 0; rnd < nround; ++rnd) {
        const i64 j = rnd * rb * nwaves + (i64)blockIdx.x * (TR_WAVES) + wave + (i64)lane * nwaves;
        const bool mine = lane < rb && j < nlist;
        const i64 i = mine ? (i64)walk_list_entry(list, tr.n_req, nfront, j) : 0;
        const u64 desc = mine ? desc_rw[i] & DESC_NONE5 : DESC_NONE5;
        int l_v = 0, n_v = 1, m_v = -1;
        float k_v = tr.k_s, gd_v = tr.g_s, gap_v = 0.0f;
        i64 off_v = 0;
        Handoff from_srv{-1, 0.0f, 0.0f}, from_dev{-1, 0.0f, 0.0f};
        const bool attempt = mine && vain < RUNS_VAIN;
        if (attempt) {
            l_v = tr.l[i]; n_v = tr.n[i];
            if (tr.k) k_v = tr.k[i];
            if (tr.g) gd_v = tr.g[i];
            if (tr.off) off_v = tr.off[i];
            if (tr.tbt) gap_v = tr.tbt[i];
            if (((desc >> (8 * TL_SRV_LAG)) & 0xFFull) != 0xFFull) m_v = summary_m(summary[i].m_enc);
            const bool sb = ((desc >> (8 * TL_SRV_BUF)) & 0xFFull) != 0xFFull, db = ((desc >> (8 * TL_DEV_BUF)) & 0xFFull) != 0xFFull;
            if (sb || db) {
                const BufSummary bs = bufsum[i];
                const float s_ttft = tr.s[i];
                from_srv = handoff_at(false, sb ? summary_m(bs.m_s) : -1, tr.arr, off_v, l_v, s_ttft, k_v, tr.c, gap_v, gd_v);
                from_dev = handoff_at(true, db ? summary_m(bs.m_d) : -1, tr.arr, off_v, l_v, s_ttft, k_v, tr.c, gap_v, gd_v);
            }
        }
        // a device slower than the reader moves the maximum at every token: no attempt at a timeline with many of its tokens
        // (kinds: those to be tried, a bit each; from bit 8 on those that went to the pool)
        unsigned kinds = 0u;
        if (attempt && paced_ok(tau, n_v)) {
            const bool slow = gd_v > 1.01f * tau;
#pragma unroll
            for (int kind = 0; kind < TL_KINDS; ++kind) {
                const bool many = kind == TL_DEV ? n_v > 64 : (kind == TL_SRV_LAG ? m_v >= 0 && n_v - m_v > 64 : (kind == TL_DEV_BUF ? from_dev.m > 64 : false));
                if (((desc >> (8 * kind)) & 0xFFull) != 0xFFull && !(slow && many)) kinds |= 1u << kind;
            }
        }
        u64 walkers = __ballot(kinds != 0u);
        // requests that read the token array: all but those of the device's own timeline alone
        static_assert(TL_DEV == 0, "the lowest bit");
        const u64 memw = tr.arr != nullptr ? __ballot(kinds > 1u) : 0ull;
        float ahead[4] = {0.f, 0.f, 0.f, 0.f};
        auto load_ahead = [&](u64 todo) {
            if (!todo) return;
            const int r = __ffsll((long long)todo) - 1;
            if ((memw >> r) & 1ull) load_first(tr.arr, (i64)bcast_u64((u64)off_v, r), bcast_i(n_v, r), n_tok, align, lane, ahead);
        };
        load_ahead(walkers);
        while (walkers) {
            const int rq = __ffsll((long long)walkers) - 1;
            walkers &= walkers - 1;
            const u64 dsc = bcast_u64(desc, rq);
            const unsigned todo = (unsigned)bcast_i((int)kinds, rq);
            const int n = bcast_i(n_v, rq), l = bcast_i(l_v, rq);
            const float gd = bcast_f(gd_v, rq), gap = bcast_f(gap_v, rq), k = bcast_f(k_v, rq);
            const i64 off = tr.arr ? (i64)bcast_u64((u64)off_v, rq) : 0;
            const float chunk[4] = {ahead[0], ahead[1], ahead[2], ahead[3]};
            load_ahead(walkers);                             // the next request's first chunk, while this one is walked
#pragma unroll 1
            for (int kind = 0; kind < TL_KINDS; ++kind) {
                if (((todo >> kind) & 1u) == 0u) continue;
                const unsigned row = (unsigned)(dsc >> (8 * kind)) & 0xFFu;
                const Handoff& v = kind == TL_DEV_BUF ? from_dev : from_srv;
                const Handoff ho{0, bcast_f(v.base, rq), bcast_f(v.a_m, rq)};
                // first token of the target
                const int last = kind >= TL_SRV_BUF ? bcast_i(v.m, rq) : (kind == TL_SRV_LAG ? bcast_i(m_v, rq) - 1 : -2);
                const int m = last >= 0 ? last + 1 : 0x7FFFFFFF;
                int ns, n1;
                const bool done = walk_runs(rl[wave], ns, n1, kind, n, tr.arr, off, n_tok, align, chunk, gap, gd, l, k, tr.c, m, ho, tau, kt, lane) &&
                                  emit_runs(rl[wave], ns, n1, row, tau, pool, runs.cap, &used, lane);
                if (done) {
                    kinds |= lane == rq ? 0x100u << kind : 0u;
                    vain = 0;
                } else {
                    vain = *(volatile unsigned*)&used >= runs.cap ? RUNS_VAIN : vain + 1;
                    if (vain >= RUNS_VAIN) walkers = 0ull;
                }
            }
        }
        u64 left = desc;
#pragma unroll
        for (int kind = 0; kind < TL_KINDS; ++kind)
            if ((kinds >> (8 + kind)) & 1u) left |= 0xFFull << (8 * kind);
        if (left != desc) desc_rw[i] = left;
        constexpr u64 FAST = 0xFFFFFFull;                    // the streaming kinds' bytes
        some_fast = some_fast || __ballot((left & FAST) != FAST) != 0ull;
        some_buf = some_buf || __ballot((left | FAST) != DESC_NONE5) != 0ull;
    }
    // (stored, not counted: an addition per wave and round to one address cost 145 us with 10^6 requests on the list)
    if (lane == 0 && some_fast) tl.left_fast = 1u;
    if (lane == 0 && some_buf) tl.left_buf = 1u;
    __syncthreads();
    if (threadIdx.x == 0) pool[0] = make_uint2(used < runs.cap ? used : runs.cap - 1u, 0u);
}

}  // namespace

// Once per selection, after the classification: descriptors of all requests, analytic timelines counted per class
// and length.  `slices`: scratch for the workgroup slices (slices_bytes).
void disco_launch_tl_assign(const TraceView& v, const disco_policy* pol, int P, float tau, const void* summary, SelState* S,
                            const void* bufsum, u64* desc, unsigned* list, unsigned* slices, size_t slices_bytes,
                            unsigned* ppcnt, unsigned* ghist, unsigned* dhist, hipStream_t stream)
{
    if (v.n_req <= 0) return;
    i64 b = (v.n_req + 49151) / 49152;             // at most 65535 requests per workgroup: 16-bit counts in LDS
    // one workgroup per CU (128 KB of LDS each, at most 64 rounds per thread); fewer where every request has a thread of
    // its own, as each workgroup writes up to 128 KB of counts (10^4 requests x 16 columns: 22 us with 250 of
    // them, 13 with 10, and 8 -> 3 us for their sum)
    const i64 threads = (v.n_req + AS_BLOCK - 1) / AS_BLOCK, cus = threads < 250 ? threads : 250;
    if (b < cus) b = cus;
    const i64 fit = (i64)(slices_bytes / ((size_t)PP_LDS_CLS * PP_WORDS * sizeof(unsigned)));
    int use_lds = 1;
    // tens of millions of requests (or the testing aid that shrinks the grids): counts in device memory
    if (b > fit || disco_grid_divisor() > 1) { b = (v.n_req + 65535) / 65536; use_lds = 0; }
    const bool small = disco_small(v.n_req);
    if (small) use_lds = 0;
    hipLaunchKernelGGL(k_tl_assign, dim3((unsigned)b), dim3(AS_BLOCK), 0, stream, v, pol, P, tau, (const TlSummary*)summary,
                       (const BufSummary*)bufsum, S, desc, list, slices, ppcnt, dhist, use_lds);
    if (small) return;                             // (their bins are cleared in the launch that stages the policy table)
    hipLaunchKernelGGL(k_pp_reduce, dim3(PP_LDS_CLS, (PP_WORDS + 255) / 256), dim3(1024), 0, stream, (const SelState*)S, (int)b, (const unsigned*)slices,
                       ppcnt, ghist, use_lds);
}

void disco_launch_tl_runs(const TraceView& v, i64 n_tok, TimelineArgs& a, void* scratch, size_t scratch_bytes, hipStream_t stream)
{
    i64 b = (v.n_req + TR_WAVES - 1) / TR_WAVES;                   // at most one request per wave
    if (b < 1) b = 1;
    if (b > TR_MAX_BLOCKS) b = TR_MAX_BLOCKS;
    b /= disco_grid_divisor();
    if (b < 1) b = 1;
    a.runs.pool = (uint2*)scratch;
    a.runs.cap = (unsigned)(scratch_bytes / sizeof(uint2) / (size_t)b);
    a.runs.n = (int)b;
    const int align = (int)(((uintptr_t)v.arr >> 2) & 3);
    hipLaunchKernelGGL(k_tl_runs, dim3((unsigned)b), dim3(TR_BLOCK), 0, stream, v, n_tok, align, a.tau, a.kt, a.S, a.desc, a.list,
                       (const TlSummary*)a.summary, (const BufSummary*)a.bufsum, a.runs);
}
