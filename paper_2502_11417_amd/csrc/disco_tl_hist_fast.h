// One class-mode TBT histogram pass over the timelines of the streaming
// kinds (device source, server source, server source with the lag trigger;
// Sec. 4.3): the walker and the workgroup body, shared by the kernel of the
// regular passes and the kernel of the spare passes.
#pragma once
#include "disco_tl_walk.h"

namespace {

constexpr int TH_BLOCK = 1024;               // histogram workgroups: 16 waves share 64 KB of bins
// Workgroups of a pass over the pools alone: each one clears its bins and adds them to the device-wide ones.  Little depends on
// their number: order statistics with 48 / 128 / as many as walk, at most 256, of 10^4 requests x 8 columns 101 / 99 / 99 us, 10^5 x 8
// 158 / 152 / 154, 10^5 x 12 waits 239 / 227 / 226, 4 10^5 x 8 204 / 196 / 197, 10^6 x 8 263 / 248 / 249, 10^6 x 12 waits 720 / 686 / 686.
constexpr unsigned HIST_POOL_BLOCKS = 128;

// ------------------------------------------------------------------ plan ---

// Bin counts of a slot that k_tbt_select sums up in registers (two per thread, the rows of eight classes in flight).  Tables
// without walked timelines (constant gaps) have room for digits of 13 and 14 bits, but their 21-bit window takes two
// passes either way, and an unstaged slot of 8192 bins reads the rows of its classes bin by bin: 10^4 requests x 16 columns
// 120 us with 13 bits, 28 us with 11.
constexpr int SEL_DIRECT_BITS = 11;

// The plan of a pass (first wave of a workgroup; `out` in LDS): prefix groups of the live slots, digit width that fits, or
// the per-slot fallback.  Every workgroup of the launch that opens a pass does this, some 2 us beside its other start-up; the
// last workgroup of the pass before did it behind a ticket, with the bins still to clear: 10 us of an 18 us launch.
__device__ __forceinline__ void tbt_plan(const SelState* S, int pass, int P, int nq, TlPlan& out)
{
    static_assert(DISCO_MAX_SLOTS == 128, "two slots per lane");
    const TlSel& tl = S->tl;
    const TlPlan& prev = tl.plan[pass];
    const int lane = threadIdx.x & 63, ns = P * nq;
    const int ncls = tl.ncls, nwalk = tl.nwalk, walks = (tl.left_fast != 0u ? 1 : 0) | (tl.left_buf != 0u ? 2 : 0);
    unsigned p0 = 0u, p1 = 0u;
    bool live0 = false, live1 = false;
    if (lane < ns) { p0 = S->slot[1][lane].prefix; live0 = !S->slot[1][lane].done; }
    if (64 + lane < ns) { p1 = S->slot[1][64 + lane].prefix; live1 = !S->slot[1][64 + lane].done; }
    int left = prev.left, window = prev.window, reset = 0;
    unsigned key_lo = prev.key_lo;
    bool done = false;
    if (pass > 0) {
        done = prev.width <= 0;
        if (!done && window != 0 && tl.restart[pass - 1] != 0) {       // the window missed a rank: all slots start over on raw keys
            window = 0; key_lo = 0u; left = 31; reset = 1;
            p0 = p1 = 0u;
        } else if (!done) {
            left -= prev.width;
            done = left == 0;
        }
    }
    // the distinct prefixes in slot order, one after the other; a lane holds slots `lane` and 64 + `lane`
    u64 todo0 = __ballot(live0), todo1 = __ballot(live1);
    int G = 0, g0 = -1, g1 = -1;
    unsigned grp[DISCO_MAX_GRP] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < DISCO_MAX_GRP; ++k) {
        if ((todo0 | todo1) == 0ull) break;
        const unsigned px = todo0 ? (unsigned)bcast_i((int)p0, __ffsll((long long)todo0) - 1) : (unsigned)bcast_i((int)p1, __ffsll((long long)todo1) - 1);
        const bool h0 = live0 && p0 == px, h1 = live1 && p1 == px;
        if (h0) g0 = k;
        if (h1) g1 = k;
        todo0 &= ~__ballot(h0); todo1 &= ~__ballot(h1);
        grp[k] = px;
        G = k + 1;
    }
    int fallback = prev.fallback;
    if ((todo0 | todo1) != 0ull) {             // too many distinct prefixes: the per-slot fallback does not use groups
        fallback = 1;
        G += 1;
        if (live0 && g0 < 0) g0 = 0;
        if (live1 && g1 < 0) g1 = 0;
    }
    if (ncls > DISCO_MAX_CLS || ncls < 1) fallback = 1;
    int w;
    if (fallback) {
        w = fit_width(ns, DISCO_TL_HIST_WORDS);
    } else {
        const int gn = G > 0 ? G : 1;
        w = fit_width((long)gn * (nwalk > 0 ? nwalk : 1), DISCO_TL_HIST_WORDS);
        const int wg = fit_width((long)gn * ncls, DISCO_GHIST_WORDS);
        if (wg < w) w = wg;
        // a digit of more bins than the select step sums up in registers only where it saves a pass.  Not on raw keys with
        // timelines to walk: there may be more than four prefixes in the end, and then every bit less here can cost another
        // walk of everything (30 000 requests x 5 columns 1.15 ms of order statistics with 12 + 10 + 9 bits, 1.61 with
        // 11 + 10 + 9 + 1)
        if (w > SEL_DIRECT_BITS && (window != 0 || nwalk == 0) && (left + w - 1) / w == (left + SEL_DIRECT_BITS - 1) / SEL_DIRECT_BITS)
            w = SEL_DIRECT_BITS;
    }
    if (w < 1) w = 1;
    if (w > left) w = left;
    if (G == 0 || done) w = 0;                 // nothing left to select
    if (lane == 0) {
        out.left = left; out.shift = left - w; out.width = w; out.G = G; out.window = window; out.key_lo = key_lo;
        out.fallback = fallback; out.reset = (short)reset; out.walks = (short)walks;
#pragma unroll
        for (int k = 0; k < DISCO_MAX_GRP; ++k) out.grp_prefix[k] = grp[k];
    }
    out.slot_grp[lane] = (signed char)g0;
    out.slot_grp[64 + lane] = (signed char)g1;
}

// All threads of a workgroup of the launch that opens the pass; the first workgroup leaves the plan to the others.
__device__ __forceinline__ void tbt_open_pass(SelState* S, int pass, int P, int nq, TlPlan& plan)
{
    if (threadIdx.x < 64) tbt_plan(S, pass, P, nq, plan);
    __syncthreads();
    static_assert(sizeof(TlPlan) % 4 == 0, "copied in words");
    if (blockIdx.x == 0 && threadIdx.x < sizeof(TlPlan) / 4)
        reinterpret_cast<unsigned*>(&S->tl.plan[pass + 1])[threadIdx.x] = reinterpret_cast<const unsigned*>(&plan)[threadIdx.x];
}

struct WalkOut { int m; float M; };          // hand-off index (-1 none), running maximum over all tokens

// Histogram walk of one request and source: the delivery of every token and
// the gap in front of it -> sink(key[4]) once per chunk (tokens without a gap
// carry KEY_SKIP).
//   mem    arrivals from the CSR token array (else t * gap)
//   lag    evaluate the lag trigger (server source of a column with hand-off)
//   first  the lane's elements of the first chunk, if `have_first` (loaded ahead by the caller with load_first)
//
// Necessary condition for the trigger.  With C <= M_{t-1} (C = a running
// maximum taken earlier: u_0 in the first chunk, the carried maximum later)
// and monotone rounding,
//   lag_t = fl(r_t - fl(fl((t-1) tau + M_{t-1}) + tau)) <= fl(r_t - fl(fl((t-1) tau + C) + tau)),
// which differs from u_t - C = fl(r_t - t tau) - C by at most four roundings
// of magnitudes below 2 t tau + 2 |C| + kappa tau.  lag_fast_ok bounds t and
// `cheap` bounds |C| so that this error stays below kappa tau / 4; hence
// lag_t > kappa tau implies u_t > C + kappa tau / 2, and a chunk where no
// token satisfies the latter cannot trigger.
template <class Sink>
__device__ __forceinline__ WalkOut walk_hist(bool mem, int n, const float* __restrict__ arr, i64 off, i64 n_tok, int align,
                                             const float first[4], bool have_first, float gap, bool lag, float g_dev, int l,
                                             float k, float c, float tau, float kt, int lane, Sink&& sink)
{
    const float ninf = -INFINITY;
    const float ntau = -tau;
    const int mis = mem ? (int)((off + align) & 3) : 0;      // the window starts at the 16-byte boundary below the request
    const int lane4 = 4 * lane - mis;                        // token index of this lane's first element in chunk 0
    const i64 gbase = off + lane4;
    const int total = n + mis;
    const bool safe = mem && off - mis >= 0 && off + n + 3 <= n_tok;
    const bool fast_ok = lag_fast_ok(n, tau, kt);
    int m = -1;
    float base = 0.0f;
    float carryM = ninf;           // running maximum over the chunks so far
    float carryD = 0.0f;           // delivery of the last token of the previous chunk
    float nxt[4] = {first[0], first[1], first[2], first[3]};
    if (mem && !have_first && lane4 < n) load4s(arr, gbase, n_tok, safe, nxt);
#pragma unroll 1
    for (int e0 = 0; e0 < total; e0 += 256) {
        const int tk0 = lane4 + e0;
        const float tf0 = (float)tk0;
        const float tf[4] = {tf0, tf0 + 1.0f, tf0 + 2.0f, tf0 + 3.0f};
        float r[4], u[4];
        if (m >= 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) r[q] = __fmaf_rn((float)(tk0 + q - m + 1), g_dev, base);
        } else if (mem) {
#pragma unroll
            for (int q = 0; q < 4; ++q) r[q] = nxt[q];
            if (e0 + 256 < total && tk0 + 256 < n) load4s(arr, gbase + e0 + 256, n_tok, safe, nxt);   // next chunk in flight
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) r[q] = tf[q] * gap;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = __fmaf_rn(tf[q], ntau, r[q]);
        const bool full = e0 > 0 && e0 + 256 <= total;      // every element of the chunk is a token of the request
        if (!full) {
#pragma unroll
            for (int q = 0; q < 4; ++q) u[q] = ((unsigned)(tk0 + q) < (unsigned)n) ? u[q] : ninf;
        }
        float i0 = u[0], i1 = fmaxf(i0, u[1]), i2 = fmaxf(i1, u[2]), i3 = fmaxf(i2, u[3]);
        bool exact = false;
        if (lag && m < 0) {
            float C = carryM;
            if (e0 == 0) {                                  // u_0 = r_0: element `mis` of lane 0
                const float r0 = mis == 0 ? r[0] : (mis == 1 ? r[1] : (mis == 2 ? r[2] : r[3]));
                C = bcast_f(r0, 0);
            }
            const bool cheap = fast_ok && fabsf(C) <= 262144.0f * kt;
            exact = !cheap || __ballot(i3 > C + 0.5f * kt) != 0ull;
        }
        // running maximum before this lane's tokens: the carried one in a chunk that does not move it (most chunks of a
        // server that is faster than the reader: a pass over 17 M tokens 64 -> 59 us, 73 -> 67 us)
        float E = carryM;
        if (__ballot(i3 > carryM) != 0ull) E = fmaxf(wave_prev(wave_incl_max_dpp(i3, lane), ninf), carryM);
        if (exact) {
            const float ex[4] = {E, fmaxf(E, i0), fmaxf(E, i1), fmaxf(E, i2)};
            bool trig[4];
            float slot[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                slot[q] = __fmaf_rn(tf[q] - 1.0f, tau, ex[q]) + tau;        // delta_{t-1} + tau
                const float lg = r[q] - slot[q];
                trig[q] = (unsigned)(tk0 + q - 1) < (unsigned)(n - 1) && lg > kt;      // tokens 1 .. n-1
            }
            const u64 any = __ballot(trig[0] || trig[1] || trig[2] || trig[3]);
            if (any) {
                const int ml = __ffsll((long long)any) - 1;
                const int qf = trig[0] ? 0 : (trig[1] ? 1 : (trig[2] ? 2 : 3));
                const float sl = trig[0] ? slot[0] : (trig[1] ? slot[1] : (trig[2] ? slot[2] : slot[3]));
                m = bcast_i(tk0, ml) + bcast_i(qf, ml);
                // hand-off: decided once the token is kappa*tau overdue; the device re-prefills the
                // prompt plus the m tokens already produced, then generates at its own pace
                const float t_dec = bcast_f(sl, ml) + kt;
                const float t_mig = __fmaf_rn((float)(l + m), k, c);
                base = t_dec + t_mig;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (tk0 + q >= m) {
                        r[q] = __fmaf_rn((float)(tk0 + q - m + 1), g_dev, base);
                        u[q] = ((unsigned)(tk0 + q) < (unsigned)n) ? __fmaf_rn(tf[q], ntau, r[q]) : ninf;
                    }
                i0 = u[0]; i1 = fmaxf(i0, u[1]); i2 = fmaxf(i1, u[2]); i3 = fmaxf(i2, u[3]);
                E = fmaxf(wave_prev(wave_incl_max_dpp(i3, lane), ninf), carryM);
            }
        }
        const float M0 = fmaxf(E, i0), M1 = fmaxf(E, i1), M2 = fmaxf(E, i2), M3 = fmaxf(E, i3);
        const float d0 = __fmaf_rn(tf[0], tau, M0), d1 = __fmaf_rn(tf[1], tau, M1);
        const float d2 = __fmaf_rn(tf[2], tau, M2), d3 = __fmaf_rn(tf[3], tau, M3);
        const float p0 = wave_prev(d3, carryD);
        unsigned key[4] = {f2u(d0 - p0), f2u(d1 - d0), f2u(d2 - d1), f2u(d3 - d2)};
        if (!full) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                key[q] = ((unsigned)(tk0 + q - 1) < (unsigned)(n - 1)) ? key[q] : KEY_SKIP;     // tokens 1 .. n-1 have a gap
        }
        sink(key);
        carryM = bcast_f(M3, 63);
        carryD = bcast_f(d3, 63);
    }
    return WalkOut{m, carryM};
}

// The lane's elements of the first chunk of a request's token window (see walk_hist).
__device__ __forceinline__ void load_first(const float* __restrict__ arr, i64 off, int n, i64 n_tok, int align, int lane,
                                           float out[4])
{
    const int mis = (int)((off + align) & 3);
    if (4 * lane - mis < n) load4(arr, off - mis + 4 * lane, n_tok, out);
}

// ------------------------------------------------------------- histogram ---

// What every histogram pass needs to know of a request, worked out once per selection (k_tl_assign): the LDS
// row of each of its timelines (device source, server source, server source with the lag trigger, the two buffer
// hand-off kinds; one byte each in the order of the TL_ kinds, 0xFF = nothing to walk: no such timeline, or one
// that is histogrammed analytically).  The kernel below walks the first three kinds.
constexpr u64 DESC_NONE5 = 0xFFFFFFFFFFull;
constexpr unsigned DESC_NONE = 0xFFFFFFu;

// One histogram pass of the class-mode TBT selection, workgroup `bid` of `nblk`: the gaps of the pools, then the timelines
// that have tokens to walk (few: those whose gaps fill no pool, disco_tl_runs.h), by the descriptors; the walk list names their
// requests.  `smem`: DISCO_TL_HIST_WORDS words of LDS.
__device__ __forceinline__ void tl_hist_fast_body(unsigned* smem, const TraceView& tr, i64 n_tok, int align, const HistArgs& a,
                                                  const TlPlan& pl, unsigned bid, unsigned nblk)
{
    const TlSel* tl = &a.S->tl;
    const int width = __builtin_amdgcn_readfirstlane(pl.width);
    // (a pass over the pools alone takes fewer workgroups)
    const bool walks = (__builtin_amdgcn_readfirstlane(pl.walks) & 1) != 0;
    if (!walks && nblk > HIST_POOL_BLOCKS) nblk = HIST_POOL_BLOCKS;
    if (bid >= nblk) return;
    if (width <= 0 || pl.fallback) return;        // selection finished, or per-slot histograms (other kernel)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ncls = tl->ncls, nwalk = tl->nwalk;
    const HistCtx h = hist_ctx(smem, pl, nwalk);
    const int words = (h.G * nwalk) << width;
    for (int i = threadIdx.x; i < words; i += TH_BLOCK) smem[i] = 0u;
    __syncthreads();
    hist_runs(h, a.runs, bid, nblk);
    const float tau = a.tau, kt = a.kt;
    const bool mem = tr.arr != nullptr;
    // the walk list is shared out in batches of rb entries (lane = entry) so that every wave gets some
    const i64 nwaves = (i64)nblk * (TH_BLOCK / 64);
    const i64 nfront = (i64)tl->nlist, nlist = walks ? nfront + (i64)tl->nlist_back : 0;
    i64 rb = (nlist + nwaves - 1) / nwaves;
    rb = rb < 1 ? 1 : (rb > 64 ? 64 : rb);
    // wave w of a round takes the entries w, w + W, ... (lane = which of them), W = waves x rounds needed
    const i64 nround = (nlist + rb * nwaves - 1) / (rb * nwaves);
    for (i64 rnd = 0; rnd < nround; ++rnd) {
        const i64 gw = (i64)bid * (TH_BLOCK / 64) + wave;
        const i64 j = rnd * rb * nwaves + gw + (i64)lane * nwaves;
        const bool mine = lane < rb && j < nlist;
        const i64 i = mine ? (i64)walk_list_entry(a.list, tr.n_req, nfront, j) : 0;
        const unsigned desc = mine ? (unsigned)(a.desc[i] & 0xFFFFFFull) : DESC_NONE;
        u64 walkers = __ballot(desc != DESC_NONE);
        if (!walkers) continue;
        // the fields of the requests that are walked
        int l_v = 0, n_v = 1;
        float k_v = tr.k_s, gd_v = tr.g_s, gap_v = 0.0f;
        i64 off_v = 0;
        if (desc != DESC_NONE) {
            l_v = tr.l[i]; n_v = tr.n[i];
            if (tr.k) k_v = tr.k[i];
            if (tr.g) gd_v = tr.g[i];
            if (tr.off) off_v = tr.off[i];
            if (tr.tbt) gap_v = tr.tbt[i];
        }
        const u64 memw = mem ? __ballot((desc & 0xFFFF00u) != 0xFFFF00u) : 0ull;     // requests that read the token array
        float pre[4] = {0.f, 0.f, 0.f, 0.f};
        {
            const int r0 = __ffsll((long long)walkers) - 1;
            if ((memw >> r0) & 1ull) load_first(tr.arr, (i64)bcast_u64((u64)off_v, r0), bcast_i(n_v, r0), n_tok, align, lane, pre);
        }
        while (walkers) {
            const int rq = __ffsll((long long)walkers) - 1;
            walkers &= walkers - 1;
            const unsigned dsc = (unsigned)bcast_i((int)desc, rq);
            const int n = bcast_i(n_v, rq), l = bcast_i(l_v, rq);
            const float gd = bcast_f(gd_v, rq);
            const float cur[4] = {pre[0], pre[1], pre[2], pre[3]};
            bool have = (memw >> rq) & 1ull;
            if (walkers) {                          // the next request's first chunk is loaded while this one is walked
                const int r1 = __ffsll((long long)walkers) - 1;
                if ((memw >> r1) & 1ull)
                    load_first(tr.arr, (i64)bcast_u64((u64)off_v, r1), bcast_i(n_v, r1), n_tok, align, lane, pre);
            }
#pragma unroll 1
            for (int variant = 2; variant >= 0; --variant) {
                const unsigned sl = (dsc >> (8 * variant)) & 0xFFu;
                if (sl == 0xFFu) continue;
                const unsigned row_base = sl << width;
                auto sink = [&](const unsigned key[4]) { hist_keys(h, key, row_base, lane); };
                const bool dev = variant == 0;
                const float gap = dev ? gd : bcast_f(gap_v, rq);
                const bool from_mem = !dev && mem;
                const i64 off = from_mem ? (i64)bcast_u64((u64)off_v, rq) : 0;
                walk_hist(from_mem, n, tr.arr, off, n_tok, align, cur, from_mem && have, gap, variant == 2, gd, l,
                          bcast_f(k_v, rq), tr.c, tau, kt, lane, sink);
                if (from_mem) have = false;
            }
        }
    }
    __syncthreads();
    // LDS rows (group, walked class) -> device-wide rows (group, class)
    const unsigned dmask = (1u << width) - 1u;
    for (int i = threadIdx.x; i < words; i += TH_BLOCK) {
        const unsigned cnt = smem[i];
        if (!cnt) continue;
        const int row = i >> width;
        const int g = row / nwalk, sl = row - g * nwalk;
        const int c = tl->slot_cls[sl];
        atomicAdd(&a.ghist[((size_t)(g * ncls + c) << width) | ((unsigned)i & dmask)], cnt);
    }
}

}  // namespace
