// One class-mode TBT histogram pass over the timelines with a buffer hand-off
// (Sec. 4.3) that have tokens to walk: the workgroup body, shared by the
// kernel of the regular passes and the kernel of the spare passes.
#pragma once
#include "disco_tl_general.h"
#include "disco_tl_hist_fast.h"
#include "disco_tl_walk.h"

namespace {

constexpr int TBH_BLOCK = 1024;              // histogram workgroups: 16 waves share the LDS bins

struct BufHistArgs {
    HistArgs h;
    const BufSummary* bufsum;      // the hand-offs, as the statistics of the timelines found them (k_tl_classify has checked them)
    const unsigned* buffer_flag;
};

// A hand-off at source token m (-1: none): base = the instant the target's arrivals count from, a_m = the server's own
// arrival offset of token m (device source: its tokens behind the hand-off follow the token array).
struct Handoff { int m; float base, a_m; };

__device__ __forceinline__ Handoff handoff_at(bool src_dev, int m, const float* __restrict__ arr, i64 off, int l, float s_ttft, float k,
                                              float c, float gap, float g_dev)
{
    Handoff h{m, 0.0f, 0.0f};
    if (m < 0) return h;
    // the source's arrival at the hand-off and the target's prefill
    const float r_m = src_dev ? (float)m * g_dev : (arr ? arr[off + m] : (float)m * gap);
    h.base = r_m + (src_dev ? s_ttft : __fmaf_rn((float)(l + m + 1), k, c));
    if (src_dev && arr) h.a_m = arr[off + m];
    return h;
}

// Histogram walk of one timeline whose hand-off is known: the operations of the general walker on the spliced
// arrivals, without its search for the hand-off -- a test of every token with a double-precision cost comparison -- and
// without the scan of chunks in which the running maximum does not move.  Gaps -> sink(key[4]) as in walk_hist.
//   src_dev  device source, the server's tokens behind the hand-off; else the other way round
//   first    the lane's elements of the first chunk of the token window (not used without a token array)
// Bound by vector issue.  A pass over 10^6 requests x 8 columns 74 and 87 us with the general walker, 59 and 73 us; 10^5
// requests x 12 wait columns 28 -> 24 us.
template <class Sink>
__device__ __forceinline__ void walk_hist_known(bool src_dev, int n, const float* __restrict__ arr, i64 off, i64 n_tok, int align,
                                                const float first[4], float gap, float g_dev, const Handoff& ho, float tau, int lane,
                                                Sink&& sink)
{
    const float ninf = -INFINITY;
    const bool mem = arr != nullptr;
    const int mis = mem ? (int)((off + align) & 3) : 0;
    const int lane4 = 4 * lane - mis, total = n + mis, m = ho.m;
    const i64 gbase = off + lane4;
    float carryM = ninf, carryD = 0.0f;
    float nxt[4] = {first[0], first[1], first[2], first[3]};
#pragma unroll 1
    for (int e0 = 0; e0 < total; e0 += 256) {
        const int tk0 = lane4 + e0;
        const int t_next = e0 + 256 - mis;                   // the next chunk's first token
        const float tf0 = (float)tk0;
        const float tf[4] = {tf0, tf0 + 1.0f, tf0 + 2.0f, tf0 + 3.0f};
        const float a[4] = {nxt[0], nxt[1], nxt[2], nxt[3]};
        // the next chunk in flight, where it has tokens of the server's
        if (mem && t_next < n && (src_dev ? (m >= 0 && t_next + 255 > m) : (m < 0 || t_next <= m)) && tk0 + 256 < n)
            load4(arr, gbase + e0 + 256, n_tok, nxt);
        float r[4], u[4];
        if (m < 0 || e0 - mis <= m) {                        // tokens of the source
#pragma unroll
            for (int q = 0; q < 4; ++q) r[q] = src_dev ? tf[q] * g_dev : (mem ? a[q] : tf[q] * gap);
        }
        if (m >= 0 && t_next - 1 > m) {                      // tokens of the target
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float since = a[q] - ho.a_m;
                const float at = src_dev ? (mem ? ho.base + since : __fmaf_rn((float)(tk0 + q - m), gap, ho.base))
                                         : __fmaf_rn((float)(tk0 + q - m), g_dev, ho.base);
                r[q] = tk0 + q > m ? at : r[q];
            }
        }
        const bool full = e0 > 0 && e0 + 256 <= total;       // every element of the chunk is a token of the request
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u[q] = __fmaf_rn(-tf[q], tau, r[q]);
            if (!full) u[q] = (unsigned)(tk0 + q) < (unsigned)n ? u[q] : ninf;
        }
        const float i0 = u[0], i1 = fmaxf(i0, u[1]), i2 = fmaxf(i1, u[2]), i3 = fmaxf(i2, u[3]);
        float M[4] = {carryM, carryM, carryM, carryM};
        if (__ballot(i3 > carryM) != 0ull) {
            const float E = fmaxf(wave_prev(wave_incl_max_dpp(i3, lane), ninf), carryM);
            M[0] = fmaxf(E, i0); M[1] = fmaxf(E, i1); M[2] = fmaxf(E, i2); M[3] = fmaxf(E, i3);
        }
        float d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q] = __fmaf_rn(tf[q], tau, M[q]);
        const float p0 = wave_prev(d[3], carryD);
        unsigned key[4] = {f2u(d[0] - p0), f2u(d[1] - d[0]), f2u(d[2] - d[1]), f2u(d[3] - d[2])};
        if (!full) {
#pragma unroll
            for (int q = 0; q < 4; ++q) key[q] = (unsigned)(tk0 + q - 1) < (unsigned)(n - 1) ? key[q] : KEY_SKIP;
        }
        sink(key);
        carryM = bcast_f(M[3], 63);
        carryD = bcast_f(d[3], 63);
    }
}

// Workgroup `bid` of `nblk`: bytes 3 and 4 of a request's descriptor name the LDS rows of its two hand-off kinds,
// the walk list of the selection names the requests.  `smem`: DISCO_TL_HIST_WORDS words of LDS.
__device__ __forceinline__ void tl_hist_buf_body(unsigned* smem, const TraceView& tr, i64 n_tok, int align, const BufHistArgs& ba,
                                                 const TlPlan& pl, unsigned bid, unsigned nblk)
{
    const HistArgs& a = ba.h;
    const TlSel* tl = &a.S->tl;
    const int width = __builtin_amdgcn_readfirstlane(pl.width);
    if (*ba.buffer_flag == 0u || (__builtin_amdgcn_readfirstlane(pl.walks) & 2) == 0 || width <= 0 || pl.fallback) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ncls = tl->ncls, nwalk = tl->nwalk;
    const HistCtx h = hist_ctx(smem, pl, nwalk);
    const int words = (h.G * nwalk) << width;
    for (int i = threadIdx.x; i < words; i += TBH_BLOCK) smem[i] = 0u;
    __syncthreads();
    const i64 nwaves = (i64)nblk * (TBH_BLOCK / 64);
    const i64 nfront = (i64)tl->nlist, nlist = nfront + (i64)tl->nlist_back;
    i64 rb = (nlist + nwaves - 1) / nwaves;
    rb = rb < 1 ? 1 : (rb > 64 ? 64 : rb);
    const i64 nround = (nlist + rb * nwaves - 1) / (rb * nwaves);
    for (i64 rnd = 0; rnd < nround; ++rnd) {
        const i64 gw = (i64)bid * (TBH_BLOCK / 64) + wave;
        const i64 j = rnd * rb * nwaves + gw + (i64)lane * nwaves;
        const bool mine = lane < rb && j < nlist;
        const i64 il = mine ? (i64)walk_list_entry(a.list, tr.n_req, nfront, j) : 0;
        const unsigned desc = mine ? (unsigned)((a.desc[il] >> 24) & 0xFFFFull) : 0xFFFFu;
        u64 walkers = __ballot(desc != 0xFFFFu);
        if (!walkers) continue;
        int l_v = 0, n_v = 1;
        float k_v = tr.k_s, gd_v = tr.g_s, gap_v = 0.0f, s_v = 0.0f;
        i64 off_v = 0;
        Handoff from_srv{-1, 0.0f, 0.0f}, from_dev{-1, 0.0f, 0.0f};
        if (desc != 0xFFFFu) {
            l_v = tr.l[il]; n_v = tr.n[il]; s_v = tr.s[il];
            if (tr.k) k_v = tr.k[il];
            if (tr.g) gd_v = tr.g[il];
            if (tr.off) off_v = tr.off[il];
            if (tr.tbt) gap_v = tr.tbt[il];
            const BufSummary bs = ba.bufsum[il];
            const int m_s = (desc & 0xFFu) != 0xFFu ? summary_m(bs.m_s) : -1, m_d = (desc >> 8) != 0xFFu ? summary_m(bs.m_d) : -1;
            from_srv = handoff_at(false, m_s, tr.arr, off_v, l_v, s_v, k_v, tr.c, gap_v, gd_v);
            from_dev = handoff_at(true, m_d, tr.arr, off_v, l_v, s_v, k_v, tr.c, gap_v, gd_v);
        }
        float ahead[4] = {0.f, 0.f, 0.f, 0.f};
        auto load_ahead = [&](u64 left) {
            if (!left || !tr.arr) return;
            const int r = __ffsll((long long)left) - 1;
            load_first(tr.arr, (i64)bcast_u64((u64)off_v, r), bcast_i(n_v, r), n_tok, align, lane, ahead);
        };
        load_ahead(walkers);
        while (walkers) {
            const int rq = __ffsll((long long)walkers) - 1;
            walkers &= walkers - 1;
            const unsigned dsc = (unsigned)bcast_i((int)desc, rq);
            const int n = bcast_i(n_v, rq);
            const float gd = bcast_f(gd_v, rq), gap = bcast_f(gap_v, rq);
            const i64 off = tr.arr ? (i64)bcast_u64((u64)off_v, rq) : 0;
            const float chunk[4] = {ahead[0], ahead[1], ahead[2], ahead[3]};
            load_ahead(walkers);                             // the next request's first chunk, while this one is walked
#pragma unroll 1
            for (int kind = 1; kind >= 0; --kind) {
                const unsigned sl = (dsc >> (8 * kind)) & 0xFFu;
                if (sl == 0xFFu) continue;
                const unsigned row_base = sl << width;
                auto sink = [&](const unsigned key[4]) { hist_keys(h, key, row_base, lane); };
                const Handoff& v = kind ? from_dev : from_srv;
                const Handoff ho{bcast_i(v.m, rq), bcast_f(v.base, rq), bcast_f(v.a_m, rq)};
                walk_hist_known(kind != 0, n, tr.arr, off, n_tok, align, chunk, gap, gd, ho, a.tau, lane, sink);
            }
        }
    }
    __syncthreads();
    // LDS rows (group, walked class) -> device-wide rows (group, class)
    const unsigned dmask = (1u << width) - 1u;
    for (int i = threadIdx.x; i < words; i += TBH_BLOCK) {
        const unsigned cnt = smem[i];
        if (!cnt) continue;
        const int row = i >> width;
        const int g = row / nwalk, sl = row - g * nwalk;
        const int c = tl->slot_cls[sl];
        atomicAdd(&a.ghist[((size_t)(g * ncls + c) << width) | ((unsigned)i & dmask)], cnt);
    }
}

}  // namespace
