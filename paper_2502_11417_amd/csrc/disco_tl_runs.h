// TBT selection: the gaps of the timelines that are not analytic, counted per
// value once, so that the histogram passes need not walk their tokens again.
//
// A timeline's running maximum M moves at a few tokens (stalls, hand-offs) and
// stands still in between, where delta_t = fma(t, tau, M).  The gaps of such a
// stretch follow without its tokens.  Inside a binade of delta, with spacing u
// of the floats there, delta_t = u RN(x_t / u) for the exact x_t = t tau + M,
// so a gap is u (RN(y + s) - RN(y)) with s = tau / u: an integer in
// [s - 1, s + 1], i.e. floor(s) or ceil(s) where s is no integer.  (A token that
// is rounded up to the binade's lower end from below would round to it with
// spacing u as well.)  The sum of the gaps says how many there are of each.
// Where s is an integer every gap is tau, unless the x_t are ties and s is odd:
// then they are gone through one by one.  Differences of floats of a binade are
// exact.  The gap across the lower end of a binade is taken by itself.
// Conditions (paced_ok): 2^-20 <= tau <= 2^20, fewer than 2^22 tokens,
// 0 <= M <= 2^20; then t is exact in fp32, there are fewer than 64 binades, and
// all scalings by powers of two are exact.
//
// A timeline with more than RQ_LEN - 1 moves, or one whose gaps do not fit the
// workgroup's pool, is left to the passes, which walk it token by token.
#pragma once
#include "disco_tl_hist_buf.h"

namespace {

__device__ __forceinline__ bool paced_ok(float tau, int n)
{
    return tau >= 9.5367431640625e-07f && tau <= 1048576.0f && n < (1 << 22);
}
__device__ __forceinline__ bool paced_max_ok(float M) { return M >= 0.0f && M <= 1048576.0f; }

// Stretches (tokens ta .. tb, M from token ta - 1 on) and single gaps of the timeline that a wave has in hand, in LDS.
struct Stretch { float M; int ta, tb; int pad; };
constexpr int RQ_LEN = 20, RQ_UNDO = 40;
struct RunLds {
    Stretch st[RQ_LEN];
    unsigned single[RQ_LEN];       // bit patterns
    uint2 undo[RQ_UNDO];           // what of the pool the timeline has taken so far
};

// One timeline as stretches and single gaps; false: too many of them, or a maximum out of bounds.
//   kind   TL_ kind; m: first token of the target, 0x7FFFFFFF without hand-off (TL_SRV_LAG: from the token walk's summary)
//   ho     buffer hand-offs: base and a_m (handoff_at)
//   first  the lane's elements of the first chunk of the token window (not used without a token array)
// Same operations on the arrivals as the walkers of the passes.
__device__ __forceinline__ bool walk_runs(RunLds& q, int& ns, int& n1, int kind, int n, const float* __restrict__ arr, i64 off, i64 n_tok,
                                          int align, const float first[4], float gap, float g_dev, int l, float k, float c, int m,
                                          const Handoff& ho, float tau, float kt, int lane)
{
    const float ninf = -INFINITY;
    const bool src_dev = kind == TL_DEV || kind == TL_DEV_BUF, mem = arr != nullptr && kind != TL_DEV;
    const int mis = mem ? (int)((off + align) & 3) : 0;
    const int lane4 = 4 * lane - mis, total = n + mis;
    const i64 gbase = off + lane4;
    float M = ninf, base = ho.base;
    int ta = 1;
    ns = 0; n1 = 0;
    float nxt[4] = {first[0], first[1], first[2], first[3]};
#pragma unroll 1
    for (int e0 = 0; e0 < total; e0 += 256) {
        const int tk0 = lane4 + e0, t_here = e0 - mis, t_next = t_here + 256;      // the chunk's first token, the next one's
        const float tf0 = (float)tk0;
        const float a[4] = {nxt[0], nxt[1], nxt[2], nxt[3]};
        // the next chunk in flight, where it has tokens of the server's
        if (mem && t_next < n && (src_dev ? t_next + 255 >= m : t_next < m) && tk0 + 256 < n) load4(arr, gbase + e0 + 256, n_tok, nxt);
        float u[4] = {ninf, ninf, ninf, ninf};
        if (t_here < m) {                                    // tokens of the source
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const float tf = tf0 + (float)z, r = src_dev ? tf * g_dev : (mem ? a[z] : tf * gap);
                u[z] = __fmaf_rn(-tf, tau, r);
            }
            if (e0 == 0) {                                   // u_0 = r_0: element `mis` of lane 0
                M = bcast_f(mis == 0 ? u[0] : (mis == 1 ? u[1] : (mis == 2 ? u[2] : u[3])), 0);
                if (!paced_max_ok(M)) return false;
            }
        }
        if (t_next > m) {                                    // tokens of the target
            if (kind == TL_SRV_LAG && t_here <= m) {
                // the hand-off is decided once token m is kappa tau overdue, after the maximum through token m - 1
                float before = M;
                if (t_here < m) {
                    float mine = ninf;
#pragma unroll
                    for (int z = 0; z < 4; ++z) mine = tk0 + z >= 0 && tk0 + z < m ? fmaxf(mine, u[z]) : mine;
                    before = fmaxf(M, wave_max_f32(mine));
                }
                const float slot = __fmaf_rn((float)(m - 1), tau, before) + tau;
                const float t_dec = slot + kt, t_mig = __fmaf_rn((float)(l + m), k, c);
                base = t_dec + t_mig;
            }
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const float tf = tf0 + (float)z, since = a[z] - ho.a_m;
                const int j = tk0 + z - m + 1;
                const float r = !src_dev ? __fmaf_rn((float)j, g_dev, base) : (mem ? base + since : __fmaf_rn((float)j, gap, base));
                const float x = __fmaf_rn(-tf, tau, r);
                u[z] = tk0 + z >= m ? x : u[z];
            }
        }
        if (e0 == 0 || e0 + 256 > total) {
#pragma unroll
            for (int z = 0; z < 4; ++z) u[z] = (unsigned)(tk0 + z) < (unsigned)n ? u[z] : ninf;
        }
        const float i0 = u[0], i1 = fmaxf(i0, u[1]), i2 = fmaxf(i1, u[2]), i3 = fmaxf(i2, u[3]);
        if (__ballot(i3 > M) == 0ull) continue;
        // the tokens that move the maximum, one after the other
        const float E = fmaxf(wave_prev(wave_incl_max_dpp(i3, lane), ninf), M);
        u64 rec[4] = {__ballot(i0 > E), __ballot(u[1] > fmaxf(E, i0)), __ballot(u[2] > fmaxf(E, i1)), __ballot(u[3] > fmaxf(E, i2))};
        if (n1 + __popcll(rec[0]) + __popcll(rec[1]) + __popcll(rec[2]) + __popcll(rec[3]) >= RQ_LEN) return false;
        while ((rec[0] | rec[1] | rec[2] | rec[3]) != 0ull) {
            const int ln = __ffsll((long long)(rec[0] | rec[1] | rec[2] | rec[3])) - 1;
            const u64 bit = 1ull << ln;
            const int z = (rec[0] & bit) ? 0 : ((rec[1] & bit) ? 1 : ((rec[2] & bit) ? 2 : 3));
            if (z == 0) rec[0] &= ~bit; else if (z == 1) rec[1] &= ~bit; else if (z == 2) rec[2] &= ~bit; else rec[3] &= ~bit;
            const float up = bcast_f(z == 0 ? u[0] : (z == 1 ? u[1] : (z == 2 ? u[2] : u[3])), ln);
            const int t = t_here + 4 * ln + z;
            if (!paced_max_ok(up)) return false;
            if (lane == 0) {
                if (t > ta) q.st[ns] = Stretch{M, ta, t - 1, 0};
                q.single[n1] = f2u(__fmaf_rn((float)t, tau, up) - __fmaf_rn((float)(t - 1), tau, M));
            }
            ns += t > ta ? 1 : 0;
            n1 += 1;
            M = up;
            ta = t + 1;
        }
    }
    if (ta < n) {
        if (lane == 0) q.st[ns] = Stretch{M, ta, n - 1, 0};
        ns += 1;
    }
    return true;
}

// The gaps of a timeline into the workgroup's pool (`used`: entries taken, in LDS); false, and nothing added, if they do
// not fit.  Four stretches side by side, 15 binades at a time by 16 lanes each.
__device__ __forceinline__ bool emit_runs(RunLds& q, int ns, int n1, unsigned row, float tau, uint2* __restrict__ pool, unsigned cap,
                                          unsigned* used, int lane)
{
    const unsigned tag = row << RUN_COUNT_BITS;
    int undo = 0;
    bool ok = true;
    // entries of the wave: up to three per lane
    auto add = [&](const unsigned gap[3], const unsigned count[3]) {
        u64 has[3];
        unsigned before = 0u, all = 0u;
#pragma unroll
        for (int z = 0; z < 3; ++z) {
            has[z] = __ballot(count[z] != 0u);
            before += (unsigned)__popcll(has[z] & ((1ull << lane) - 1ull));
            all += (unsigned)__popcll(has[z]);
        }
        if (all == 0u) return;
        unsigned at = 0u;
        if (lane == 0) at = atomicAdd(used, all);
        at = 1u + (unsigned)__builtin_amdgcn_readfirstlane((int)at);
        ok = ok && undo < RQ_UNDO && at + all <= cap;
        if (lane == 0 && undo < RQ_UNDO) q.undo[undo] = make_uint2(at, all);
        undo += undo < RQ_UNDO ? 1 : 0;
        unsigned mine = at + before;
#pragma unroll
        for (int z = 0; z < 3; ++z)
            if (count[z] != 0u) {
                if (mine < cap) pool[mine] = make_uint2(gap[z], ok ? count[z] | tag : 0u);
                mine += 1u;
            }
    };
    __builtin_amdgcn_wave_barrier();
    const int sub = lane & 15;
    const float per_tau = 1.0f / tau;
    // the single gaps: in the lanes that close the groups of 16, three each, of the first step if they fit there
    int singles = n1;
    if (ns == 0 || n1 > 12) {
        const unsigned gap[3] = {q.single[lane < n1 ? lane : 0], 0u, 0u}, count[3] = {lane < n1 ? 1u : 0u, 0u, 0u};
        add(gap, count);
        singles = 0;
    }
#pragma unroll 1
    for (int e = 0; e < ns && ok; e += 4) {
        const bool on = e + (lane >> 4) < ns;
        const Stretch st = q.st[on ? e + (lane >> 4) : e];
        const float M = st.M;
        const int ta = st.ta, tb = st.tb;
        auto delta = [&](int t) { return __fmaf_rn((float)t, tau, M); };
        const int E0 = (int)(f2u(delta(ta)) >> 23), E1 = (int)(f2u(delta(tb)) >> 23);
#pragma unroll 1
        for (int E = E0 + sub; __ballot(on && E - sub <= E1) != 0ull && ok; E += 15) {
            // the first token of the lane's binade, tb + 1 if there is none
            int from = tb + 1;
            if (E == E0) from = ta;
            else if (E <= E1) {
                const float low = u2f((unsigned)E << 23);
                int t = (int)ceilf((low - M) * per_tau);
                t = t < ta ? ta : (t > tb ? tb : t);
                while (t > ta && delta(t - 1) >= low) --t;
                while (t <= tb && delta(t) < low) ++t;
                from = t;
            }
            const int last = __shfl_down(from, 1, 16) - 1;
            const bool mine = on && sub != 15 && E <= E1 && last >= from;
            unsigned gap[3] = {0u, 0u, 0u}, count[3] = {0u, 0u, 0u};
            int one_by_one = 0;                              // ties: gaps left to go through
            if (mine) {
                const float d0 = delta(from);
                gap[0] = f2u(d0 - delta(from - 1)); count[0] = 1u;
                const unsigned cnt = (unsigned)(last - from);
                const float u = u2f((unsigned)(E - 23) << 23), per_u = u2f((unsigned)(277 - E) << 23);
                const float s = tau * per_u, f = floorf(s);
                if (s == f && ((unsigned)f & 1u) != 0u && M * per_u - floorf(M * per_u) == 0.5f) {
                    one_by_one = (int)cnt;
                } else {
                    const unsigned more = (unsigned)(int)((delta(last) - d0) * per_u) - cnt * (unsigned)f;   // (mod 2^32: at most cnt)
                    gap[1] = f2u(f * u); count[1] = cnt - more;
                    gap[2] = f2u((f + 1.0f) * u); count[2] = more;
                }
            }
            if (singles != 0 && sub == 15) {
#pragma unroll
                for (int z = 0; z < 3; ++z) {
                    const int at = 3 * (lane >> 4) + z;
                    gap[z] = q.single[at]; count[z] = at < singles ? 1u : 0u;
                }
            }
            singles = 0;
            add(gap, count);
            for (int z = 0; __ballot(z < one_by_one) != 0ull && ok; ++z) {
                const unsigned g1[3] = {z < one_by_one ? f2u(delta(from + 1 + z) - delta(from + z)) : 0u, 0u, 0u};
                const unsigned c1[3] = {z < one_by_one ? 1u : 0u, 0u, 0u};
                add(g1, c1);
            }
        }
    }
    if (!ok) {
        __builtin_amdgcn_wave_barrier();
        for (int z = 0; z < undo; ++z) {
            const uint2 x = q.undo[z];
            for (unsigned i = x.x + (unsigned)lane; i < x.x + x.y && i < cap; i += 64u) pool[i] = make_uint2(0u, 0u);
        }
    }
    __builtin_amdgcn_wave_barrier();
    return ok;
}

}  // namespace
