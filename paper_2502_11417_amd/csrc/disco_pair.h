// Per-pair dispatch evaluation specialised on the kind of policy table, and
// the LDS staging record of the dispatch-type passes.
#pragma once
#include "disco_device.h"

namespace {

constexpr int DP_BLOCK = 1024;
constexpr int DP_WAVES = DP_BLOCK / 64;
constexpr int DP_MAX_BLOCKS = 256;          // one workgroup per CU: the ticket chain stays short

struct Staged { int l; float s; int n; float d; };      // 16 bytes, one per request of the batch
// What a race decides does not depend on the column: d = device TTFT, m = TTFT of a race (ties go to the server), pn = decode
// tokens with a count of one above them (n < 2^16, so 64 of them add up below bit 22), and, in an array of its
// own, pnr = pn if the device wins the race, else 0.  A threshold column (Alg. 3) only selects between the
// device-only and the race values.
struct StagedRace { int l; unsigned d, m, pn; };         // d, m: bit patterns of the two TTFT candidates
constexpr unsigned PN_COUNT_SHIFT = 22;

// ------------------------------------------------------------ per pair ----

struct PairResult { bool srv_started, dev_started, dev_win; float ttft; };

// MODE 0: every column is server-constrained (Alg. 3), 1: every column is
// device-constrained (Alg. 2 / Eq. 1), 2: mixed table or stochastic baseline columns.
template <int MODE>
__device__ __forceinline__ PairResult pair_eval(const disco_policy& p, int l, float s, float d, i64 i, bool have_u = false,
                                                float u = 0.0f)
{
    PairResult r;
    if (MODE == 0) {
        const bool dev_only = l < p.l_th;               // strict: Alg. 3
        r.srv_started = !dev_only;
        r.dev_started = true;
        r.dev_win = dev_only || (d < s);                // ties go to the server
        r.ttft = r.dev_win ? d : s;
    } else if (MODE == 1) {
        float ramp = p.beta * (float)l;
        float w = (ramp < p.w_tail) ? ramp : p.w_tail;  // a NaN ramp falls through to w_tail
        w = (l == p.l_mid) ? p.w_mid : w;
        w = (l <= p.l_th) ? 0.0f : w;
        const float x = w + d;
        r.srv_started = true;
        r.dev_started = s > w;                          // a server token at exactly w cancels the device
        r.dev_win = r.dev_started && (x < s);
        r.ttft = r.dev_win ? x : s;
    } else {
        unsigned dec; float t;
        dispatch_pair_u(p, l, s, d, i, have_u, u, dec, t);
        r.srv_started = (dec & 1u) != 0u;
        r.dev_started = (dec & 2u) != 0u;
        r.dev_win = (dec & 4u) != 0u;
        r.ttft = t;
    }
    return r;
}

// Stochastic baseline columns (Sec. 5.1) of the same run share the uniform variate of a request: the levels of a
// run are nested.  Per wave (lane = column): up to STOCH_SHARE distinct runs among the columns, lane k keeps run
// k.  Per batch of 64 requests every lane draws the variates of the request it loaded (lane = request), one per
// run; a column lane then fetches the variate of (its run, the request it evaluates) from the lane that holds it:
// R draws per request instead of one per (request, column) pair.
constexpr int STOCH_SHARE = 8;
struct StochRuns { int R; int ridx; int run_of_lane; bool on; };     // on: some stochastic column, at most STOCH_SHARE runs

__device__ __forceinline__ StochRuns stoch_runs(const disco_policy& p, bool colv, int lane)
{
    const bool st = colv && p.mode >= DISCO_MODE_STOCH_SERVER;
    u64 todo = __ballot(st);
    StochRuns s{0, -1, 0, todo != 0ull};
    while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int r0 = bcast_i(p.l_mid, leader);
        const u64 same = __ballot(st && p.l_mid == r0);
        if (st && p.l_mid == r0) s.ridx = s.R;
        if (lane == s.R) s.run_of_lane = r0;
        s.R += 1;
        todo &= ~same;
    }
    if (s.R > STOCH_SHARE) s.on = false;
    return s;
}

// lane = request i of the batch
__device__ __forceinline__ void stoch_draw(const StochRuns& s, i64 i, float u[STOCH_SHARE])
{
#pragma unroll
    for (int k = 0; k < STOCH_SHARE; ++k)
        if (k < s.R) u[k] = route_uniform(bcast_i(s.run_of_lane, k), i);
}

// the variate of (this lane's run, the request that lane `src` holds); UNIFORM: `src` is the same in every lane
template <bool UNIFORM>
__device__ __forceinline__ float stoch_fetch(const StochRuns& s, const float u[STOCH_SHARE], int src)
{
    float x = 0.0f;
#pragma unroll
    for (int k = 0; k < STOCH_SHARE; ++k)
    {
        const float v = UNIFORM ? bcast_f(u[k], src) : __shfl(u[k], src, 64);
        x = (k == s.ridx) ? v : x;
    }
    return x;
}

// Tables of stochastic columns alone: the variates of a batch are staged in LDS by (run, request), CH of the G requests
// of every sub-group at a time (c-th of G / CH rounds; the area is private to the wave), and a column lane reads the one
// of its run next to the request's record: a comparison and a selection per pair instead of STOCH_SHARE lane reads and
// the arithmetic of the other modes.  Rows are four banks apart.
template <int G, int CH>
struct StochStage {
    static constexpr int SLOTS = 64 / G * CH, STRIDE = SLOTS + 4, WORDS = STOCH_SHARE * STRIDE;
    static __device__ __forceinline__ void put(const StochRuns& s, const float u[STOCH_SHARE], float* area, int lane, int c)
    {
        __builtin_amdgcn_wave_barrier();
        if ((lane & (G - 1)) / CH == c) {
            const int slot = lane / G * CH + (lane & (CH - 1));
#pragma unroll
            for (int k = 0; k < STOCH_SHARE; ++k)
                if (k < s.R) area[k * STRIDE + slot] = u[k];
        }
        __builtin_amdgcn_wave_barrier();
    }
    static __device__ __forceinline__ float get(const float* area, int ridx, int sub, int q) { return area[ridx * STRIDE + sub * CH + q]; }
};
__device__ __forceinline__ bool all_stochastic(const disco_policy& p, bool colv)
{
    return __ballot(colv && p.mode < DISCO_MODE_STOCH_SERVER) == 0ull;
}

__device__ __forceinline__ int table_mode(const disco_policy& p, bool colv)
{
    const bool any_d = __ballot(colv && p.mode == DISCO_MODE_DEVICE_CONSTRAINED) != 0ull;
    const bool any_s = __ballot(colv && p.mode == DISCO_MODE_SERVER_CONSTRAINED) != 0ull;
    const bool any_x = __ballot(colv && p.mode >= DISCO_MODE_STOCH_SERVER) != 0ull;
    return any_x ? 2 : (any_d ? (any_s ? 2 : 1) : 0);
}

// --------------------------------------------------- per-pair outputs ----

struct PairOut { uint8_t* decision; float* ttft; };      // policy-major, nullable

// Four consecutive elements of a row that starts anywhere (gfx950 stores them in one instruction).
typedef float PairFloats __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned PairBytes __attribute__((aligned(1)));

// Workgroup `bid` of `nblk`: four consecutive requests per lane, so that a wave writes 1 KB of a TTFT row and 256 B of a decision
// row at a time; a task is a block of requests and MAT_COLS columns.
constexpr int MAT_COLS = 8;
__device__ __forceinline__ void mat_body(const TraceView& tr, const disco_policy* pol, int P, const PairOut& out, int bid, int nblk)
{
    const i64 blocks = (tr.n_req + 4 * DP_BLOCK - 1) / (4 * DP_BLOCK);
    const int chunks = (P + MAT_COLS - 1) / MAT_COLS;
    for (i64 task = bid; task < blocks * chunks; task += nblk) {
        const i64 i0 = (task / chunks) * (4 * DP_BLOCK) + 4 * (int)threadIdx.x;
        const int j0 = (int)(task % chunks) * MAT_COLS, j1 = j0 + MAT_COLS < P ? j0 + MAT_COLS : P;
        if (i0 >= tr.n_req) continue;
        const int cnt = tr.n_req - i0 < 4 ? (int)(tr.n_req - i0) : 4;
        int l[4];
        float s[4], d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const i64 i = i0 + (q < cnt ? q : 0);
            l[q] = tr.l[i]; s[q] = tr.s[i];
            d[q] = __fmaf_rn((float)l[q], tr.k ? tr.k[i] : tr.k_s, tr.c);
        }
        // a race that starts both endpoints at once (Alg. 3): the same for every column; ties go to the server
        unsigned race[4];
        float first[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) { race[q] = d[q] < s[q] ? 7u : 3u; first[q] = d[q] < s[q] ? d[q] : s[q]; }
#pragma unroll 1
        for (int j = j0; j < j1; ++j) {
            const disco_policy p = pol[j];                       // (the same for all lanes, as is its kind)
            unsigned dec[4];
            float t[4];
            if (p.mode == DISCO_MODE_SERVER_CONSTRAINED) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool dev_only = l[q] < p.l_th;         // strict: Alg. 3
                    dec[q] = dev_only ? 6u : race[q];
                    t[q] = dev_only ? d[q] : first[q];
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) dispatch_pair(p, l[q], s[q], d[q], i0 + q, dec[q], t[q]);
            }
            const size_t at = (size_t)j * tr.n_req + i0;
            if (cnt == 4) {
                if (out.ttft) *reinterpret_cast<PairFloats*>(out.ttft + at) = PairFloats{t[0], t[1], t[2], t[3]};
                if (out.decision) *reinterpret_cast<PairBytes*>(out.decision + at) = dec[0] | (dec[1] << 8) | (dec[2] << 16) | (dec[3] << 24);
            } else {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (q < cnt) {
                        if (out.ttft) out.ttft[at + q] = t[q];
                        if (out.decision) out.decision[at + q] = (uint8_t)dec[q];
                    }
            }
        }
    }
}

}  // namespace
