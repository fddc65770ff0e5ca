// disco_gen_trace: synthetic trace on the device.
//
// Stand-in for the measured server traces and device profiles of Sec. 5.1;
// the recipe (log-normal prompt length and server TTFT, server TTFT
// independent of prompt length, device TTFT linear in it) follows Sec. 3 and
// the scalability study of Sec. 5.3.  Random numbers come from Philox4x32-10
// (Salmon et al., SC'11) keyed by the seed and counted by (element index,
// field), so every element is independent of the launch geometry.  The
// elementary functions are fixed sequences of IEEE fp32 operations, which
// makes the trace reproducible bit for bit by any other implementation of the
// same definition.
#include "disco_common.h"
#include "disco_device.h"

namespace {

// Correctly rounded f / d and sqrt(x) for the operands below without the scaling steps of the general operations
// (no operand here is near the ends of the exponent range): an approximate reciprocal (reciprocal root), one Newton
// step, and a last correction with the exact remainder (Markstein's scheme).  That the last rounding is right for
// every operand is not left to the theorem's conditions: the generator only ever takes logarithms of the 2^23
// variates of u23, and for all of them the tests compare both results with IEEE operations (disco_gen_math_probe).
__device__ __forceinline__ float gen_div(float f, float d)
{
    const float r0 = __builtin_amdgcn_rcpf(d);
    const float r = __fmaf_rn(__fmaf_rn(-d, r0, 1.0f), r0, r0);
    const float q = f * r;
    return __fmaf_rn(__fmaf_rn(-d, q, f), r, q);
}
__device__ __forceinline__ float gen_sqrt(float x)
{
    const float y = __builtin_amdgcn_rsqf(x);
    float g = x * y, h = 0.5f * y;
    const float e = __fmaf_rn(-h, g, 0.5f);
    g = __fmaf_rn(g, e, g);
    h = __fmaf_rn(h, e, h);
    return __fmaf_rn(__fmaf_rn(-g, g, x), h, g);
}

// ln of a positive normal number: x = 2^e m with m in (sqrt(1/2), sqrt(2)],
// ln m = 2 atanh(s), s = (m - 1) / (m + 1), odd series through s^11.
struct LnParts { float f; int e; };                      // x = 2^e (1 + f)
__device__ __forceinline__ LnParts gen_ln_parts(float x)
{
    // m = the fraction of x, halved (and e + 1) where it is above 1.41421354: the bit pattern is rebased to the
    // successor of half that number
    constexpr unsigned LOW = 0x3F3504F4u;
    const unsigned rel = f2u(x) + (0x3F800000u - LOW);
    const int e = (int)(rel >> 23) - 127;
    const float m = u2f((rel & 0x007FFFFFu) + LOW);
    return LnParts{m - 1.0f, e};
}
__device__ __forceinline__ float gen_ln(float x)
{
    const LnParts q = gen_ln_parts(x);
    const float f = q.f;
    const int e = q.e;
    float s = gen_div(f, 2.0f + f);
    float z = s * s;
    float p = __fmaf_rn(z, 0.181818187f, 0.222222224f);
    p = __fmaf_rn(z, p, 0.285714298f);
    p = __fmaf_rn(z, p, 0.400000006f);
    p = __fmaf_rn(z, p, 0.666666687f);
    float sz = s * z;
    float lnm = __fmaf_rn(sz, p, 2.0f * s);
    return __fmaf_rn((float)e, 0.693147182f, lnm);
}

// Adding this to |x| < 2^22 rounds x to the nearest integer (ties to even) and leaves it in the sum's low bits.
constexpr float GEN_RINT = 12582912.0f;

// exp on [-86, 88]: n = rint(x log2 e), r = x - n ln 2 (two-part ln 2),
// series of e^r through r^7, exact scaling by 2^n.
__device__ __forceinline__ float gen_exp(float x)
{
    // (a NaN stays one; the median of the three in one instruction would make a bound of it)
    x = __builtin_elementwise_minimum(__builtin_elementwise_maximum(x, -86.0f), 88.0f);
    float t = x * 1.44269502f + GEN_RINT;
    float n = t - GEN_RINT;
    float r = __fmaf_rn(n, -0.693145752f, x);
    r = __fmaf_rn(n, -1.42860677e-06f, r);
    float p = __fmaf_rn(r, 1.98412701e-04f, 1.38888892e-03f);
    p = __fmaf_rn(r, p, 8.33333377e-03f);
    p = __fmaf_rn(r, p, 4.16666679e-02f);
    p = __fmaf_rn(r, p, 0.166666672f);
    p = __fmaf_rn(r, p, 0.5f);
    p = __fmaf_rn(r, p, 1.0f);
    p = __fmaf_rn(r, p, 1.0f);
    return p * u2f((f2u(t) << 23) + 0x3F800000u);            // 2^n: the shift leaves n alone of the sum's bits
}

// cos(2 pi u), u in (0,1): quadrant q = rint(4u), v = u - q/4 exactly,
// a = 2 pi v in [-pi/4, pi/4], series of cos and sin.
__device__ __forceinline__ float gen_cos2pi(float u)
{
    const float t = __fmaf_rn(4.0f, u, GEN_RINT);            // (4 u is exact: the same as in two operations)
    float q = t - GEN_RINT;
    float v = __fmaf_rn(q, -0.25f, u);
    float a = v * 6.28318548f;
    float a2 = a * a;
    float c = __fmaf_rn(a2, -2.75573200e-07f, 2.48015876e-05f);
    c = __fmaf_rn(a2, c, -1.38888892e-03f);
    c = __fmaf_rn(a2, c, 4.16666679e-02f);
    c = __fmaf_rn(a2, c, -0.5f);
    c = __fmaf_rn(a2, c, 1.0f);
    float s = __fmaf_rn(a2, -2.50521079e-08f, 2.75573188e-06f);
    s = __fmaf_rn(a2, s, -1.98412701e-04f);
    s = __fmaf_rn(a2, s, 8.33333377e-03f);
    s = __fmaf_rn(a2, s, -0.166666672f);
    s = __fmaf_rn(a2, s, 1.0f);
    s = s * a;
    const unsigned qi = f2u(t);
    const float res = (qi & 1u) ? s : c;
    // q = 0: c, 1: -s, 2: -c, 3: s
    return u2f(f2u(res) ^ (((qi + 1u) << 30) & 0x80000000u));
}

__device__ __forceinline__ float gen_normal(unsigned w0, unsigned w1)
{
    float rad = gen_sqrt(-2.0f * gen_ln(u23(w0)));
    return rad * gen_cos2pi(u23(w1));
}

// The division and the square root of every variate u23 can take: operands and results.
__global__ __launch_bounds__(256) void k_gen_math_probe(float* __restrict__ out)
{
    const unsigned i = blockIdx.x * 256u + threadIdx.x;
    constexpr unsigned N = 1u << 23;
    const float u = u23(i << 9), f = gen_ln_parts(u).f, x = -2.0f * gen_ln(u);
    out[i] = f; out[N + i] = gen_div(f, 2.0f + f);
    out[2 * N + i] = x; out[3 * N + i] = gen_sqrt(x);
}

__device__ __forceinline__ float gen_lognormal(unsigned w0, unsigned w1, float mu, float sigma)
{
    return gen_exp(__fmaf_rn(sigma, gen_normal(w0, w1), mu));
}

__device__ __forceinline__ int floor_clamp(float v, int lo, int hi)
{
    float f = floorf(v);
    f = (f < (float)lo) ? (float)lo : f;
    f = (f > (float)hi) ? (float)hi : f;
    return (int)f;
}

enum { F_PROMPT = 0, F_OUTPUT = 1, F_TTFT = 2, F_TBT = 3, F_DEVICE = 4, F_GAP = 5 };

__global__ __launch_bounds__(256) void k_gen_requests(disco_gen_params g, int32_t* prompt_len, int32_t* output_len,
                                                      float* srv_ttft, float* srv_tbt, float* dev_pre_spt,
                                                      float* dev_dec_spt)
{
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n_req) return;
    Words w = philox4x32_10(g.seed, (u64)i, F_PROMPT);
    prompt_len[i] = floor_clamp(gen_lognormal(w.w0, w.w1, g.prompt_mu, g.prompt_sigma), g.prompt_lo, g.prompt_hi);
    w = philox4x32_10(g.seed, (u64)i, F_OUTPUT);
    output_len[i] = floor_clamp(gen_lognormal(w.w0, w.w1, g.out_mu, g.out_sigma), g.out_lo, g.out_hi);
    w = philox4x32_10(g.seed, (u64)i, F_TTFT);
    float s;
    if (u23(w.w2) < g.ttft_pareto_p) {
        float inv_alpha = __fdiv_rn(1.0f, g.ttft_pareto_alpha);
        float e = -gen_ln(u23(w.w3));
        e = e * inv_alpha;
        s = g.ttft_pareto_xm * gen_exp(e);
    } else {
        s = gen_lognormal(w.w0, w.w1, g.ttft_mu, g.ttft_sigma);
    }
    srv_ttft[i] = s;
    w = philox4x32_10(g.seed, (u64)i, F_TBT);
    srv_tbt[i] = gen_lognormal(w.w0, w.w1, g.tbt_mu, g.tbt_sigma);
    w = philox4x32_10(g.seed, (u64)i, F_DEVICE);
    float dec, pre;
    if (g.dev_mode == 0) {
        dec = g.dev_a; pre = g.dev_b;
    } else {
        float rate;
        if (g.dev_mode == 1) rate = __fmaf_rn(u23(w.w0), g.dev_b - g.dev_a, g.dev_a);
        else rate = (u23(w.w0) < g.dev_p) ? g.dev_a : g.dev_b;
        dec = __fdiv_rn(1.0f, rate);
        pre = __fdiv_rn(dec, g.dev_pre_ratio);
    }
    dev_dec_spt[i] = dec;
    dev_pre_spt[i] = pre;
}

// Exclusive prefix sum of output_len into tok_off[0..n] in two launches: the sum of every tile, then per tile the
// sum of the tiles in front of it and a scan of its own elements.  Integer sums: any order gives the same offsets.
constexpr int GO_BLOCK = 1024;
constexpr int GO_MAX_TILES = 65536;
// Tile sums between the two launches (device memory of the library's code object, referenced by device code only).
// Calls of disco_gen_trace on one GPU share it: they must not overlap in time.
__device__ i64 g_tile_sum[GO_MAX_TILES];

__device__ __forceinline__ i64 block_sum_1024(i64 v, i64* sh)
{
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    i64 t = 0;
    for (int w = 0; w < GO_BLOCK / 64; ++w) t += sh[w];
    return t;
}

__global__ __launch_bounds__(GO_BLOCK) void k_gen_tile_sums(i64 n, i64 per_thread, const int32_t* __restrict__ output_len)
{
    __shared__ i64 sh[GO_BLOCK / 64];
    const i64 tile = per_thread * GO_BLOCK;
    const i64 lo = (i64)blockIdx.x * tile;
    i64 acc = 0;
    for (i64 q = 0; q < per_thread; ++q) {                   // coalesced: consecutive threads, consecutive elements
        const i64 i = lo + q * GO_BLOCK + threadIdx.x;
        if (i < n) acc += output_len[i];
    }
    acc = block_sum_1024(acc, sh);
    if (threadIdx.x == 0) g_tile_sum[blockIdx.x] = acc;
}

__global__ __launch_bounds__(GO_BLOCK) void k_gen_offsets(i64 n, i64 per_thread, const int32_t* __restrict__ output_len,
                                                          i64* __restrict__ tok_off)
{
    __shared__ i64 sh[GO_BLOCK / 64];
    __shared__ i64 wsum[GO_BLOCK / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const i64 tile = per_thread * GO_BLOCK;
    const i64 lo = (i64)blockIdx.x * tile;
    i64 before = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += GO_BLOCK) before += g_tile_sum[b];
    i64 run = block_sum_1024(before, sh);                    // tokens of the tiles in front
    // the tile in rounds of 1024 consecutive elements: scan across the workgroup, carry `run`
    for (i64 q = 0; q < per_thread; ++q) {
        const i64 i = lo + q * GO_BLOCK + threadIdx.x;
        const i64 v = i < n ? (i64)output_len[i] : 0;
        i64 inc = v;
        for (int d = 1; d < 64; d <<= 1) {
            const i64 o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        __syncthreads();
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        i64 front = 0, all = 0;
        for (int w = 0; w < GO_BLOCK / 64; ++w) { const i64 t = wsum[w]; front += w < wave ? t : 0; all += t; }
        if (i < n) tok_off[i] = run + front + inc - v;
        run += all;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) tok_off[n] = run;
}

// Per-token gap in front of global token index j.  stall_below: the variates u23 of which are below the stall
// probability are those of w >> 9 below this number (a uniform bound instead of a conversion per token).
__device__ __forceinline__ unsigned gen_stall_below(float p)
{
    unsigned lo = 0u, hi = 1u << 23;                         // u23 grows with its bits: the first that is not below p
    while (lo < hi) {
        const unsigned mid = (lo + hi) >> 1;
        if (u23(mid << 9) < p) lo = mid + 1u; else hi = mid;
    }
    return lo;
}
__device__ __forceinline__ float gen_gap(const disco_gen_params& g, unsigned stall_below, u64 j)
{
    const Words w = philox4x32_10(g.seed, j, F_GAP);
    const float stall = __fmaf_rn(u23(w.w3), g.gap_stall_hi - g.gap_stall_lo, g.gap_stall_lo);
    const float gap = gen_lognormal(w.w0, w.w1, g.gap_mu, g.gap_sigma);
    return (w.w2 >> 9) < stall_below ? stall : gap;
}

// Arrival offsets: running fp32 sum of a request's gaps in index order (the first token's offset is 0, its gap
// unused).  The order of the additions is part of the trace's definition, so one lane adds up a request token after
// token; everything else is spread over the wave.  A wave owns R requests and goes through them in pieces of
// K = 1024 / R tokens, as long as any has tokens left: all lanes make the gaps of one row's piece after the other
// (the work follows the tokens, not the longest request), the owner of each row adds them up in LDS, all lanes store
// the offsets.  Pieces start at multiples of 32 tokens, so they are whole lines of the token array but for a
// request's ends.
// Bound by the arithmetic of the gaps: 168 vector instructions per 64 tokens at 3.3 cycles each (18 of them wide
// multiplications of the counter-based generator); the gaps never reach device memory.  4.3 KB of LDS and 56
// registers per wave leave eight waves per SIMD (16 KB tiles of 64 requests: four waves, a tenth slower).
// 491 M tokens of 10^6 requests: 1.75 ms; gaps and sums in two kernels with the gaps in device memory between them
// took 1.9 + 5.2 ms, the second waiting for the longest of every 256 requests.  1 M tokens of 2000 requests: 1.07 ms
// -> 0.06 ms.
constexpr int GT_LOG_TILE = 10;

template <int LOG_R, bool WIDE>
__global__ __launch_bounds__(64) void k_gen_tokens(disco_gen_params g, i64 n_req, const i64* __restrict__ tok_off,
                                                   float* __restrict__ tok_arr)
{
    constexpr int R = 1 << LOG_R, LOG_K = GT_LOG_TILE - LOG_R, K = 1 << LOG_K;
    constexpr int KS = K + 4;                                // row stride: 16-byte accesses of a lane per row spread over the banks
    static_assert(LOG_K >= 6, "a step is 64 tokens of one row");
    __shared__ __align__(16) float tile[R * KS];
    const int lane = threadIdx.x;
    const unsigned stall_below = gen_stall_below(g.gap_stall_p);
    const i64 i = (i64)blockIdx.x * R + lane;
    i64 at = 0;                                              // token index of the row's next piece (a multiple of 32)
    int lo = 0, left = 0;                                    // the request's first token in the first piece, tokens left from its start
    if (lane < R && i < n_req) {
        const i64 a = tok_off[i];
        at = a & ~(i64)31;
        lo = (int)(a - at);
        left = (int)(tok_off[i + 1] - at);
    }
    float acc = 0.0f;
    // Short requests: where all tokens of the wave's requests fit the tile, their gaps are made as one stretch instead of
    // row by row (a row of a few tokens leaves most lanes idle: 400 000 requests of 1 to 3 tokens 82 us,
    // now 17).
    const i64 start = (i64)bcast_u64((u64)at, 0);
    const u64 valid = __ballot(lane < R && i < n_req);       // (never empty)
    const int last = 63 - __clzll((long long)valid);
    const i64 stretch = (i64)bcast_u64((u64)(at + left), last) - start;
    if (R > 1 && stretch <= R * K) {
        const int lead = bcast_i(lo, 0), end = (int)stretch;
        for (int q = lane; q - lane < end; q += 64) {
            u64 j = (u64)start + (u64)q;
            if (!WIDE) j = (unsigned)start + (unsigned)q;
            tile[q] = gen_gap(g, stall_below, j);
        }
        __builtin_amdgcn_wave_barrier();
        if (left > lo) {                                     // (left counts from the row's boundary, lo is its first token)
            const int first = (int)(at - start) + lo, behind = (int)(at - start) + left;
            tile[first] = 0.0f;
#pragma unroll 4
            for (int q = first + 1; q < behind; ++q) { acc = acc + tile[q]; tile[q] = acc; }
        }
        __builtin_amdgcn_wave_barrier();
        for (int q = lane; q < end; q += 64)
            if (q >= lead) tok_arr[start + q] = tile[q];
        return;
    }
    int gap_lo = lo + 1;                                     // first token of the piece that a gap is added for
    for (u64 m = __ballot(left > 0); m != 0ull; m = __ballot(left > 0)) {
        // (a lone request's last piece ends with its tokens: 8000 requests of up to 200 tokens 67 -> 20 us; with more rows a
        // piece is short enough as it is)
        const int len = R == 1 && bcast_i(left, 0) < K ? (bcast_i(left, 0) + 63) & ~63 : K;
        for (u64 rows = m; rows != 0ull; rows &= rows - 1ull) {
            const int r = __ffsll((long long)rows) - 1;
            const u64 base = bcast_u64((u64)at, r);
            const int r_lo = bcast_i(gap_lo, r), r_hi = bcast_i(left, r);
#pragma unroll 2
            for (int q0 = 0; q0 < len; q0 += 64) {
                const int q = q0 + lane;
                float gap = 0.0f;
                if (q0 < r_hi) {                             // (the same in every lane)
                    u64 j = base + (u64)q;
                    if (!WIDE) j = (unsigned)base + (unsigned)q;     // (all token indices below 2^32: the counter's high word is 0)
                    gap = gen_gap(g, stall_below, j);
                    gap = (q >= r_lo && q < r_hi) ? gap : 0.0f;      // (a gap of 0 leaves the sum as it is)
                }
                tile[r * KS + q] = gap;
            }
        }
        __builtin_amdgcn_wave_barrier();                     // one wave per workgroup: LDS accesses are in order
        if (left > 0) {
            float4* row = reinterpret_cast<float4*>(&tile[lane * KS]);
#pragma unroll 8
            for (int q = 0; q < len / 4; ++q) {
                float4 v = row[q];
                v.x = acc + v.x; v.y = v.x + v.y; v.z = v.y + v.z; v.w = v.z + v.w;
                acc = v.w;
                row[q] = v;
            }
        }
        __builtin_amdgcn_wave_barrier();
        for (u64 rows = m; rows != 0ull; rows &= rows - 1ull) {
            const int r = __ffsll((long long)rows) - 1;
            float* dst = tok_arr + (i64)bcast_u64((u64)at, r);
            const int r_lo = bcast_i(lo, r), r_hi = bcast_i(left, r);
#pragma unroll 2
            for (int q0 = 0; q0 < len; q0 += 64) {
                const int q = q0 + lane;
                if (q >= r_lo && q < r_hi) dst[q] = tile[r * KS + q];
            }
        }
        __builtin_amdgcn_wave_barrier();
        at += K; left -= K; lo = 0; gap_lo = 0;
    }
}

template <int LOG_R>
void launch_tokens(const disco_gen_params& g, i64 n, i64 n_tok, const i64* tok_off, float* tok_arr, hipStream_t stream)
{
    const dim3 grid((unsigned)((n + (1 << LOG_R) - 1) >> LOG_R));
    if (n_tok <= 0xFFFFFFFFll) hipLaunchKernelGGL((k_gen_tokens<LOG_R, false>), grid, dim3(64), 0, stream, g, n, tok_off, tok_arr);
    else hipLaunchKernelGGL((k_gen_tokens<LOG_R, true>), grid, dim3(64), 0, stream, g, n, tok_off, tok_arr);
}

}  // namespace

extern "C" int32_t disco_gen_math_probe(void* out, void* stream_)
{
    if (!out) return DISCO_ERR_NULL;
    if (((uintptr_t)out & 3u) != 0) return DISCO_ERR_SHAPE;
    hipLaunchKernelGGL(k_gen_math_probe, dim3((1u << 23) / 256u), dim3(256), 0, (hipStream_t)stream_, (float*)out);
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

extern "C" int32_t disco_gen_trace(const disco_gen_params* g, disco_trace* tr, int32_t stages, void* stream_)
{
    if (!g || !tr) return DISCO_ERR_NULL;
    hipStream_t stream = (hipStream_t)stream_;
    if (g->n_req < 0 || tr->n_req != g->n_req) return DISCO_ERR_SHAPE;
    if (g->prompt_lo > g->prompt_hi || g->out_lo > g->out_hi || g->out_lo < 1 || g->prompt_lo < 0) return DISCO_ERR_SHAPE;
    if (!(stages & (DISCO_GEN_REQUESTS | DISCO_GEN_TOKENS))) return DISCO_ERR_RANGE;
    auto prob = [](float p) { return p >= 0.0f && p <= 1.0f; };
    if (!(g->prompt_sigma >= 0) || !(g->out_sigma >= 0) || !(g->ttft_sigma >= 0) || !(g->tbt_sigma >= 0) ||
        !(g->gap_sigma >= 0) || !prob(g->ttft_pareto_p) || !prob(g->gap_stall_p) || !prob(g->dev_p) ||
        !(g->ttft_pareto_alpha > 0) || !(g->ttft_pareto_xm > 0) || g->dev_mode < 0 || g->dev_mode > 2 ||
        !(g->dev_a > 0) || !(g->dev_b > 0) || (g->dev_mode != 0 && !(g->dev_pre_ratio > 0)) ||
        (g->dev_mode == 1 && g->dev_b < g->dev_a) || g->gap_stall_hi < g->gap_stall_lo || g->gap_stall_lo < 0)
        return DISCO_ERR_RANGE;
    const i64 n = g->n_req;
    if (stages & DISCO_GEN_REQUESTS) {
        if (!tr->tok_off) return DISCO_ERR_NULL;
        if (n > 0 && (!tr->prompt_len || !tr->output_len || !tr->srv_ttft || !tr->srv_tbt || !tr->dev_pre_spt ||
                      !tr->dev_dec_spt))
            return DISCO_ERR_NULL;
        if (n > 0) {
            unsigned blocks = (unsigned)((n + 255) / 256);
            hipLaunchKernelGGL(k_gen_requests, dim3(blocks), dim3(256), 0, stream, *g, tr->prompt_len, tr->output_len,
                               tr->srv_ttft, tr->srv_tbt, tr->dev_pre_spt, tr->dev_dec_spt);
        }
        {
            i64 per_thread = 4;                              // tiles of 4096 requests while the tile sums fit
            while ((n + per_thread * GO_BLOCK - 1) / (per_thread * GO_BLOCK) > GO_MAX_TILES) per_thread *= 2;
            i64 tiles = (n + per_thread * GO_BLOCK - 1) / (per_thread * GO_BLOCK);
            if (tiles < 1) tiles = 1;
            hipLaunchKernelGGL(k_gen_tile_sums, dim3((unsigned)tiles), dim3(GO_BLOCK), 0, stream, n, per_thread, tr->output_len);
            hipLaunchKernelGGL(k_gen_offsets, dim3((unsigned)tiles), dim3(GO_BLOCK), 0, stream, n, per_thread, tr->output_len,
                               tr->tok_off);
        }
        DISCO_HIP(hipGetLastError());
        i64 total = 0;
        DISCO_HIP(hipMemcpyAsync(&total, tr->tok_off + n, sizeof(i64), hipMemcpyDeviceToHost, stream));
        DISCO_HIP(hipStreamSynchronize(stream));
        tr->n_tok = total;
    }
    if (stages & DISCO_GEN_TOKENS) {
        if (tr->n_tok < 0) return DISCO_ERR_SHAPE;
        if (tr->n_tok > 0) {
            if (!tr->tok_arr || !tr->tok_off) return DISCO_ERR_NULL;
            // requests per wave: 16 where that leaves two waves per SIMD, fewer on smaller batches, so that their tokens are
            // not a few waves' serial work (20 000 requests: 106 us with 4 per wave, 226 with 1; 2000: 68 with 1)
            if (n >= 2048 * 16) launch_tokens<4>(*g, n, tr->n_tok, tr->tok_off, tr->tok_arr, stream);
            else if (n >= 2048 * 4) launch_tokens<2>(*g, n, tr->n_tok, tr->tok_off, tr->tok_arr, stream);
            else launch_tokens<0>(*g, n, tr->n_tok, tr->tok_off, tr->tok_arr, stream);
            DISCO_HIP(hipGetLastError());
        }
    }
    return DISCO_OK;
}
