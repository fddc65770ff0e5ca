// Recorded traces (Sec. 5.1: the evaluation is driven by traces of production
// services and on-device profiles) and the log-normal fit of the scalability
// study (Sec. 5.3: prompt length and server TTFT laws fitted by the mean and
// standard deviation of the logarithm).
//
//   k_ingest        wall-clock timestamps -> server TTFT, output length and
//                   token arrival offsets relative to the request's first token:
//                   a wave takes the tokens of one request after the other, its
//                   lanes stride them; a difference is taken in fp64 and rounded
//                   once to fp32.  Streams 12 B per token (8 read, 4 written).
//   k_fit_sum / k_fit_final   mean of ln x, then mean squared deviation, each a
//                   grid-stride pass with per-workgroup partial sums folded in a
//                   fixed order by one workgroup (the result does not depend on
//                   the order in which workgroups finish).
#include <math.h>
#include <string.h>

#include "disco_launch.h"
#include "disco_device.h"

namespace {

constexpr int IG_BLOCK = 256;
constexpr int IG_WAVES = IG_BLOCK / 64;
constexpr int FIT_BLOCK = 256;
constexpr int FIT_MAX_BLOCKS = 1024;

// A wave owns R consecutive requests (their tokens are one contiguous stretch).  Lane r < R takes request r: its
// offsets, first timestamp and per-request outputs are loaded and stored for all R at once, so the chain
// offset -> first timestamp -> tokens is waited for once per R requests and not per request.  The tokens then pass in
// steps of 512 per wave, all loads of a step issued before its first store.  Neither side is read again here, so the
// stores go past the caches, and so do the loads (PAST) where the timestamps do not fit the last level anyway.  Bound by
// device memory: 491 M tokens of 10^6 requests, 5.9 GB, in 1185 us = 5.0 TB/s (a wave per request with one load in flight:
// 1312 us; an elementwise fp32 -> fp64 conversion of that size runs at 5.1 TB/s).
template <int R, bool PAIR, bool PAST>
__global__ __launch_bounds__(IG_BLOCK) void k_ingest(i64 n_req, const double* __restrict__ t_send,
                                                     const double* __restrict__ t_token, const i64* __restrict__ off,
                                                     float* __restrict__ srv_ttft, int32_t* __restrict__ output_len,
                                                     float* __restrict__ tok_arr)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    constexpr int STEP = 4;                             // 16-byte loads in flight per lane
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const i64 ngroups = (n_req + R - 1) / R;
    for (i64 gr = (i64)blockIdx.x * IG_WAVES + wave; gr < ngroups; gr += (i64)gridDim.x * IG_WAVES) {
        const i64 i = gr * R + lane;
        const bool v = lane < R && i < n_req;
        const i64 oa = v ? off[i] : 0, ob = v ? off[i + 1] : 0;
        const double fv = ob > oa ? t_token[oa] : 0.0;
        if (v) {
            output_len[i] = ob > oa ? (int32_t)(ob - oa) : 0;
            srv_ttft[i] = ob > oa ? (float)(fv - t_send[i]) : NAN;      // a request without tokens has no first token
        }
#pragma unroll 1
        for (int r = 0; r < R; ++r) {
            const i64 a = (i64)bcast_u64((u64)oa, r), b = (i64)bcast_u64((u64)ob, r);
            if (b <= a) continue;
            const double first = __longlong_as_double((long long)bcast_u64((u64)__double_as_longlong(fv), r));
            if (PAIR) {
                // two timestamps per lane and load (16-byte loads, 8-byte stores) from the first even token on
                const i64 a2 = (a + 1) & ~(i64)1;
                if (lane == 0 && a2 > a) tok_arr[a] = 0.0f;
                if (lane == 1 && (b & 1) && b > a2) tok_arr[b - 1] = (float)(t_token[b - 1] - first);
                const i64 pairs = (b - a2) >> 1;        // (b < a2 only for a single odd token: none)
                const d2* src = reinterpret_cast<const d2*>(t_token + a2);
                f2* dst = reinterpret_cast<f2*>(tok_arr + a2);
                for (i64 j = lane; j < pairs; j += 64 * STEP) {
                    d2 x[STEP];
#pragma unroll
                    for (int q = 0; q < STEP; ++q)
                        if (j + 64 * q < pairs) x[q] = PAST ? __builtin_nontemporal_load(src + j + 64 * q) : src[j + 64 * q];
#pragma unroll
                    for (int q = 0; q < STEP; ++q)
                        if (j + 64 * q < pairs) {
                            f2 o;
                            o.x = (float)(x[q].x - first); o.y = (float)(x[q].y - first);
                            __builtin_nontemporal_store(o, dst + j + 64 * q);
                        }
                }
            } else {
                constexpr int ONES = R >= 8 ? 1 : STEP;  // (many short requests per wave: a step covers most of them)
                for (i64 j = a + lane; j < b; j += 64 * ONES) {
                    double x[ONES];
#pragma unroll
                    for (int q = 0; q < ONES; ++q)
                        if (j + 64 * q < b) x[q] = t_token[j + 64 * q];
#pragma unroll
                    for (int q = 0; q < ONES; ++q)
                        if (j + 64 * q < b) tok_arr[j + 64 * q] = (float)(x[q] - first);
                }
            }
        }
    }
}

struct FitPartial { double sum; u64 used; };

__device__ __forceinline__ double value_of(const void* x, int kind, i64 i)
{
    return kind == 0 ? (double)((const int32_t*)x)[i] : (double)((const float*)x)[i];
}

// pass 0: sum of ln x; pass 1: sum of (ln x - mu)^2 with mu from pass 0.
__global__ __launch_bounds__(FIT_BLOCK) void k_fit_sum(const void* __restrict__ x, int kind, i64 n, int pass,
                                                       const disco_lognormal_fit* fit, FitPartial* part)
{
    __shared__ double ssum[FIT_BLOCK / 64];
    __shared__ u64 sused[FIT_BLOCK / 64];
    const double mu = pass ? fit->mu : 0.0;
    double sum = 0.0;
    u64 used = 0;
    for (i64 i = (i64)blockIdx.x * FIT_BLOCK + threadIdx.x; i < n; i += (i64)gridDim.x * FIT_BLOCK) {
        const double v = value_of(x, kind, i);
        if (v > 0.0) {                                  // NaN and non-positive values have no logarithm
            const double lv = log(v);
            const double dv = lv - mu;
            sum += pass ? dv * dv : lv;
            used += 1;
        }
    }
    sum = wave_sum_f64(sum);
    used = wave_sum_u64(used);
    if ((threadIdx.x & 63) == 0) { ssum[threadIdx.x >> 6] = sum; sused[threadIdx.x >> 6] = used; }
    __syncthreads();
    if (threadIdx.x == 0) {
        FitPartial p{0.0, 0};
        for (int w = 0; w < FIT_BLOCK / 64; ++w) { p.sum += ssum[w]; p.used += sused[w]; }
        part[blockIdx.x] = p;
    }
}

__global__ __launch_bounds__(64) void k_fit_final(int nblocks, i64 n, int pass, const FitPartial* part, disco_lognormal_fit* fit)
{
    double sum = 0.0;
    u64 used = 0;
    for (int b = threadIdx.x; b < nblocks; b += 64) { sum += part[b].sum; used += part[b].used; }
    sum = wave_sum_f64(sum);
    used = wave_sum_u64(used);
    if (threadIdx.x != 0) return;
    if (pass == 0) {
        fit->mu = used ? sum / (double)used : NAN;
        fit->sigma = NAN;
        fit->n_used = (i64)used;
        fit->n_skipped = n - (i64)used;
    } else {
        fit->sigma = used ? sqrt(sum / (double)used) : NAN;
    }
}

// On-device configurations of Sec. 5.1: prefill / decode speed in tokens per second.
const double kProfiles[3][2] = {{31.32, 13.93}, {51.80, 20.14}, {79.90, 21.47}};
const char* const kProfileNames[3] = {"Pixel 7 Pro / Bloom 1.1B", "Pixel 7 Pro / Bloom 560M", "Xiaomi 14 / Qwen 1.5 0.5B"};

}  // namespace

template <int R>
static void launch_ingest(i64 n_req, i64 n_tok, const double* t_send, const double* t_token, const i64* off, float* srv_ttft,
                          int32_t* output_len, float* tok_arr, hipStream_t stream)
{
    i64 b = (n_req + R * IG_WAVES - 1) / (R * IG_WAVES);
    if (b < 1) b = 1;
    if (b > 8192) b = 8192;
    const bool pair = (((uintptr_t)t_token) & 15u) == 0 && (((uintptr_t)tok_arr) & 7u) == 0;
    // 256 MB of timestamps: the last-level cache.  9.9 M tokens 22 us with loads through it and 24 past it, 69 M tokens 163 and 153
    const bool past = n_tok > (i64)(256 << 20) / 8;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)b), dim3(IG_BLOCK), 0, stream, n_req, t_send, t_token, off, srv_ttft, output_len, tok_arr);
    };
    if (!pair) go(k_ingest<R, false, false>);
    else if (past) go(k_ingest<R, true, true>);
    else go(k_ingest<R, true, false>);
}

void disco_launch_ingest(i64 n_req, i64 n_tok, const double* t_send, const double* t_token, const i64* off, float* srv_ttft,
                         int32_t* output_len, float* tok_arr, hipStream_t stream)
{
    // The shorter the requests, the more of them share a wave (the wait for offsets and first timestamps is a request's own
    // cost), as long as the waves keep half the chip's slots busy.  With 1, 2, 8 and 16 per wave: 10^6 requests of 492 tokens
    // 1185, 1211, 1227 and 1241 us, of 215 tokens 522, 476, 498 and 516, of 71 tokens 268 with 2 and 211 with 8, of 34 tokens 333, 232, 177 and 174, of 2 tokens 207, 134,
    // 91 and 83; 140 000 of 34 tokens 39, 28 and 24 us with 1, 2 and 8.
    const i64 mean = n_req > 0 ? n_tok / n_req : 0;
    if (mean < 24 && n_req >= 16 * 4096) launch_ingest<16>(n_req, n_tok, t_send, t_token, off, srv_ttft, output_len, tok_arr, stream);
    else if (mean < 128 && n_req >= 8 * 4096) launch_ingest<8>(n_req, n_tok, t_send, t_token, off, srv_ttft, output_len, tok_arr, stream);
    else if (mean < 256 && n_req >= 2 * 4096) launch_ingest<2>(n_req, n_tok, t_send, t_token, off, srv_ttft, output_len, tok_arr, stream);
    else launch_ingest<1>(n_req, n_tok, t_send, t_token, off, srv_ttft, output_len, tok_arr, stream);
}

size_t disco_fit_scratch_bytes(void) { return sizeof(FitPartial) * FIT_MAX_BLOCKS; }

void disco_launch_fit(const void* x, int kind, i64 n, disco_lognormal_fit* fit, void* scratch, hipStream_t stream)
{
    i64 b = (n + FIT_BLOCK - 1) / FIT_BLOCK;
    if (b < 1) b = 1;
    if (b > FIT_MAX_BLOCKS) b = FIT_MAX_BLOCKS;
    FitPartial* part = (FitPartial*)scratch;
    for (int pass = 0; pass < 2; ++pass) {
        hipLaunchKernelGGL(k_fit_sum, dim3((unsigned)b), dim3(FIT_BLOCK), 0, stream, x, kind, n, pass, fit, part);
        hipLaunchKernelGGL(k_fit_final, dim3(1), dim3(64), 0, stream, (int)b, n, pass, part, fit);
    }
}

extern "C" int32_t disco_device_profile(int32_t index, disco_device_preset* out)
{
    if (!out) return DISCO_ERR_NULL;
    if (index < 0 || index >= 3) return DISCO_ERR_RANGE;
    memset(out, 0, sizeof(*out));
    out->prefill_tok_per_s = kProfiles[index][0];
    out->decode_tok_per_s = kProfiles[index][1];
    out->dev_pre_spt_s = (float)(1.0 / kProfiles[index][0]);
    out->dev_dec_spt_s = (float)(1.0 / kProfiles[index][1]);
    out->dev_ttft_c = 0.0f;
    strncpy(out->name, kProfileNames[index], sizeof(out->name) - 1);
    return DISCO_OK;
}
