// Opt-in validation of a trace before it is evaluated (recorded traces enter through disco_ingest_trace; the
// evaluation kernels trust the arrays they are given: a token offset that does not match the output length
// makes them read outside the token array).  One pass over the requests, then -- if the offsets are sound, so
// that the pass cannot leave the token array, which the second kernel reads from the first one's findings -- one
// pass over the tokens.
#include <math.h>

#include "disco_common.h"
#include "disco_device.h"

namespace {

enum { BAD_CSR = 1, BAD_RANGE = 2 };

struct ValidateFound { unsigned flag, pad; u64 falls; };        // falls: decreases inside requests (token pass)

constexpr int VD_BLOCK = 256;
constexpr int VD_WAVES = VD_BLOCK / 64;

__device__ __forceinline__ bool bad_time(float x) { return !(x >= 0.0f) || x == INFINITY; }      // negative, NaN or infinite

// Requests: lengths, times and rates in range; offsets start at 0, advance by the output length and, with a token
// array, end at n_tok.
__global__ __launch_bounds__(VD_BLOCK) void k_validate_requests(TraceView tr, i64 n_tok, const i64* __restrict__ tok_off,
                                                                 unsigned* __restrict__ flag)
{
    unsigned bad = 0u;
    for (i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x; i < tr.n_req; i += (i64)gridDim.x * blockDim.x) {
        const int l = tr.l[i], n = tr.n[i];
        if (l < 0 || n < 1) bad |= BAD_RANGE;
        if (bad_time(tr.s[i])) bad |= BAD_RANGE;
        if (tr.tbt && bad_time(tr.tbt[i])) bad |= BAD_RANGE;
        if (tr.k && bad_time(tr.k[i])) bad |= BAD_RANGE;
        if (tr.g && bad_time(tr.g[i])) bad |= BAD_RANGE;
        if (tok_off) {
            const i64 a = tok_off[i], b = tok_off[i + 1];
            if (a < 0 || b < a || b - a != (i64)n) bad |= BAD_CSR;
            if (i == 0 && a != 0) bad |= BAD_CSR;
            if (tr.arr && (b > n_tok || (i == tr.n_req - 1 && b != n_tok))) bad |= BAD_CSR;      // (n_tok counts a token array)
        }
    }
    if (__ballot(bad != 0u) != 0ull) {
        const unsigned all = (__ballot((bad & BAD_CSR) != 0u) ? (unsigned)BAD_CSR : 0u) |
                             (__ballot((bad & BAD_RANGE) != 0u) ? (unsigned)BAD_RANGE : 0u);
        if ((threadIdx.x & 63) == 0) atomicOr(flag, all);
    }
}

// Tokens: arrival offsets start at 0, never decrease inside a request, are finite.  Returns at once where the
// requests' pass has found the offsets unsound, so it cannot leave the token array.
//
// The pass does not go by requests: the array is read once as it lies, in vectors of four, and counted are the
// places where a value is below the one in front of it.  Every first token is 0 and no value is negative, so such a
// place at a request's first token is one whose predecessor is above 0: these are counted from the offsets, and the
// decreases inside requests are what remains.  (A NaN takes part in no decrease but is out of range by itself.)
// Bound by device memory: 491 M tokens, 2.0 GB, in 336 us = 5.8 TB/s; a wave per request with 4-byte loads of a token
// and its predecessor took 890 us.
constexpr int VT_STEP = 4;                       // vectors per lane and step: loads in flight

__global__ __launch_bounds__(VD_BLOCK) void k_validate_tokens(i64 n_req, i64 n_tok, const i64* __restrict__ tok_off,
                                                              const float* __restrict__ arr, ValidateFound* __restrict__ found)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    if (found->flag & BAD_CSR) return;
    const i64 tid = (i64)blockIdx.x * VD_BLOCK + threadIdx.x, nthr = (i64)gridDim.x * VD_BLOCK;
    const int lane = threadIdx.x & 63;
    bool bad = false;
    u64 falls = 0;                               // decreases of the array less those in front of a first token
    for (i64 i = tid; i < n_req; i += nthr) {
        const i64 a = tok_off[i], b = tok_off[i + 1];
        if (b <= a) continue;
        if (arr[a] != 0.0f) bad = true;
        if (a > 0 && arr[a - 1] > arr[a]) falls -= 1;
    }
    // up to three tokens in front of the first aligned vector and behind the last one, then whole vectors
    const i64 head = min((i64)((16u - ((uintptr_t)arr & 15u)) & 15u) / 4, n_tok);
    const i64 nvec = (n_tok - head) >> 2;
    const i64 ends = n_tok - 4 * nvec;
    if (tid < ends) {
        const i64 j = tid < head ? tid : tid + 4 * nvec;
        if (bad_time(arr[j])) bad = true;
        if (j > 0 && arr[j - 1] > arr[j]) falls += 1;
    }
    // a wave takes VT_STEP x 64 consecutive vectors at a time
    const f4* vec = reinterpret_cast<const f4*>(arr + head);
    const i64 wave = tid >> 6, nwaves = nthr >> 6;
    for (i64 base = wave * (64 * VT_STEP); base < nvec; base += nwaves * (64 * VT_STEP)) {
        f4 x[VT_STEP];
#pragma unroll
        for (int q = 0; q < VT_STEP; ++q) {
            const i64 k = base + 64 * q + lane;
            if (k < nvec) x[q] = __builtin_nontemporal_load(vec + k);
        }
        // the value in front of the step's first one (none in front of the array)
        const i64 at = head + 4 * base;
        float before = at > 0 ? arr[at - 1] : 0.0f;
        unsigned n = 0;
#pragma unroll
        for (int q = 0; q < VT_STEP; ++q) {
            const bool in = base + 64 * q + lane < nvec;
            const float up = __shfl_up(x[q].w, 1, 64);
            const float prev = lane == 0 ? before : up;
            before = bcast_f(x[q].w, 63);
            if (in) {
                bad = bad || bad_time(x[q].x) || bad_time(x[q].y) || bad_time(x[q].z) || bad_time(x[q].w);
                n += (prev > x[q].x ? 1u : 0u) + (x[q].x > x[q].y ? 1u : 0u) + (x[q].y > x[q].z ? 1u : 0u) + (x[q].z > x[q].w ? 1u : 0u);
            }
        }
        falls += n;
    }
    if (__ballot(bad) != 0ull && lane == 0) atomicOr(&found->flag, (unsigned)BAD_RANGE);
    falls = wave_sum_u64(falls);
    __shared__ u64 sfalls[VD_WAVES];
    if (lane == 0) sfalls[threadIdx.x >> 6] = falls;
    __syncthreads();
    if (threadIdx.x == 0) {
        u64 f = 0;
        for (int w = 0; w < VD_WAVES; ++w) f += sfalls[w];
        if (f) atomicAdd((unsigned long long*)&found->falls, (unsigned long long)f);
    }
}

}  // namespace

extern "C" int32_t disco_validate_trace(const disco_trace* t, int32_t check_tokens, void* ws_, size_t ws_bytes, void* stream_)
{
    if (!t) return DISCO_ERR_NULL;
    if (t->n_req < 0 || t->n_tok < 0) return DISCO_ERR_SHAPE;
    if (t->n_req > 0 && (!t->prompt_len || !t->output_len || !t->srv_ttft)) return DISCO_ERR_NULL;
    if ((t->tok_arr != nullptr) && !t->tok_off) return DISCO_ERR_CSR;
    if (!ws_ || ws_bytes < 256 || ((uintptr_t)ws_ & 255u) != 0) return DISCO_ERR_WORKSPACE;
    if (!(t->dev_ttft_c >= 0.0f) || (!t->dev_pre_spt && !(t->dev_pre_spt_s >= 0.0f)) || (!t->dev_dec_spt && !(t->dev_dec_spt_s >= 0.0f)))
        return DISCO_ERR_RANGE;
    if (t->n_req == 0) return t->n_tok == 0 || !t->tok_off ? DISCO_OK : DISCO_ERR_CSR;
    hipStream_t stream = (hipStream_t)stream_;
    ValidateFound* dev = (ValidateFound*)ws_;
    TraceView v;
    v.n_req = t->n_req;
    v.l = t->prompt_len; v.n = t->output_len; v.s = t->srv_ttft; v.tbt = t->srv_tbt;
    v.k = t->dev_pre_spt; v.g = t->dev_dec_spt; v.off = t->tok_off; v.arr = t->tok_arr;
    v.k_s = t->dev_pre_spt_s; v.g_s = t->dev_dec_spt_s; v.c = t->dev_ttft_c;
    ValidateFound found{0u, 0u, 0ull};
    DISCO_HIP(hipMemcpyAsync(dev, &found, sizeof(found), hipMemcpyHostToDevice, stream));
    i64 b = (t->n_req + VD_BLOCK - 1) / VD_BLOCK;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(k_validate_requests, dim3((unsigned)b), dim3(VD_BLOCK), 0, stream, v, t->n_tok, t->tok_off, &dev->flag);
    DISCO_HIP(hipGetLastError());
    if (check_tokens && t->tok_arr) {
        i64 units = (t->n_tok + 4 * VT_STEP - 1) / (4 * VT_STEP);        // threads for the tokens, at least those of the requests
        if (units < t->n_req) units = t->n_req;
        i64 wb = (units + VD_BLOCK - 1) / VD_BLOCK;
        if (wb > 2048) wb = 2048;
        hipLaunchKernelGGL(k_validate_tokens, dim3((unsigned)wb), dim3(VD_BLOCK), 0, stream, t->n_req, t->n_tok, t->tok_off,
                           t->tok_arr, dev);
        DISCO_HIP(hipGetLastError());
    }
    DISCO_HIP(hipMemcpyAsync(&found, dev, sizeof(found), hipMemcpyDeviceToHost, stream));
    DISCO_HIP(hipStreamSynchronize(stream));
    if (found.flag & BAD_CSR) return DISCO_ERR_CSR;
    return (found.flag & BAD_RANGE) || found.falls ? DISCO_ERR_RANGE : DISCO_OK;
}
