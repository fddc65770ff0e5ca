// Evaluation kernels and entry points of libdisco: dispatch, token timelines
// with lag-triggered migration, order-statistic selection, budget search.
//
// Work decomposition
//   dispatch-type passes: a wave holds up to 64 policy columns in its lanes
//     and walks the requests in batches; per-column totals stay in registers
//     until the end of the kernel and are then added into device-wide totals.
//   timeline passes: one wave per request, four tokens per lane, 256-token
//     chunks with a carried running maximum.
//   a sequence of passes (budget search, radix selection) advances its state
//     on the device, so it needs no host round trip.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <mutex>

#include "disco_final.h"
#include "disco_launch.h"
#include "disco_stage.h"
#include "disco_state.h"

namespace {

__global__ __launch_bounds__(STAGE_THREADS) void k_store_policies(PolTable t, int P, disco_policy* dst, unsigned* tickets, u64* totals,
                                                                  SelInit si)
{
    stage_table(t.p, P, dst, tickets, totals, si, (int)blockIdx.x, (int)gridDim.x);
}

// (dst may be src: the selection's workgroup then reads what the first one writes back unchanged)
__global__ __launch_bounds__(STAGE_THREADS) void k_copy_policies(const disco_policy* src, int P, disco_policy* dst, unsigned* tickets, u64* totals,
                                                                 SelInit si)
{
    stage_table(src, P, dst, tickets, totals, si, (int)blockIdx.x, (int)gridDim.x);
}

// ------------------------------------------------------------ final stats --

__global__ __launch_bounds__(FINAL_THREADS) void k_stats_final(FinalArgs f)
{
    __shared__ FinalLds lds;
    stats_final((int)blockIdx.x, f, lds, f.tbt ? &f.S->tl.plan[DISCO_TBT_MAX_PASS] : nullptr);
}

// Mean over the runs of a group of columns: floating-point fields in fp64, summed in run order; integer
// totals summed; ranks taken from the first run.
__global__ void k_average_runs(const disco_stats* __restrict__ in, int groups, int runs, disco_stats* __restrict__ out)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= groups) return;
    const disco_stats* r = in + (size_t)g * runs;
    disco_stats o;
    memset(&o, 0, sizeof(o));
    double d[7] = {0, 0, 0, 0, 0, 0, 0}, q[2 * DISCO_MAX_Q];
    for (int k = 0; k < 2 * DISCO_MAX_Q; ++k) q[k] = 0.0;
    for (int k = 0; k < DISCO_MAX_Q; ++k) { o.ttft_rank[k] = r[0].ttft_rank[k]; o.tbt_rank[k] = r[0].tbt_rank[k]; }
    for (int j = 0; j < runs; ++j) {
        const disco_stats s = r[j];
        d[0] += s.mean_ttft; d[1] += s.mean_tbt; d[2] += s.server_cost; d[3] += s.device_energy;
        d[4] += s.device_cost; d[5] += s.total_cost; d[6] += s.mean_delay_num;
        o.s_pre += s.s_pre; o.s_dec += s.s_dec; o.d_pre += s.d_pre; o.d_dec += s.d_dec;
        o.n_req += s.n_req; o.tbt_count += s.tbt_count; o.n_migrated += s.n_migrated;
        o.n_dev_started += s.n_dev_started; o.n_dev_win += s.n_dev_win;
        for (int k = 0; k < DISCO_MAX_Q; ++k) { q[k] += (double)s.ttft_q[k]; q[DISCO_MAX_Q + k] += (double)s.tbt_q[k]; }
    }
    const double n = (double)runs;
    o.mean_ttft = d[0] / n; o.mean_tbt = d[1] / n; o.server_cost = d[2] / n; o.device_energy = d[3] / n;
    o.device_cost = d[4] / n; o.total_cost = d[5] / n; o.mean_delay_num = d[6] / n;
    for (int k = 0; k < DISCO_MAX_Q; ++k) { o.ttft_q[k] = (float)(q[k] / n); o.tbt_q[k] = (float)(q[DISCO_MAX_Q + k] / n); }
    out[g] = o;
}

// ----------------------------------------------------------- search setup --

// Brackets of the searches; `pol` holds their templates on entry.  They move to `templ` and `pol` gets the candidate
// columns of the first bisection pass (2^depth - 1 per search).
__global__ void k_search_init(SpecTable t, int n, SearchState* st, disco_policy* pol, disco_policy* templ, int depth)
{
    const int c = threadIdx.x;
    SearchState s;
    disco_policy p;
    if (c < n) {
        s = t.s[c];
        p = pol[c];
        if (s.which_param == DISCO_PARAM_L_TH) { s.lo = (int)s.lo; s.hi = (int)s.hi; }
        else { s.lo = (double)(float)s.lo; s.hi = (double)(float)s.hi; }
        s.step = 0;
        st[c] = s;
    }
    __syncthreads();                        // all templates have been read
    if (c >= n) return;
    templ[c] = p;
    search_write_candidates(s, p, &pol[c * ((1 << depth) - 1)], depth);
}

// ------------------------------------------------------------- host side --

thread_local char g_hip_error[256] = "";

TraceView view_of(const disco_trace* t)
{
    TraceView v;
    v.n_req = t->n_req;
    v.l = t->prompt_len; v.n = t->output_len; v.s = t->srv_ttft; v.tbt = t->srv_tbt;
    v.k = t->dev_pre_spt; v.g = t->dev_dec_spt;
    v.off = t->tok_arr ? t->tok_off : nullptr;
    v.arr = t->tok_arr;
    v.k_s = t->dev_pre_spt_s; v.g_s = t->dev_dec_spt_s; v.c = t->dev_ttft_c;
    return v;
}

int check_trace(const disco_trace* t)
{
    if (!t) return DISCO_ERR_NULL;
    if (t->n_req < 0 || t->n_tok < 0) return DISCO_ERR_SHAPE;
    if (t->n_req > 0 && (!t->prompt_len || !t->output_len || !t->srv_ttft)) return DISCO_ERR_NULL;
    if ((t->tok_arr != nullptr) != (t->tok_off != nullptr) && t->tok_arr) return DISCO_ERR_CSR;
    return DISCO_OK;
}

int check_policies(const disco_policy* pol, int P)
{
    if (!pol) return DISCO_ERR_NULL;
    if (P < 1 || P > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;
    for (int j = 0; j < P; ++j) {
        if (pol[j].mode < DISCO_MODE_SERVER_CONSTRAINED || pol[j].mode > DISCO_MODE_STOCH_DEVICE) return DISCO_ERR_RANGE;
        if (pol[j].mode >= DISCO_MODE_STOCH_SERVER && !(pol[j].beta >= 0.0f && pol[j].beta <= 1.0f))
            return DISCO_ERR_RANGE;                         // the routing probability of a stochastic baseline
        if (pol[j].mig_mode != DISCO_MIG_NONE && pol[j].mig_mode != DISCO_MIG_LAG && pol[j].mig_mode != DISCO_MIG_BUFFER)
            return DISCO_ERR_RANGE;
        if (pol[j].w_mid != pol[j].w_mid || pol[j].beta != pol[j].beta || pol[j].w_tail != pol[j].w_tail)
            return DISCO_ERR_RANGE;
    }
    return DISCO_OK;
}

int check_ws(void* ws, size_t ws_bytes, int P)
{
    if (!ws) return DISCO_ERR_WORKSPACE;
    if (ws_bytes < disco_ws_layout(P).total) return DISCO_ERR_WORKSPACE;
    if (((uintptr_t)ws & 255u) != 0) return DISCO_ERR_WORKSPACE;
    return DISCO_OK;
}

// Prices of the buffer hand-off's cost test from the unified cost rates (Sec. 4.1): a server source saves
// cs_dec - lambda e_dec per token and pays lambda e_pre per re-prefilled token; a device source the mirror image.
// Without rates nothing is ever saved (no hand-off).
BufCostArgs buffer_prices(const disco_cost_params* c)
{
    BufCostArgs b{0.0, 0.0, 0.0, 0.0};
    if (c) {
        const double dev_dec = c->lambda * c->e_dec, dev_pre = c->lambda * c->e_pre;
        b.dc_srv = c->cs_dec - dev_dec; b.cp_srv = dev_pre;
        b.dc_dev = dev_dec - c->cs_dec; b.cp_dev = c->cs_pre;
    }
    return b;
}

bool is_device_pointer(const void* p)
{
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
        (void)hipGetLastError();          // ordinary host memory is not known to the runtime
        return false;
    }
    return attr.type == hipMemoryTypeDevice;
}

// Host tables are validated and travel as a kernel argument; device tables
// (e.g. the pol_out of a budget search) are copied on the device, unvalidated.
int stage_policies(const disco_policy* pol, int P, char* ws, const WsLayout& L, hipStream_t stream, const SelInit* sel = nullptr)
{
    SelInit si;
    memset(&si, 0, sizeof(si));
    if (sel) si = *sel;
    const unsigned workgroups = !sel ? 1u : (sel->with_tbt ? 3u + STAGE_CLEAR : 2u);
    if (!pol) return DISCO_ERR_NULL;
    if (P < 1 || P > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;
    if (is_device_pointer(pol)) {
        hipLaunchKernelGGL(k_copy_policies, dim3(workgroups), dim3(STAGE_THREADS), 0, stream, pol, P, (disco_policy*)(ws + L.pol),
                           (unsigned*)(ws + L.ticket), (u64*)(ws + L.part), si);
        return DISCO_OK;
    }
    int rc = check_policies(pol, P);
    if (rc) return rc;
    PolTable t;
    memset(&t, 0, sizeof(t));
    memcpy(t.p, pol, sizeof(disco_policy) * (size_t)P);
    hipLaunchKernelGGL(k_store_policies, dim3(workgroups), dim3(STAGE_THREADS), 0, stream, t, P, (disco_policy*)(ws + L.pol),
                       (unsigned*)(ws + L.ticket), (u64*)(ws + L.part), si);
    return DISCO_OK;
}

// The table of a call as the kernels of small traces take it: `host` filled in and validated, or *device set.
int small_table(const disco_policy* pol, int P, PolTable& host, const disco_policy** device)
{
    memset(&host, 0, sizeof(host));
    *device = nullptr;
    if (is_device_pointer(pol)) { *device = pol; return DISCO_OK; }
    const int rc = check_policies(pol, P);
    if (rc == DISCO_OK) memcpy(host.p, pol, sizeof(disco_policy) * (size_t)P);
    return rc;
}

// Dispatch totals of every column and, if asked, the per-pair outputs; `part`: device-wide totals, `ws + L.*`: scratch.
int eval_dispatch(const TraceView& v, const disco_policy* pol, int P, const disco_pair_out* out, disco_accum* acc, char* ws,
                  const WsLayout& L, hipStream_t stream)
{
    uint8_t* decision = out && v.n_req > 0 ? out->decision : nullptr;
    float* ttft = out && v.n_req > 0 ? out->ttft : nullptr;
    if (disco_small(v.n_req)) {
        PolTable t;
        const disco_policy* device;
        const int rc = small_table(pol, P, t, &device);
        if (rc) return rc;
        disco_launch_small_dispatch(v, t, device, P, acc, decision, ttft, stream);
    } else {
        const int rc = stage_policies(pol, P, ws, L, stream);        // also puts the flag words and the totals at their identity
        if (rc) return rc;
        DispFin fin;
        memset(&fin, 0, sizeof(fin));
        fin.kind = 0;
        fin.need = 2;
        fin.acc = acc;
        disco_launch_dispatch_acc(v, (const disco_policy*)(ws + L.pol), P, (u64*)(ws + L.part), fin, stream, decision, ttft);
    }
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

}  // namespace

void disco_set_hip_error(hipError_t e, const char* what)
{
    snprintf(g_hip_error, sizeof(g_hip_error), "%s: %s", what, hipGetErrorString(e));
}

WsLayout disco_ws_layout(int32_t P)
{
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    WsLayout L;
    size_t o = 0;
    L.pol = o; o += up(sizeof(disco_policy) * DISCO_MAX_COLS);
    L.ticket = o; o += up(sizeof(unsigned) * 64);
    L.search = o; o += up(sizeof(SearchState) * DISCO_MAX_COLS);
    L.sel = o; o += up(sizeof(SelState));
    L.ghist = o; o += up(sizeof(unsigned) * DISCO_GHIST_WORDS);
    L.part = o;
    (void)P;
    o += up((size_t)DISCO_MAX_BLOCKS * 64 * 64);     // workgroups x columns x 64-byte partial
    L.ppcnt = o; o += up(sizeof(unsigned) * DISCO_MAX_CLS * (DISCO_PP_NMAX + 1));
    L.dhist = o; o += up(sizeof(unsigned) * DISCO_MAX_COLS * DISCO_DELAY_BINS);
    L.templ = o; o += up(sizeof(disco_policy) * DISCO_MAX_COLS);
    L.wcount = o; o += up(sizeof(unsigned) * 1024);
    L.slices = o; o += up((size_t)256 * (2 * DISCO_MAX_COLS + 2) * 256 * sizeof(unsigned));   // 256 workgroups x rows x bins
    L.total = o;
    return L;
}

// The fixed regions, then one byte and 16 bytes per request (see disco_ws_bytes_region).
extern "C" size_t disco_workspace_bytes(int64_t n_req, int32_t P)
{
    return disco_ws_full_bytes(disco_ws_layout(P), n_req);
}

extern "C" const char* disco_strerror(int32_t code)
{
    switch (code) {
    case DISCO_OK: return "ok";
    case DISCO_ERR_NULL: return "a required pointer is NULL";
    case DISCO_ERR_SHAPE: return "negative or inconsistent sizes";
    case DISCO_ERR_RANGE: return "parameter out of range";
    case DISCO_ERR_CSR: return "token arrays missing or inconsistent";
    case DISCO_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case DISCO_ERR_HIP: return "HIP runtime error";
    default: return "unknown error code";
    }
}

extern "C" const char* disco_last_hip_error(void) { return g_hip_error; }

// Alg. 1: the policy type from the unified cost rates (device costs in money = lambda x energy per token).
extern "C" int32_t disco_policy_type(const disco_cost_params* c, int32_t* mode)
{
    if (!c || !mode) return DISCO_ERR_NULL;
    const double cd_p = c->lambda * c->e_pre, cd_d = c->lambda * c->e_dec;
    const double dev_min = cd_p < cd_d ? cd_p : cd_d, srv_max = c->cs_pre > c->cs_dec ? c->cs_pre : c->cs_dec;
    if (dev_min != dev_min || srv_max != srv_max || c->cs_pre != c->cs_pre || c->cs_dec != c->cs_dec) return DISCO_ERR_RANGE;
    *mode = dev_min > srv_max ? DISCO_MODE_DEVICE_CONSTRAINED : DISCO_MODE_SERVER_CONSTRAINED;
    return DISCO_OK;
}

static int g_grid_divisor = 1;
int disco_grid_divisor() { return g_grid_divisor; }
extern "C" int32_t disco_set_grid_divisor(int32_t d)
{
    if (d < 1 || d > 1024) return DISCO_ERR_RANGE;
    g_grid_divisor = d;
    return DISCO_OK;
}
extern "C" int32_t disco_version(void) { return 100; }

extern "C" int32_t disco_eval_dispatch(const disco_trace* trace, const disco_policy* pol, int32_t P,
                                       const disco_pair_out* out, disco_accum* acc, void* ws_, size_t ws_bytes,
                                       void* stream_)
{
    int rc = check_trace(trace);
    if (rc) return rc;
    if (!pol || !acc) return DISCO_ERR_NULL;
    if (P < 1 || P > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;
    rc = check_ws(ws_, ws_bytes, P);
    if (rc) return rc;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)ws_;
    const WsLayout L = disco_ws_layout(P);
    return eval_dispatch(view_of(trace), pol, P, out, acc, ws, L, stream);
}

// ---------------------------------------------------- fixed scratch area --
// Scratch of disco_eval_dispatch_static: the three workspace regions a dispatch pass touches (staged policy
// table, flag words, device-wide totals), in device memory that belongs to the library's code object.  Every
// GPU holds its own copy at its own address, which host code obtains once per device from the runtime; the
// array's name is never used as an address on the host.
namespace {
constexpr size_t SS_POL = 0;
constexpr size_t SS_TICKET = SS_POL + sizeof(disco_policy) * DISCO_MAX_COLS;
constexpr size_t SS_PART = SS_TICKET + sizeof(unsigned) * 64;
constexpr size_t SS_TOTALS_BYTES = (size_t)DISCO_NCOPY * 64 * (sizeof(DispPartial) + sizeof(MigPartial));
constexpr size_t SS_BYTES = SS_PART + SS_TOTALS_BYTES;
static_assert(SS_TICKET % 256 == 0 && SS_PART % 256 == 0, "regions of the fixed scratch are 256-byte aligned");
static_assert(SS_BYTES == DISCO_STATIC_SCRATCH_BYTES, "the size the public header states");
}  // namespace

static __device__ __align__(256) unsigned char scratch[SS_BYTES];

namespace {
constexpr int SS_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
char* g_scratch_ptr[SS_MAX_DEVICES];       // device address of `scratch` on each GPU, looked up on first use

int static_scratch(char** out)
{
    int dev = -1;
    DISCO_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= SS_MAX_DEVICES) return DISCO_ERR_RANGE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        DISCO_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || ((uintptr_t)p & 255u) != 0) return DISCO_ERR_WORKSPACE;
        g_scratch_ptr[dev] = (char*)p;
    }
    *out = g_scratch_ptr[dev];
    return DISCO_OK;
}
}  // namespace

extern "C" int32_t disco_eval_dispatch_static(const disco_trace* trace, const disco_policy* pol, int32_t P,
                                              const disco_pair_out* out, disco_accum* acc, void* stream_)
{
    int rc = check_trace(trace);
    if (rc) return rc;
    if (!pol || !acc) return DISCO_ERR_NULL;
    if (P < 1 || P > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;       // the scratch holds DISCO_MAX_COLS columns
    char* ws = nullptr;
    rc = static_scratch(&ws);
    if (rc) return rc;
    hipStream_t stream = (hipStream_t)stream_;
    WsLayout L;
    memset(&L, 0, sizeof(L));
    L.pol = SS_POL; L.ticket = SS_TICKET; L.part = SS_PART; L.total = SS_BYTES;
    return eval_dispatch(view_of(trace), pol, P, out, acc, ws, L, stream);
}

extern "C" int32_t disco_eval_migration(const disco_trace* trace, const disco_timeline_params* tl,
                                        const disco_policy* pol, int32_t P, const disco_mig_out* out,
                                        disco_accum* acc, void* ws_, size_t ws_bytes, void* stream_)
{
    int rc = check_trace(trace);
    if (rc) return rc;
    if (!tl || !pol || !acc) return DISCO_ERR_NULL;
    if (P < 1 || P > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;
    if (!(tl->tau > 0.0f) || !(tl->kappa_lag >= 0.0f)) return DISCO_ERR_RANGE;
    if (trace->n_req > 0 && !trace->tok_arr && !trace->srv_tbt) return DISCO_ERR_CSR;
    if (out && out->delivered && (!trace->tok_off || out->delivered_col < 0 || out->delivered_col >= P))
        return DISCO_ERR_CSR;
    rc = check_ws(ws_, ws_bytes, P);
    if (rc) return rc;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)ws_;
    const WsLayout L = disco_ws_layout(P);
    if (!(out && out->delivered) && ws_bytes < disco_ws_full_bytes(L, trace->n_req)) return DISCO_ERR_WORKSPACE;
    TraceView v = view_of(trace);
    if (out && out->delivered) v.off = trace->tok_off;      // offsets index `delivered` even without tok_arr
    const bool small = disco_small(v.n_req) && !(out && out->delivered);
    PolTable host;
    const disco_policy* device = nullptr;
    rc = small ? small_table(pol, P, host, &device) : stage_policies(pol, P, ws, L, stream);
    if (rc) return rc;
    TimelineArgs a;
    memset(&a, 0, sizeof(a));
    a.tau = tl->tau;
    a.kt = tl->kappa_lag * tl->tau;
    a.P = P; a.nq = 1; a.pass = -1;
    if (out) {
        a.mig_idx = out->mig_idx; a.n_src_tok = out->n_src_tok; a.t_last = out->t_last;
        a.delivered = out->delivered; a.delivered_col = out->delivered_col;
        a.delay_num = out->delay_num;
    }
    a.bc = buffer_prices(tl->cost);
    a.buffer_flag = (unsigned*)(ws + L.ticket) + DISCO_FLAG_BUFFER;
    a.part = (MigPartial*)(ws + L.part);
    a.ticket = (unsigned*)(ws + L.ticket);
    a.acc = acc;
    a.S = (SelState*)(ws + L.sel);
    a.ghist = (unsigned*)(ws + L.ghist);
    // Streaming kernels (token walk into per-request summaries, per-column totals from them, then the pairs with a
    // buffer hand-off), unless per-token deliveries are wanted: then the general kernel.
    if (a.delivered) {
        disco_launch_timeline_general(v, trace->n_tok, (const disco_policy*)(ws + L.pol), a, stream);
    } else {
        a.wflags = (unsigned char*)(ws + L.total);
        a.summary = ws + disco_ws_summary_offset(L, v.n_req);
        a.counter = (unsigned*)(ws + L.wcount);
        a.bufsum = ws + disco_ws_bufsum_offset(L, v.n_req);
        if (small)
            disco_launch_small_stats(v, trace->n_tok, host, device, (disco_policy*)(ws + L.pol), (unsigned*)(ws + L.ticket), a,
                                     tl_totals((u64*)(ws + L.part)), stream);
        else
            disco_launch_tl_stats_fast(v, trace->n_tok, (const disco_policy*)(ws + L.pol), a,
                                   tl_totals((u64*)(ws + L.part)), stream);
    }
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

// Measurement aid: the streaming token walk of disco_eval_migration, timed alone with HIP events on `stream`.
extern "C" int32_t disco_time_token_walk(const disco_trace* trace, const disco_timeline_params* tl, const disco_policy* pol,
                                         int32_t P, void* ws_, size_t ws_bytes, int32_t reps, double* mean_ms, double* min_ms,
                                         void* stream_)
{
    int rc = check_trace(trace);
    if (rc) return rc;
    if (!tl || !pol || !mean_ms || !min_ms) return DISCO_ERR_NULL;
    if (P < 1 || P > DISCO_MAX_COLS || reps < 1 || reps > 1000) return DISCO_ERR_SHAPE;
    if (!(tl->tau > 0.0f) || !(tl->kappa_lag >= 0.0f)) return DISCO_ERR_RANGE;
    if (trace->n_req <= 0 || !trace->tok_arr) return DISCO_ERR_CSR;          // the streaming walk reads a token array
    rc = check_ws(ws_, ws_bytes, P);
    if (rc) return rc;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)ws_;
    const WsLayout L = disco_ws_layout(P);
    if (ws_bytes < disco_ws_full_bytes(L, trace->n_req)) return DISCO_ERR_WORKSPACE;
    const TraceView v = view_of(trace);
    rc = stage_policies(pol, P, ws, L, stream);
    if (rc) return rc;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    DISCO_HIP(hipEventCreate(&e0));
    DISCO_HIP(hipEventCreate(&e1));
    double sum = 0.0, best = 1e300;
    for (int r = 0; r <= reps && rc == DISCO_OK; ++r) {          // the first run warms up and is not counted
        disco_launch_tl_walk(v, trace->n_tok, (const disco_policy*)(ws + L.pol), P, tl->tau, tl->kappa_lag * tl->tau,
                             (unsigned char*)(ws + L.total), ws + disco_ws_summary_offset(L, v.n_req), (unsigned*)(ws + L.wcount),
                             stream, e0, e1);
        hipError_t e = hipEventSynchronize(e1);
        float ms = 0.0f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) { disco_set_hip_error(e, "timing the token walk"); rc = DISCO_ERR_HIP; }
        if (r > 0) { sum += ms; if (ms < best) best = ms; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    *mean_ms = sum / reps;
    *min_ms = best;
    return DISCO_OK;
}

extern "C" int32_t disco_reduce_stats(const disco_trace* trace, const disco_cost_params* cost,
                                      const disco_timeline_params* tl, const disco_policy* pol, int32_t P,
                                      const disco_accum* acc, const disco_quantile* q, int32_t nq, disco_stats* out,
                                      void* ws_, size_t ws_bytes, void* stream_)
{
    int rc = check_trace(trace);
    if (rc) return rc;
    if (!cost || !acc || !out || !pol) return DISCO_ERR_NULL;
    if (P < 1 || P > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;
    if (nq < 0 || nq > DISCO_MAX_Q || (nq > 0 && !q)) return nq > 0 && !q ? DISCO_ERR_NULL : DISCO_ERR_SHAPE;
    if (P * nq > DISCO_MAX_SLOTS) return DISCO_ERR_SHAPE;
    for (int i = 0; i < nq; ++i)
        if (q[i].den <= 0 || q[i].num < 0 || q[i].num > q[i].den) return DISCO_ERR_RANGE;
    if (tl && (!(tl->tau > 0.0f) || !(tl->kappa_lag >= 0.0f))) return DISCO_ERR_RANGE;
    if (tl && trace->n_req > 0 && !trace->tok_arr && !trace->srv_tbt) return DISCO_ERR_CSR;
    if (tl && nq > 0 && trace->n_req > 0xFFFFFFFFll) return DISCO_ERR_SHAPE;     // the walk list holds 32-bit request indices
    rc = check_ws(ws_, ws_bytes, P);
    if (rc) return rc;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)ws_;
    const WsLayout L = disco_ws_layout(P);
    if (tl && nq > 0 && ws_bytes < disco_ws_full_bytes(L, trace->n_req)) return DISCO_ERR_WORKSPACE;
    const TraceView v = view_of(trace);
    SelState* S = (SelState*)(ws + L.sel);
    unsigned* gh = (unsigned*)(ws + L.ghist);
    disco_quantile qs[4] = {{0, 1}, {0, 1}, {0, 1}, {0, 1}};
    for (int i = 0; i < nq; ++i) qs[i] = q[i];
    SelInit si;
    memset(&si, 0, sizeof(si));
    si.S = S; si.nq = nq; si.acc = acc; si.n_req = v.n_req;
    for (int i = 0; i < 4; ++i) si.q[i] = qs[i];
    si.with_tbt = tl != nullptr;
    si.ppcnt = (unsigned*)(ws + L.ppcnt); si.dhist = (unsigned*)(ws + L.dhist);
    si.ghist = disco_small(v.n_req) ? gh : nullptr;        // (the general TTFT passes use the bins in between)
    FinalArgs fin;
    memset(&fin, 0, sizeof(fin));
    fin.nq = nq; fin.with_tl = tl ? 1 : 0; fin.tbt = tl && nq > 0 ? 1 : 0; fin.n_req = v.n_req; fin.cost = *cost;
    for (int i = 0; i < DISCO_MAX_Q; ++i) fin.q[i] = qs[i];
    fin.acc = acc; fin.S = S; fin.dhist = (const unsigned*)(ws + L.dhist); fin.out = out;
    const bool small = nq > 0 && disco_small(v.n_req);
    if (small) {
        // staging, the starts of the selections and the whole TTFT selection, without timelines the records as well
        PolTable host;
        const disco_policy* device;
        rc = small_table(pol, P, host, &device);
        if (rc) return rc;
        disco_launch_small_begin(v, host, device, P, (disco_policy*)(ws + L.pol), (unsigned*)(ws + L.ticket), si, fin, stream);
    } else {
        rc = stage_policies(pol, P, ws, L, stream, nq > 0 ? &si : nullptr);        // with the start of the TTFT selection
        if (rc) return rc;
    }
    if (nq > 0) {
        unsigned char* ubytes = ws_bytes >= L.total + (size_t)v.n_req ? (unsigned char*)(ws + L.total) : nullptr;
        // (the descriptors of the TBT selection are written after the TTFT passes)
        u64* masks = ws_bytes >= disco_ws_full_bytes(L, v.n_req) ? (u64*)(ws + disco_ws_desc_offset(L, v.n_req)) : nullptr;
        for (int pass = 0; !small && pass < disco_ttft_passes(v.n_req, P, nq); ++pass)
            disco_launch_ttft_pass(v, (const disco_policy*)(ws + L.pol), P, nq, pass, S, (unsigned*)(ws + L.slices), gh,
                                   ubytes, masks, stream);
        if (tl) {
            TimelineArgs a;
            memset(&a, 0, sizeof(a));
            a.tau = tl->tau;
            a.kt = tl->kappa_lag * tl->tau;
            a.P = P; a.nq = nq;
            a.ticket = (unsigned*)(ws + L.ticket);
            a.S = S; a.ghist = gh;
            a.bc = buffer_prices(tl->cost);
            a.dhist = (unsigned*)(ws + L.dhist);
            a.buffer_flag = (unsigned*)(ws + L.ticket) + DISCO_FLAG_BUFFER;
            // column sets -> classes, then the radix passes; the digits are sized on the device and
            // launches after the last needed pass return at once
            a.ppcnt = (unsigned*)(ws + L.ppcnt);
            const disco_policy* dpol = (const disco_policy*)(ws + L.pol);
            // what the token walk found per request: left in the workspace by disco_eval_migration, or walked now
            a.wflags = (unsigned char*)(ws + L.total);
            a.summary = ws + disco_ws_summary_offset(L, v.n_req);
            a.counter = (unsigned*)(ws + L.wcount);
            a.bufsum = ws + disco_ws_bufsum_offset(L, v.n_req);
            if (!tl->reuse_walk) {
                if (disco_small(v.n_req)) {
                    PolTable none;
                    memset(&none, 0, sizeof(none));
                    disco_launch_small_walk(v, trace->n_tok, none, dpol, P, a.tau, a.kt, a.summary, nullptr, nullptr, nullptr, stream);
                } else {
                    disco_launch_tl_walk(v, trace->n_tok, dpol, P, a.tau, a.kt, a.wflags, a.summary, a.counter, stream);
                }
                disco_launch_tl_stats_buf(v, trace->n_tok, dpol, a, nullptr, stream);      // summaries only
            }
            disco_launch_tl_classify(v, dpol, P, a.summary, a.bufsum, a.bc, S, stream);
            a.desc = (u64*)(ws + disco_ws_desc_offset(L, v.n_req));
            a.list = (unsigned*)(a.desc + v.n_req);
            unsigned* slices = (unsigned*)(ws + L.slices);
            disco_launch_tl_assign(v, dpol, P, tl->tau, a.summary, S, a.bufsum, a.desc, a.list, slices, L.total - L.slices, a.ppcnt, gh,
                                   a.dhist, stream);
            // (the slices of the assignment have been added up by then; the second set of bins lies in front of the pools)
            const size_t bins = DISCO_GHIST_WORDS * sizeof(unsigned);
            disco_launch_tl_runs(v, trace->n_tok, a, ws + L.slices + bins, L.total - L.slices - bins, stream);
            for (int pass = 0; pass < DISCO_TBT_MAX_PASS; ++pass) {
                // the passes take turns with two sets of bins: one is counted into while the other one is cleared
                a.pass = pass;
                a.ghist = pass & 1 ? slices : gh;
                a.gclear = pass & 1 ? gh : slices;
                disco_launch_tbt_pass(v, trace->n_tok, dpol, a, fin, stream);       // (the last one makes the records)
            }
        }
    }
    if (fin.tbt || small) {
        DISCO_HIP(hipGetLastError());
        return DISCO_OK;
    }
    hipLaunchKernelGGL(k_stats_final, dim3((unsigned)P), dim3(FINAL_THREADS), 0, stream, fin);
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

extern "C" int32_t disco_average_runs(const disco_stats* in, int32_t groups, int32_t runs, disco_stats* out, void* stream_)
{
    if (!in || !out) return DISCO_ERR_NULL;
    if (groups < 0 || runs < 1) return DISCO_ERR_SHAPE;
    if (groups == 0) return DISCO_OK;
    hipLaunchKernelGGL(k_average_runs, dim3((unsigned)((groups + 63) / 64)), dim3(64), 0, (hipStream_t)stream_, in, groups, runs,
                       out);
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

extern "C" int32_t disco_ingest_trace(const disco_raw_trace* raw, disco_trace* trace, void* stream_)
{
    if (!raw || !trace) return DISCO_ERR_NULL;
    if (raw->n_req < 0 || raw->n_tok < 0) return DISCO_ERR_SHAPE;
    if (raw->n_req > 0 && (!raw->t_send || !raw->tok_off || !trace->srv_ttft || !trace->output_len)) return DISCO_ERR_NULL;
    if (raw->n_tok > 0 && (!raw->t_token || !trace->tok_arr)) return DISCO_ERR_NULL;
    trace->n_req = raw->n_req;
    trace->n_tok = raw->n_tok;
    trace->tok_off = const_cast<int64_t*>(raw->tok_off);
    if (raw->n_req == 0) return DISCO_OK;
    disco_launch_ingest(raw->n_req, raw->n_tok, raw->t_send, raw->t_token, raw->tok_off, trace->srv_ttft, trace->output_len,
                        trace->tok_arr, (hipStream_t)stream_);
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

extern "C" int32_t disco_fit_lognormal(const void* x, int32_t kind, int64_t n, disco_lognormal_fit* out, void* ws_,
                                       size_t ws_bytes, void* stream_)
{
    if (!out || (n > 0 && !x)) return DISCO_ERR_NULL;
    if (n < 0) return DISCO_ERR_SHAPE;
    if (kind != DISCO_FIT_INT32 && kind != DISCO_FIT_FLOAT32) return DISCO_ERR_RANGE;
    int rc = check_ws(ws_, ws_bytes, 1);
    if (rc) return rc;
    const WsLayout L = disco_ws_layout(1);
    if (disco_fit_scratch_bytes() > L.total - L.slices) return DISCO_ERR_WORKSPACE;
    disco_launch_fit(x, kind, n, out, (char*)ws_ + L.slices, (hipStream_t)stream_);
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

extern "C" int32_t disco_solve_policy(const disco_trace* trace, const disco_solve_spec* spec, int32_t n, disco_policy* pol_out,
                                      disco_solve_out* out, void* ws_, size_t ws_bytes, void* stream_)
{
    int rc = check_trace(trace);
    if (rc) return rc;
    if (!spec || !pol_out) return DISCO_ERR_NULL;
    if (n < 1 || n > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;
    for (int j = 0; j < n; ++j) {
        const disco_solve_spec& s = spec[j];
        if (s.mode != DISCO_MODE_SERVER_CONSTRAINED && s.mode != DISCO_MODE_DEVICE_CONSTRAINED) return DISCO_ERR_RANGE;
        if (s.b_den < 1 || s.b_den > 32768 || s.b_num < 0 || s.b_num > s.b_den) return DISCO_ERR_RANGE;
        if (s.mode == DISCO_MODE_DEVICE_CONSTRAINED &&
            (s.a_den < 1 || s.a_den > 32768 || s.a_num <= 0 || s.a_num >= s.a_den))
            return DISCO_ERR_RANGE;
        if (s.mig_mode < DISCO_MIG_NONE || s.mig_mode > DISCO_MIG_BUFFER) return DISCO_ERR_RANGE;
    }
    rc = check_ws(ws_, ws_bytes, n);
    if (rc) return rc;
    char* ws = (char*)ws_;
    const WsLayout L = disco_ws_layout(n);
    if (disco_solve_state_bytes() > L.ghist - L.sel) return DISCO_ERR_WORKSPACE;      // the selection state region holds it
    const TraceView v = view_of(trace);
    disco_launch_solve(v, spec, n, ws + L.sel, (u64*)(ws + L.ppcnt),
                       (unsigned*)(ws + L.slices), L.total - L.slices, pol_out, out, (hipStream_t)stream_);
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}

extern "C" int32_t disco_budget_search(const disco_trace* trace, const disco_cost_params* cost,
                                       const disco_policy* templ, const disco_search_spec* spec, int32_t n_search,
                                       disco_search_out* out, disco_policy* pol_out, disco_accum* acc_out, void* ws_,
                                       size_t ws_bytes, void* stream_)
{
    int rc = check_trace(trace);
    if (rc) return rc;
    if (!cost || !spec || !out || !templ) return DISCO_ERR_NULL;
    if (n_search < 1 || n_search > DISCO_MAX_COLS) return DISCO_ERR_SHAPE;
    const int n_steps = spec[0].n_steps;
    if (n_steps < 1 || n_steps > DISCO_MAX_STEPS) return DISCO_ERR_SHAPE;
    SpecTable t;
    memset(&t, 0, sizeof(t));
    const bool host_templ = !is_device_pointer(templ);
    for (int j = 0; j < n_search && host_templ; ++j)                          // the stochastic baselines have no searched parameter
        if (templ[j].mode >= DISCO_MODE_STOCH_SERVER) return DISCO_ERR_RANGE;
    for (int j = 0; j < n_search; ++j) {
        if (spec[j].n_steps != n_steps) return DISCO_ERR_SHAPE;
        if (spec[j].which_param < DISCO_PARAM_L_TH || spec[j].which_param > DISCO_PARAM_BETA) return DISCO_ERR_RANGE;
        if (spec[j].which_acc < DISCO_ACC_TOTAL_COST || spec[j].which_acc > DISCO_ACC_DEVICE_PREFILL_TOK)
            return DISCO_ERR_RANGE;
        if (!(spec[j].lo <= spec[j].hi) || spec[j].target != spec[j].target) return DISCO_ERR_RANGE;
        if (spec[j].which_param == DISCO_PARAM_L_TH && (spec[j].lo < -2147483647.0 || spec[j].hi > 2147483647.0))
            return DISCO_ERR_RANGE;
        t.s[j].lo = spec[j].lo; t.s[j].hi = spec[j].hi; t.s[j].target = spec[j].target;
        t.s[j].which_param = spec[j].which_param; t.s[j].which_acc = spec[j].which_acc;
        t.s[j].step = 0; t.s[j].n_steps = n_steps;
    }
    rc = check_ws(ws_, ws_bytes, n_search);
    if (rc) return rc;
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)ws_;
    const WsLayout L = disco_ws_layout(n_search);
    const TraceView v = view_of(trace);
    // Length thresholds of server-constrained columns against a prompt-token budget: the accumulator is a
    // function of the threshold alone and is tabulated once (Alg. 3's sorted running totals); all bisection
    // steps then read the table.  Needs a host-resident template table (its modes are inspected here).
    bool tabulated = v.n_req > 0 && host_templ;
    double max_hi = 0.0;
    for (int j = 0; j < n_search && tabulated; ++j) {
        tabulated = templ[j].mode == DISCO_MODE_SERVER_CONSTRAINED && spec[j].which_param == DISCO_PARAM_L_TH &&
                    (spec[j].which_acc == DISCO_ACC_SERVER_PREFILL_TOK || spec[j].which_acc == DISCO_ACC_DEVICE_PREFILL_TOK) &&
                    spec[j].lo >= 0.0 && spec[j].hi + 2.0 <= (double)disco_search_table_max_bins();
        if (spec[j].hi > max_hi) max_hi = spec[j].hi;
    }
    if (tabulated && disco_small(v.n_req)) {
        rc = check_policies(templ, n_search);
        if (rc) return rc;
        PolTable pt;
        SmallSearches sp;
        memset(&pt, 0, sizeof(pt));
        memset(&sp, 0, sizeof(sp));
        memcpy(pt.p, templ, sizeof(disco_policy) * (size_t)n_search);
        for (int j = 0; j < n_search; ++j)
            sp.s[j] = SmallSearch{spec[j].target, (int)spec[j].lo, (int)spec[j].hi, spec[j].which_acc, 0};
        disco_launch_small_search(v, pt, sp, n_search, n_steps, (int)max_hi + 2, *cost, out, pol_out, acc_out, stream);
        DISCO_HIP(hipGetLastError());
        return DISCO_OK;
    }
    // bisection passes only need the totals their accumulators are made of
    int need = 0;
    for (int j = 0; j < n_search; ++j)
        if (spec[j].which_acc != DISCO_ACC_SERVER_PREFILL_TOK && spec[j].which_acc != DISCO_ACC_DEVICE_PREFILL_TOK) need = 1;
    // Waits and ramp slopes of device-constrained columns: the outcomes of a request are step functions of the
    // parameter, a pass takes ten bisection steps (disco_search.hip), where that is the faster way.  The bounds are such
    // that no midpoint overflows and no ramp is infinity times zero.
    bool waits = !tabulated && host_templ;
    for (int j = 0; j < n_search && waits; ++j)
        waits = templ[j].mode == DISCO_MODE_DEVICE_CONSTRAINED && spec[j].which_param != DISCO_PARAM_L_TH &&
                 spec[j].lo >= -1e37 && spec[j].hi <= 1e37;
    const bool small_waits = waits && disco_small(v.n_req) && v.n_req <= WAIT_SMALL_REQ;
    const bool binned = waits && !small_waits && disco_search_bins_bytes(n_search) <= L.total - L.slices &&
                        disco_search_bins_pays(v.n_req, n_search, n_steps, need != 0);
    PolTable host;
    if (small_waits || binned) {
        memset(&host, 0, sizeof(host));
        rc = check_policies(templ, n_search);
        if (rc == DISCO_OK) memcpy(host.p, templ, sizeof(disco_policy) * (size_t)n_search);
    } else {
        rc = stage_policies(templ, n_search, ws, L, stream);
    }
    if (rc) return rc;
    if (small_waits) {
        disco_launch_small_wait_search(v, host, n_search, n_steps, t, *cost, out, pol_out, acc_out, stream);
        DISCO_HIP(hipGetLastError());
        return DISCO_OK;
    }
    DispFin fin;
    memset(&fin, 0, sizeof(fin));
    fin.kind = 1;
    fin.cost = *cost;
    fin.st = (SearchState*)(ws + L.search);
    fin.sout = out;
    fin.pol_out = pol_out;
    fin.acc = acc_out;
    fin.pol_rw = (disco_policy*)(ws + L.pol);
    fin.templ = (const disco_policy*)(ws + L.templ);
    fin.n_search = n_search;
    if (tabulated) {
        disco_launch_search_table(v, t, n_search, (int)max_hi + 2, (unsigned*)(ws + L.slices), L.total - L.slices,
                                  (u64*)(ws + L.ppcnt), fin.st, fin.pol_rw, out, stream);
    } else if (binned) {
        disco_launch_search_bins(v, host, n_search, n_steps, t, *cost, ws + L.slices, L.total - L.slices, (SearchState*)(ws + L.search),
                                 fin.pol_rw, (disco_policy*)(ws + L.templ), (unsigned*)(ws + L.ticket), (u64*)(ws + L.part), out, stream);
    } else {
        // Every pass evaluates the next `depth` levels of each search's bisection tree as columns of their own and so
        // takes `depth` bisection steps; the recorded steps are those of the plain bisection.
        const int depth = disco_search_depth(n_search);
        hipLaunchKernelGGL(k_search_init, dim3(1), dim3(64), 0, stream, t, n_search, fin.st, fin.pol_rw,
                           (disco_policy*)(ws + L.templ), depth);
        const int npass = (n_steps + depth - 1) / depth;
        fin.depth = depth;
        fin.need = need;
        for (int pass = 0; pass < npass; ++pass) {
            fin.last = pass == npass - 1;
            disco_launch_dispatch_acc(v, (const disco_policy*)(ws + L.pol), n_search * ((1 << depth) - 1), (u64*)(ws + L.part),
                                      fin, stream);
        }
    }
    // the evaluation at the answers
    fin.depth = 0; fin.last = 0; fin.need = 2;
    disco_launch_dispatch_acc(v, (const disco_policy*)(ws + L.pol), n_search, (u64*)(ws + L.part), fin, stream);
    DISCO_HIP(hipGetLastError());
    return DISCO_OK;
}
