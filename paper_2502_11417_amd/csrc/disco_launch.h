// Host-side launch interface between the translation units of libdisco.
#pragma once
#include "disco_state.h"

// dc = price difference of a decode token (source minus target), cp = target's prefill price; _srv: server
// source handing off to the device, _dev: device source handing off to the server.
struct BufCostArgs { double dc_srv, cp_srv, dc_dev, cp_dev; };

// Gaps counted per value: pool b (`cap` entries, the first one its header: entries written, 0) is filled by workgroup b of the
// launch that makes the runs and read by every pass.  An entry: bit pattern of the gap, number of such gaps in the low
// RUN_COUNT_BITS bits of the other word, above them the LDS row of the timeline.
constexpr int RUN_COUNT_BITS = 26;
struct RunPool { uint2* pool; unsigned cap; int n; };

// Start of the order-statistic selections (disco_stage.h).
struct SelInit {
    SelState* S; int nq; disco_quantile q[4]; const disco_accum* acc; i64 n_req; int with_tbt;
    unsigned *ppcnt, *dhist;       // counts of the TBT selection, cleared in the launch that starts it
    unsigned* ghist;               // ... and its bins (nullable)
};

// What the result records are made from (disco_final.h).
struct FinalArgs {
    int nq, with_tl, tbt;          // tbt: there was a TBT selection
    i64 n_req;
    disco_cost_params cost;
    disco_quantile q[DISCO_MAX_Q];
    const disco_accum* acc;
    const SelState* S;
    const unsigned* dhist;
    disco_stats* out;
};

struct TimelineArgs {
    float tau, kt;            // pacing interval, kappa_lag * tau
    int P, nq, pass;          // -1: statistics pass, >= 0: TBT histogram pass
    int32_t* mig_idx; int32_t* n_src_tok; float* t_last; float* delivered; int delivered_col;
    MigPartial* part; unsigned* ticket; disco_accum* acc;
    SelState* S;
    unsigned* ghist;          // device-wide bins of the pass
    unsigned* gclear;         // histogram passes: those of the next one, cleared in the meantime
    unsigned* ppcnt;          // pure-pacing timelines per class and length (histogram passes)
    int32_t* delay_num;       // materialised delayed-token counts (buffer hand-off), nullable
    BufCostArgs bc;           // prices of the buffer hand-off's cost test
    const unsigned* buffer_flag;   // device: 1 if the staged table has a buffer hand-off column
    unsigned* dhist;               // histogram passes: migrated requests by number of delayed tokens, per column
    unsigned char* wflags;         // one byte per request: the walks it needs (written by the statistics pass)
    void* summary;                 // TlSummary per request: what the token walk found (16 bytes each)
    unsigned* counter;             // batch counters of the token walk, one per queue (zeroed by the flags kernel)
    u64* desc;                     // per request: LDS rows of its timelines with tokens to walk, one byte per kind (histogram passes)
    void* bufsum;                  // BufSummary per request: what the walk of its buffer hand-off timelines found
    unsigned* list;                // the requests that have such a timeline, one word each (histogram passes)
    RunPool runs;                  // gaps of the timelines that need no walk (histogram passes)
};

// How the kernel behind a dispatch pass hands on the column totals.
struct DispFin {
    int kind;                     // 0: write disco_accum, 1: advance a budget search
    int need;                     // totals wanted: 0 prefill tokens, 1 + decode split, 2 + TTFT sum and range
    disco_accum* acc;
    disco_cost_params cost;
    SearchState* st;
    disco_search_out* sout;
    disco_policy* pol_out;
    disco_policy* pol_rw;         // the table the next pass reads
    // Bisection passes of a search evaluate a whole subtree of the bisection at once: search j owns the
    // 2^depth - 1 columns j * (2^depth - 1) ..., one per node of the next `depth` levels (heap order), so one pass
    // takes `depth` bisection steps; depth 0: the columns are the searches themselves (final evaluation).
    int n_search, depth;
    int last;                     // the last bisection pass: leave the answers' policies in pol_rw[0 .. n_search)
    const disco_policy* templ;    // the searches' template records
};

// Traces of up to SMALL_REQ requests take kernels of one workgroup per policy column (disco_small.h): as many as the keys of
// an order statistic fit LDS, and the column kernels are still the faster way there (32 000 requests, whole calls: search,
// totals and order statistics of 64 threshold columns 100 us with the general kernels, 62 with these; of 4 88 / 52; solve,
// totals and order statistics of 12 wait columns 157 / 82; 8 levels x 8 stochastic runs 109 / 76).  The testing aid that
// shrinks the grids sends them through the general kernels.
constexpr int SMALL_REQ = 32768;
inline bool disco_small(i64 n_req) { return n_req <= SMALL_REQ && disco_grid_divisor() == 1; }
struct SmallSearch { double target; int lo, hi, which_acc, pad; };
struct SmallSearches { SmallSearch s[DISCO_MAX_COLS]; };
// Table from device memory, or from `host` where `device` is null.
void disco_launch_small_dispatch(const TraceView& v, const PolTable& host, const disco_policy* device, int P, disco_accum* acc,
                                 uint8_t* decision, float* ttft, hipStream_t stream);
// Tabulated threshold searches (templates: server-constrained columns), with the evaluation at the answers.
void disco_launch_small_search(const TraceView& v, const PolTable& templ, const SmallSearches& sp, int n_search, int n_steps, int nbins,
                               const disco_cost_params& cost, disco_search_out* sout, disco_policy* pol_out, disco_accum* acc,
                               hipStream_t stream);
// Statistics of a small trace: TTFT order statistics; with timelines (fin.with_tl) also the staging of the table and the start of
// the TBT selection, without them the records.
void disco_launch_small_begin(const TraceView& v, const PolTable& host, const disco_policy* device, int P, disco_policy* staged,
                              unsigned* tickets, const SelInit& si, const FinalArgs& fin, hipStream_t stream);

// Levels of the bisection tree one pass can evaluate for n searches (64 columns per pass).
inline int disco_search_depth(int n) { return n <= 9 ? 3 : (n <= 21 ? 2 : 1); }

// decision, ttft: per-pair outputs, nullable.
void disco_launch_dispatch_acc(const TraceView& v, const disco_policy* pol, int P, u64* part, const DispFin& fin,
                               hipStream_t stream, uint8_t* decision = nullptr, float* ttft = nullptr);
// Threshold search of server-constrained columns from a table of prompt-token sums by length.
void disco_launch_search_table(const TraceView& v, const SpecTable& spec, int n_search, int nbins, unsigned* scratch,
                               size_t scratch_bytes, u64* table, SearchState* st, disco_policy* pol, disco_search_out* sout,
                               hipStream_t stream);
// Search of w_tail or beta over device-constrained templates (the answers end in `pol`), ten steps per pass.
// `scratch`: disco_search_bins_bytes(n_search) bytes.
size_t disco_search_bins_bytes(int n_search);
bool disco_search_bins_pays(i64 n_req, int n_search, int n_steps, bool decode);
// (`host`: the templates, staged in `pol`, with the totals cleared, by the first launch)
void disco_launch_search_bins(const TraceView& v, const PolTable& host, int n_search, int n_steps, const SpecTable& spec,
                              const disco_cost_params& cost, void* scratch, size_t scratch_bytes, SearchState* st, disco_policy* pol,
                              disco_policy* templ, unsigned* tickets, u64* totals, disco_search_out* sout, hipStream_t stream);
// The same on a trace of up to WAIT_SMALL_REQ requests, with the evaluation at the answers: one launch.  2000 requests: 16, 25
// and 38 us for 4, 16 and 32 steps, the fused passes and the ones above 41, 93 and 157; 32 000: 70, 79 and 98 us against 29, 46
// and 62 of the passes above (one workgroup: 1.8 us more per 1000 requests).
constexpr int WAIT_SMALL_REQ = 8192;
void disco_launch_small_wait_search(const TraceView& v, const PolTable& host, int n_search, int n_steps, const SpecTable& spec,
                                    const disco_cost_params& cost, disco_search_out* sout, disco_policy* pol_out, disco_accum* acc,
                                    hipStream_t stream);
int disco_search_table_max_bins(void);
int disco_launch_len_table(const TraceView& v, int nbins, unsigned* scratch, size_t scratch_bytes, u64* table, hipStream_t stream);
// Pairs with the buffer hand-off in class mode: their per-request summaries (a.bufsum), from the summaries of the
// streaming walk (a.summary) and the tokens; returns at once when the staged table has no such column.
// `totals` nullable: summaries only.
void disco_launch_tl_stats_buf(const TraceView& v, i64 n_tok, const disco_policy* pol, const TimelineArgs& a,
                               MigPartial* totals, hipStream_t stream);
// Recorded traces: timestamps to relative arrays; log-normal fit (`scratch`: disco_fit_scratch_bytes() bytes).
void disco_launch_ingest(i64 n_req, i64 n_tok, const double* t_send, const double* t_token, const i64* off, float* srv_ttft,
                         int32_t* output_len, float* tok_arr, hipStream_t stream);
size_t disco_fit_scratch_bytes(void);
void disco_launch_fit(const void* x, int kind, i64 n, disco_lognormal_fit* fit, void* scratch, hipStream_t stream);
// Closed-form policy solves (Alg. 2, Alg. 3): length table, per-column plan, multi-rank selection over the server
// TTFTs, policy records.  `state` needs disco_solve_state_bytes() bytes.
size_t disco_solve_state_bytes(void);
void disco_launch_solve(const TraceView& v, const disco_solve_spec* spec, int n, void* state, u64* table,
                        unsigned* scratch, size_t scratch_bytes, disco_policy* pol_out, disco_solve_out* out,
                        hipStream_t stream);
// One TTFT radix pass: histograms per workgroup slice (class kernel or pair kernel, decided on the device),
// row sums, digit selection.
// `ubytes`: n_req bytes of scratch (nullable) where the first pass leaves, per request, the number of thresholds
// not above its prompt length for the later passes; `masks`: n_req words (nullable) where it leaves the columns that send
// a request to the server (tables of stochastic columns).
int disco_ttft_passes(i64 n_req, int P, int nq);
void disco_launch_ttft_pass(const TraceView& v, const disco_policy* pol, int P, int nq, int pass, SelState* S,
                            unsigned* slices, unsigned* rowsum, unsigned char* ubytes, u64* masks, hipStream_t stream);
// Token timelines.  Statistics pass (a.pass = -1): streaming kernel, or the general kernel when the
// per-token deliveries of a column are wanted.  TBT selection: classification, assignment and gap pools once; then
// disco_launch_tbt_pass for every pass: two launches in a regular one (a.pass < DISCO_TBT_REGULAR_PASS: plan and
// histograms, then the digits), one in a spare one, which normally returns at once; the last one also makes the
// records.
void disco_launch_tl_stats_fast(const TraceView& v, i64 n_tok, const disco_policy* pol, const TimelineArgs& a,
                                MigPartial* totals, hipStream_t stream);
// The token walk alone (flags, then one 16-byte summary per request), for a statistics call that was not handed
// the summaries of the evaluation.
void disco_launch_tl_walk(const TraceView& v, i64 n_tok, const disco_policy* pol, int P, float tau, float kt,
                          unsigned char* wflags, void* summary, unsigned* counter, hipStream_t stream,
                          hipEvent_t before = nullptr, hipEvent_t after = nullptr);
// The same for a small trace, and the statistics pass of one: the policy table (from device memory, or `host` where `device` is
// null) is staged and the totals are cleared in the first launch (staged, tickets, totals: not written if null).
void disco_launch_small_walk(const TraceView& v, i64 n_tok, const PolTable& host, const disco_policy* device, int P, float tau, float kt,
                             void* summary, disco_policy* staged, unsigned* tickets, MigPartial* totals, hipStream_t stream);
void disco_launch_small_stats(const TraceView& v, i64 n_tok, const PolTable& host, const disco_policy* device, disco_policy* staged,
                              unsigned* tickets, const TimelineArgs& a, MigPartial* totals, hipStream_t stream);
void disco_launch_timeline_general(const TraceView& v, i64 n_tok, const disco_policy* pol, const TimelineArgs& a,
                                   hipStream_t stream);
void disco_launch_tl_classify(const TraceView& v, const disco_policy* pol, int P, const void* summary, const void* bufsum,
                              const BufCostArgs& bc, SelState* S, hipStream_t stream);
void disco_launch_tl_assign(const TraceView& v, const disco_policy* pol, int P, float tau, const void* summary, SelState* S,
                            const void* bufsum, u64* desc, unsigned* list, unsigned* slices, size_t slices_bytes,
                            unsigned* ppcnt, unsigned* ghist, unsigned* dhist, hipStream_t stream);
// After the assignment: the gaps of the listed timelines into pools in `scratch`, as far as they fit (a.runs on return); their
// descriptors then name them no more.
void disco_launch_tl_runs(const TraceView& v, i64 n_tok, TimelineArgs& a, void* scratch, size_t scratch_bytes, hipStream_t stream);
void disco_launch_tbt_pass(const TraceView& v, i64 n_tok, const disco_policy* pol, const TimelineArgs& a, const FinalArgs& fin,
                           hipStream_t stream);
