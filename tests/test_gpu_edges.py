"""Kernels whose work split depends on the size of their input, at the sizes where one form gives way to the next and
at the remainders of their tiles, against the CPU oracle (bit for bit unless a test says otherwise)."""
import numpy as np
import pytest
import torch

import disco_inputs as DI
from test_gpu_buffer import slow_prefill
from test_gpu_parity import check_dispatch, check_migration, check_stats

pytestmark = pytest.mark.gpu


def same_bits(got, want, what):
    got, want = np.ascontiguousarray(got), np.ascontiguousarray(want)
    assert got.shape == want.shape, what
    bad = np.flatnonzero(got.view(np.uint8).ravel() != want.view(np.uint8).ravel())
    assert bad.size == 0, f"{what}: {bad.size} bytes differ, first at {bad[:5]}"


# the handle that the calls get is that of torch's current stream
def test_the_current_streams_handle(B):
    side = torch.cuda.Stream()
    assert B._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert B._stream() == side.cuda_stream


# requests per wave of the token generator: 1 below 8192 requests, 4 below 32768, then 16; pieces of 64, 256 and 1024
# tokens from multiples of 32 on, or all of a wave's requests in one stretch where they have at most 1024 tokens; the stall
# test at both ends of its range
@pytest.mark.parametrize("n_req,out_mu,out_hi,stall_p", [
    (1, 6.0, 1100, 0.01), (15, 6.5, 2100, 0.5), (8191, 3.0, 70, 0.01), (8192, 4.5, 600, 0.0), (8195, 3.5, 300, 1.0),
    (32767, 3.0, 65, 0.01), (32768, 3.5, 130, 0.01), (32785, 3.5, 97, 0.25),
    (8209, 5.6, 700, 0.01), (32801, 4.2, 300, 0.02), (40_001, 0.5, 3, 0.3)])
def test_generated_tokens(B, oracle, n_req, out_mu, out_hi, stall_p):
    print(f"generated tokens: n_req={n_req} out_mu={out_mu} out_hi={out_hi} stall_p={stall_p}", flush=True)
    gen = dict(DI.config(4, n_req=n_req, seed=n_req)["gen"], out_mu=out_mu, out_hi=out_hi, gap_stall_p=stall_p)
    want = oracle.gen_trace(gen)
    got = B.disco_gen_trace(gen)
    assert got.n_tok == want["n_tok"]
    same_bits(got.tok_off.cpu().numpy(), want["tok_off"], "tok_off")
    same_bits(got.tok_arr.cpu().numpy(), want["tok_arr"], "tok_arr")


# requests per wave of the ingest: 16, 8, 2 or 1 by the mean length and the number of requests; timestamps in pairs, or one
# by one where the array starts off a 16-byte boundary; loads past the caches from 2^25 timestamps on; request lengths around
# the pairs and the steps of 512
@pytest.mark.parametrize("n_req,shift,about", [(1, 0, 3), (1, 1, 3), (131_071, 0, 3), (131_072, 1, 3), (131_087, 0, 3), (32_769, 0, 3), (40_007, 0, 30),
                                               (33_001, 1, 90), (9001, 0, 150), (8193, 1, 150), (3001, 0, 400), (66_003, 0, 520), (227_007, 0, 150)])
def test_ingested_offsets(B, n_req, shift, about):
    print(f"ingested offsets: n_req={n_req} shift={shift}", flush=True)
    rng = np.random.default_rng(n_req + shift)
    n = rng.choice([0, 1, 2, 3, 7], n_req) if n_req > 1 else np.array([5])
    if about > 3:
        n += rng.integers(0, 2 * about, n_req)
    long = [0, 1, 2, 127, 128, 129, 511, 512, 513, 1025]
    for i, length in enumerate(long[:max(0, n_req - 1)]):
        n[i * n_req // len(long)] = length
    off = np.zeros(n_req + 1, np.int64)
    np.cumsum(n, out=off[1:])
    send = 1.7e9 + np.cumsum(rng.exponential(0.3, n_req))
    tok = np.repeat(send, n) + rng.random(int(off[-1])) * 30.0
    at = torch.zeros(len(tok) + shift, dtype=torch.float64, device="cuda")[shift:]
    at.copy_(torch.from_numpy(tok))
    got = B.disco_ingest_trace(torch.from_numpy(send).cuda(), at, torch.from_numpy(off).cuda(),
                               torch.ones(n_req, dtype=torch.int32, device="cuda"))
    first = tok[np.minimum(off[:-1], len(tok) - 1)]
    same_bits(got.tok_arr.cpu().numpy(), (tok - np.repeat(first, n)).astype(np.float32), "tok_arr")
    same_bits(got.output_len.cpu().numpy(), n.astype(np.int32), "output_len")
    ttft = got.srv_ttft.cpu().numpy()
    assert np.isnan(ttft[n == 0]).all()
    same_bits(ttft[n > 0], (first - send).astype(np.float32)[n > 0], "srv_ttft")


# token check: vectors of four from the first 16-byte boundary on, steps of 256 vectors; a decrease anywhere is found,
# the steps down to the next request's first token are none
@pytest.mark.parametrize("lengths", [[1], [3], [2, 1, 2], [1] * 9, [1023, 2, 1025], [4096, 1, 1, 300]])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_decreasing_tokens_are_found_anywhere(B, lengths, shift):
    print(f"token check: lengths={lengths} shift={shift}", flush=True)
    n = np.array(lengths)
    off = np.zeros(len(n) + 1, np.int64)
    np.cumsum(n, out=off[1:])
    total = int(off[-1])
    inside = np.arange(total) - np.repeat(off[:-1], n)
    arr = (0.25 * inside).astype(np.float32)
    buf = torch.zeros(total + shift, dtype=torch.float32, device="cuda")[shift:]
    ones = torch.ones(len(n), dtype=torch.int32, device="cuda")
    tr = B.Trace(n_req=len(n), n_tok=total, prompt_len=ones, output_len=torch.from_numpy(n.astype(np.int32)).cuda(),
                 srv_ttft=ones.float(), tok_off=torch.from_numpy(off).cuda(), tok_arr=buf, dev_pre_spt_s=0.1, dev_dec_spt_s=0.1)
    buf.copy_(torch.from_numpy(arr))
    assert B.disco_validate_trace(tr) == 0
    places = np.flatnonzero(inside >= 2)
    for j in places if len(places) < 8 else [*places[:4], *places[len(places) // 2:][:2], *places[-4:]]:
        planted = arr.copy()
        planted[j] = np.float32(0.25 * (inside[j] - 1) - 0.125)
        buf.copy_(torch.from_numpy(planted))
        assert B.disco_validate_trace(tr) == B.ERR["range"], j


# device -> server hand-offs: batches of 4 .. 64 requests per wave, tails of 1 token to several chunks of 256 from every
# alignment, stalls among them; twelve wait columns give the TBT digits 10 + 10 + 1 bits (the last one by the narrow select)
@pytest.mark.parametrize("n_req,max_out,stall_p", [(1, 3, 0.0), (63, 1200, 0.05), (777, 300, 0.0), (12_289, 24, 0.02),
                                                   (4097, 60, 0.05), (20_001, 9, 0.05), (32_801, 5, 0.1)])
def test_server_tails_of_wait_columns(B, oracle, n_req, max_out, stall_p):
    print(f"server tails: n_req={n_req} max_out={max_out} stall_p={stall_p}", flush=True)
    tr = slow_prefill(DI.handmade_trace(61 + n_req, n_req, tokens=True, max_out=max_out, stall_p=stall_p), 16.0)
    specs = [dict(mode=1, l_th=-1, w_tail=DI.f32(0.04 * j), mig_mode=2) for j in range(12)]
    check_migration(B, oracle, tr, specs, DI.TAU, DI.KAPPA_LAG, delivered_col=None, cost=DI.COST_D)
    check_stats(B, oracle, tr, specs, DI.COST_D, tau=DI.TAU, kappa=DI.KAPPA_LAG)


# ten bisection steps per pass: step counts around the passes, one to several searches of both parameters at once,
# arrays on and off 16-byte boundaries, exact ties at the searched wait, brackets that run out of floats
@pytest.mark.parametrize("n_req,n_steps,shift", [(0, 9, 0), (1, 1, 0), (5, 8, 0), (777, 9, 1), (4099, 32, 0), (4096, 64, 3)])
def test_wait_and_slope_searches(B, oracle, n_req, n_steps, shift):
    print(f"wait searches: n_req={n_req} n_steps={n_steps} shift={shift}", flush=True)
    tr = DI.handmade_trace(90 + n_req, n_req, tokens=False, ties=True)
    tr["srv_ttft"][: n_req // 4] = np.float32(0.5)                     # the first midpoint of the bracket [0, 1]
    total = float(tr["prompt_len"].sum(dtype=np.int64))
    searches = [  # template, parameter, accumulator, lo, hi, target
        (dict(mode=1, l_th=-1), B.PARAM_W_TAIL, "device_cost", 0.0, 1.0, 0.3 * DI.COST_D["cs_pre"] * total),
        (dict(mode=1, l_th=200, l_mid=201, w_mid=DI.f32(0.1)), B.PARAM_W_TAIL, "device_prefill_tok", 0.0, 4.0, 0.4 * total),
        (dict(mode=1, l_th=-1, beta=DI.f32(1e-3)), B.PARAM_W_TAIL, "total_cost", 0.25, 0.25, 0.0),
        (dict(mode=1, l_th=-1), B.PARAM_W_TAIL, "server_prefill_tok", -1.0, 2.0, 0.5 * total),
        (dict(mode=1, l_th=100, w_tail=DI.f32(0.8)), B.PARAM_BETA, "device_prefill_tok", 0.0, 0.01, 0.2 * total),
    ]
    dt = B.upload_trace(tr)
    for name in ("prompt_len", "output_len", "srv_ttft", "dev_pre_spt"):
        x = getattr(dt, name)
        buf = torch.zeros(x.numel() + shift, dtype=x.dtype, device="cuda")[shift:]
        buf.copy_(x)
        setattr(dt, name, buf)
    out = B.disco_budget_search(dt, DI.COST_D, [B.Policy(**s[0]) for s in searches],
                                [dict(which_param=p, which_acc=acc, n_steps=n_steps, lo=lo, hi=hi, target=target)
                                 for _, p, acc, lo, hi, target in searches])
    so = B.search_to_host(out["out"], len(searches))
    pol = B.policies_to_host(out["pol_out"], len(searches))
    for j, (templ, p, acc, lo, hi, target) in enumerate(searches):
        find = oracle.search_wait if p == B.PARAM_W_TAIL else oracle.search_slope
        x, hp, ha = find(tr, oracle.Policy(**templ), lo, hi, n_steps, acc, DI.COST_D, target)
        same_bits(so["hist_param"][j][:n_steps].astype(np.float32), hp, f"hist_param {j}")
        same_bits(so["hist_acc"][j][:n_steps], ha, f"hist_acc {j}")
        got = pol[j].w_tail if p == B.PARAM_W_TAIL else pol[j].beta
        assert np.float32(got) == np.float32(x) == np.float32(so["param"][j]), j


# tables of stochastic columns alone: the variates staged whole (dispatch) and 16 requests at a time (TTFT passes, tables
# of more than four columns), 1 .. 8 shared runs and 9 that are not shared, ragged batches, lengths beyond 24 bits
@pytest.mark.parametrize("n_req,levels,runs,huge", [(1, 1, 1, False), (64, 2, 2, False), (1027, 5, 1, False), (4096, 4, 8, True),
                                                    (2049, 8, 8, False), (1999, 7, 9, False), (3000, 3, 5, True)])
def test_tables_of_stochastic_columns(B, oracle, n_req, levels, runs, huge):
    print(f"stochastic tables: n_req={n_req} levels={levels} runs={runs} huge={huge}", flush=True)
    tr = DI.handmade_trace(130 + n_req, n_req, tokens=False, ties=True)
    if huge:
        tr["prompt_len"][n_req // 2] = (1 << 24) + 3
    specs = [dict(mode=2 + (j & 1), beta=DI.f32((j + 1) / (levels + 1)), l_mid=17 * run) for j in range(levels) for run in range(runs)]
    check_dispatch(B, oracle, tr, specs)
    check_stats(B, oracle, tr, specs, DI.COST_S)
    check_stats(B, oracle, tr, specs, DI.COST_S, ws_requests=0)         # no room for the routing: drawn again in every pass


# tabulated threshold searches: four steps per round of table reads (step counts around the rounds), tables that end at,
# in front of and behind a block of 64 lengths and the largest one, prompts longer than the table, 1 .. 64 searches
@pytest.mark.parametrize("n_req,n_search,n_steps,hi", [(0, 1, 1, 0), (1, 1, 4, 1), (700, 3, 5, 61), (700, 5, 8, 62), (4097, 64, 13, 63),
                                                       (3000, 7, 16, 1000), (5000, 33, 3, 32_770)])
def test_tabulated_threshold_searches(B, oracle, n_req, n_search, n_steps, hi):
    print(f"tabulated searches: n_req={n_req} n_search={n_search} n_steps={n_steps} hi={hi}", flush=True)
    tr = DI.handmade_trace(170 + n_req, n_req, tokens=False)
    if n_req > 1000:
        tr["prompt_len"][::7] = np.arange(len(tr["prompt_len"][::7])) * 31 % 40_000
    total = int(tr["prompt_len"].sum(dtype=np.int64))
    which = ["server_prefill_tok", "device_prefill_tok"]
    specs = [dict(which_param=B.PARAM_L_TH, which_acc=which[j % 5 == 4], n_steps=n_steps, lo=j % 2 if hi else 0, hi=hi,
                  target=total * j / n_search) for j in range(n_search)]
    res = B.disco_budget_search(B.upload_trace(tr), DI.COST_S, [B.Policy(mode=0, mig_mode=1)] * n_search, specs)
    so = B.search_to_host(res["out"], n_search)
    pol = B.policies_to_host(res["pol_out"], n_search)
    for j, s in enumerate(specs):
        l_th, hp, ha = oracle.search_lth(tr, oracle.Policy(mode=0), s["lo"], hi, n_steps, s["which_acc"], DI.COST_S, s["target"])
        assert (pol[j].l_th, pol[j].mode, pol[j].mig_mode) == (l_th, 0, 1) and int(so["param"][j]) == l_th, j
        same_bits(so["hist_param"][j][:n_steps].astype(np.int32), hp, f"hist_param {j}")
        same_bits(so["hist_acc"][j][:n_steps], ha, f"hist_acc {j}")


# order statistics of buffer hand-offs: known hand-offs at the edges of chunks and tokens, with and without a token array;
# summaries found with other prices leave the selection to the general kernel (prices twice as high decide alike)
@pytest.mark.parametrize("n_req,tokens,max_out,stall_p", [(1, True, 2, 0.0), (300, True, 40, 0.2), (700, True, 1100, 0.02),
                                                          (257, False, 600, 0.0), (5000, True, 260, 0.1)])
def test_order_statistics_of_known_handoffs(B, oracle, n_req, tokens, max_out, stall_p):
    print(f"known hand-offs: n_req={n_req} tokens={tokens} max_out={max_out} stall_p={stall_p}", flush=True)
    tr = slow_prefill(DI.handmade_trace(260 + n_req, n_req, tokens=tokens, max_out=max_out, stall_p=stall_p), 16.0)
    for cost in (DI.COST_S, DI.COST_D):
        specs = [dict(mode=0, l_th=l, mig_mode=2) for l in (0, 12, 30)] + [dict(mode=1, l_th=-1, w_tail=DI.f32(w), mig_mode=2) for w in (0.0, 0.1, 0.3)]
        check_stats(B, oracle, tr, specs, cost, tau=DI.TAU, kappa=DI.KAPPA_LAG)
        dt, P = B.upload_trace(tr), len(specs)
        pols, ws = [B.Policy(**s) for s in specs], B.workspace(n_req, P)
        acc = B.disco_eval_dispatch(dt, pols, ws=ws)["acc"]
        B.disco_eval_migration(dt, DI.TAU, DI.KAPPA_LAG, pols, ws=ws, acc=acc, cost=cost)
        twice = dict(cost, cs_pre=2 * cost["cs_pre"], cs_dec=2 * cost["cs_dec"], lam=2 * cost["lam"])
        got = [B.disco_reduce_stats(dt, cost, pols, acc, ((50, 100), (99, 100)), tau=DI.TAU, kappa=DI.KAPPA_LAG, ws=ws, mig_cost=c,
                                    reuse_walk=True).clone() for c in (cost, twice)]
        same_bits(got[1].cpu().numpy(), got[0].cpu().numpy(), "records")


# order statistics outside the window of keys above the pacing interval: the selection starts over on raw keys, with wide
# digits where few classes are walked and with more than four prefixes in the end (histograms per slot)
@pytest.mark.parametrize("n_req,max_out,P", [(1500, 90, 2), (700, 400, 5), (3000, 30, 9)])
def test_order_statistics_on_raw_keys(B, oracle, n_req, max_out, P):
    print(f"raw keys: n_req={n_req} max_out={max_out} P={P}", flush=True)
    tr = DI.handmade_trace(520 + n_req, n_req, tokens=True, max_out=max_out, stall_p=0.1)
    specs = [dict(mode=0, l_th=0, mig_mode=2), dict(mode=0, l_th=1150), dict(mode=1, l_th=0, beta=DI.f32(1e-3), w_tail=0.0, mig_mode=1)]
    specs = (specs + [dict(mode=0, l_th=300 * j) for j in range(P)])[:P]
    check_stats(B, oracle, tr, specs, DI.COST_S, quantiles=((0, 100), (50, 100), (99, 100), (100, 100)), tau=DI.TAU, kappa=1.0)


# a law with a NaN parameter gives NaN times, as in the oracle's trace, and the check of the data reports them
@pytest.mark.parametrize("law,field", [("ttft_mu", "srv_ttft"), ("tbt_mu", "srv_tbt"), ("gap_mu", "tok_arr")])
def test_a_nan_law_is_not_hidden(B, oracle, law, field):
    print(f"NaN law: {law}", flush=True)
    gen = dict(DI.config(4, n_req=300, seed=5)["gen"], out_hi=90, gap_stall_p=0.1, **{law: float("nan")})
    want, got = oracle.gen_trace(gen), B.disco_gen_trace(gen)
    x, y = got.__dict__[field].cpu().numpy(), want[field]
    assert np.isnan(y).any() and (np.isnan(x) == np.isnan(y)).all()
    same_bits(x[~np.isnan(x)], y[~np.isnan(y)], field)
    assert B.disco_validate_trace(got) == B.ERR["range"]


# many wait searches at once: few steps on many requests take the fused passes, the others ten steps per pass
@pytest.mark.parametrize("n_req,n_search,n_steps", [(300_011, 10, 1), (300_011, 64, 3), (300_011, 64, 9), (900_001, 32, 4)])
def test_many_wait_searches(B, oracle, n_req, n_search, n_steps):
    print(f"many wait searches: n_req={n_req} n_search={n_search} n_steps={n_steps}", flush=True)
    tr = DI.handmade_trace(410, n_req, tokens=False)
    total = float(tr["prompt_len"].sum(dtype=np.int64))
    specs = [dict(which_param=B.PARAM_W_TAIL, which_acc="device_prefill_tok", n_steps=n_steps, lo=0.0, hi=4.0,
                  target=total * (j + 1) / (n_search + 2)) for j in range(n_search)]
    out = B.disco_budget_search(B.upload_trace(tr), DI.COST_D, [B.Policy(mode=1, l_th=j - 1) for j in range(n_search)], specs)
    so = B.search_to_host(out["out"], n_search)
    for j in range(0, n_search, 7):
        x, hp, ha = oracle.search_wait(tr, oracle.Policy(mode=1, l_th=j - 1), 0.0, 4.0, n_steps, "device_prefill_tok", DI.COST_D, specs[j]["target"])
        same_bits(so["hist_param"][j][:n_steps].astype(np.float32), hp, f"hist_param {j}")
        same_bits(so["hist_acc"][j][:n_steps], ha, f"hist_acc {j}")
        assert np.float32(so["param"][j]) == np.float32(x), j


# order statistics with reuse_walk at prices other than those of the summaries: those of a call that walks the tokens itself
@pytest.mark.parametrize("n_req,tokens,max_out", [(1, True, 9), (500, True, 700), (300, False, 300), (6000, True, 60)])
def test_order_statistics_at_other_prices(B, n_req, tokens, max_out):
    print(f"other prices: n_req={n_req} tokens={tokens} max_out={max_out}", flush=True)
    tr = slow_prefill(DI.handmade_trace(310 + n_req, n_req, tokens=tokens, max_out=max_out, stall_p=0.1), 16.0)
    specs = [dict(mode=0, l_th=l, mig_mode=2) for l in (0, 12, 30)] + [dict(mode=1, l_th=-1, w_tail=DI.f32(w), mig_mode=2) for w in (0.0, 0.1, 0.3)]
    specs.append(dict(mode=0, l_th=10, mig_mode=1))
    dt, P, pols = B.upload_trace(tr), len(specs), [B.Policy(**s) for s in specs]
    for cost in (DI.COST_S, DI.COST_D):
        moved = False
        for other in (None, dict(cost, cs_pre=9 * cost["cs_pre"], e_pre=9 * cost["e_pre"]), dict(cost, cs_dec=0.7 * cost["cs_dec"]),
                      DI.COST_D if cost is DI.COST_S else DI.COST_S):
            ws = B.workspace(n_req, P)
            acc = B.disco_eval_dispatch(dt, pols, ws=ws)["acc"]
            B.disco_eval_migration(dt, DI.TAU, DI.KAPPA_LAG, pols, ws=ws, acc=acc, cost=cost)
            args = dict(tau=DI.TAU, kappa=DI.KAPPA_LAG)
            q = ((50, 100), (99, 100))
            got = B.disco_reduce_stats(dt, cost, pols, acc, q, ws=ws, mig_cost=other, reuse_walk=True, **args)
            want = B.disco_reduce_stats(dt, cost, pols, acc, q, mig_cost=other, **args)
            same = B.disco_reduce_stats(dt, cost, pols, acc, q, mig_cost=cost, **args)
            moved = moved or not torch.equal(want, same)
            same_bits(got.cpu().numpy(), want.cpu().numpy(), f"records at {other}")
        assert moved or n_req == 1


# the generator's own division and square root are correctly rounded for every variate it can draw
def test_generator_division_and_square_root(B):
    print("generator division and square root, all variates", flush=True)
    f, q, x, r = B.disco_gen_math_probe().cpu().numpy()
    u = (np.arange(1 << 23, dtype=np.float64) + 0.5) * 2.0 ** -23
    e = np.round(np.log2(u / (1.0 + f.astype(np.float64))))
    assert (np.ldexp(1.0 + f.astype(np.float64), e.astype(int)) == u).all() and f.min() >= np.sqrt(0.5) - 1 - 1e-7 and f.max() <= np.sqrt(2.0) - 1 + 1e-7
    assert np.abs(x + 2.0 * np.log(u)).max() <= 4e-7 * 33 and (x > 0).all()        # |2 ln u| <= 33, a few units in its last place
    same_bits(q, f / (np.float32(2.0) + f), "f / (2 + f)")
    same_bits(r, np.sqrt(x), "sqrt(x)")


# traces of more than 2^32 - 1 tokens (18 GB of offsets), in each form of the generator: requests around token 2^32 and at
# both ends against the oracle, the whole array by the check of the data
@pytest.mark.parametrize("n_req,length", [(8191, 540_000), (32_767, 135_000), (65_600, 67_001)])
def test_more_than_2_to_the_32_tokens(B, oracle, n_req, length):
    print(f"wide token indices: n_req={n_req} length={length}", flush=True)
    gen = dict(DI.config(4, n_req=n_req, seed=3)["gen"], out_lo=length, out_hi=length)
    got = B.disco_gen_trace(gen)
    assert got.n_tok == n_req * length > 1 << 32
    off = np.arange(n_req + 1, dtype=np.int64) * length
    assert (got.tok_off.cpu().numpy() == off).all()
    at = (1 << 32) // length
    for i in (0, at - 1, at, at + 1, n_req - 1):
        same_bits(got.tok_arr[off[i]:off[i + 1]].cpu().numpy(), oracle.gen_tokens(gen, off, i, i + 1), f"tokens of request {i}")
    assert B.disco_validate_trace(got) == 0


# traces of up to 32 768 requests: a workgroup per policy column takes the searches, solves, totals and TTFT order
# statistics; the same calls with the grids shrunk go through the general kernels.  Keys of a few, of all and of no different
# bits, a wave, a workgroup and a batch of eight strides more or less than full
@pytest.mark.parametrize("n_req", [0, 1, 63, 1025, 8193, 20_011, 32_767, 32_768, 32_769])
@pytest.mark.parametrize("table", ["threshold", "wait", "mixed", "ties"])
def test_small_traces_against_the_general_kernels(B, n_req, table):
    print(f"small traces: n_req={n_req} table={table}", flush=True)
    tr = DI.handmade_trace(300 + n_req, n_req, tokens=False, ties=True)
    if table == "ties":                                      # two values of the TTFT in all
        tr["srv_ttft"][:] = np.where(np.arange(n_req) % 3, np.float32(0.5), np.float32(2.0))
    if n_req > 2:
        tr["prompt_len"][1], tr["prompt_len"][2] = 32_771, 40_000           # the last length of the table, one beyond it
    dt = B.upload_trace(tr)
    inf = float("inf")
    pols = {"threshold": [B.Policy(mode=0, l_th=x) for x in (0, 1, 150, 150, 700, 32_771, 50_000)],
            "wait": [B.Policy(mode=1, l_th=-1, w_tail=x) for x in (0.0, DI.f32(0.3), inf)] +
                    [B.Policy(mode=1, l_th=90, l_mid=120, w_mid=DI.f32(0.2), beta=DI.f32(1e-3), w_tail=DI.f32(0.9))],
            "ties": [B.Policy(mode=0, l_th=50_000), B.Policy(mode=0, l_th=0), B.Policy(mode=1, l_th=-1, w_tail=inf)],
            "mixed": [B.Policy(mode=0, l_th=200), B.Policy(mode=1, l_th=-1, w_tail=DI.f32(0.4)),
                      B.Policy(mode=2, beta=0.25, l_mid=3), B.Policy(mode=3, beta=0.5, l_mid=4)]}[table]
    P = len(pols)
    total = float(tr["prompt_len"].sum(dtype=np.int64))
    quantiles = ((0, 100), (1, 1000), (50, 100), (100, 100))
    ws = B.workspace(n_req, 64)

    def run():
        acc = torch.full((P * 128,), 0x5A, dtype=torch.uint8, device="cuda")
        B.disco_eval_dispatch(dt, pols, ws=ws, acc=acc)
        st = B.stats_to_host(B.disco_reduce_stats(dt, DI.COST_S, pols, acc, quantiles, ws=ws), P).copy()
        out = [B.accum_to_host(acc, P).copy(), st]
        for which in ("server_prefill_tok", "device_prefill_tok"):
            fr = (0.0, 0.13, 0.5, 0.77, 1.0)
            specs = [dict(which_param=B.PARAM_L_TH, which_acc=which, n_steps=17, lo=j, hi=32_770, target=f * total) for j, f in enumerate(fr)]
            found = torch.full((len(fr) * 128,), 0x5A, dtype=torch.uint8, device="cuda")
            r = B.disco_budget_search(dt, DI.COST_S, [B.Policy(mode=0, mig_mode=j % 3) for j in range(len(fr))], specs, ws=ws, acc=found)
            out += [B.search_to_host(r["out"], len(fr)).copy(), r["pol_out"].cpu().numpy(), B.accum_to_host(found, len(fr)).copy()]
        solve = [dict(mode=m, b=(b, 20), alpha=(1, 10), mig_mode=b % 3) for m in (0, 1) for b in (0, 1, 2, 7, 20)]
        r = B.disco_solve_policy(dt, solve, ws=ws)
        return out + [B.solve_to_host(r["out"], len(solve)).copy(), r["pol_out"].cpu().numpy()]

    def same(a, b, what):
        if a.dtype.names is None:
            if a.dtype == np.float64 and what in ("ttft_sum", "mean_ttft"):
                assert np.allclose(a, b, rtol=1e-12, atol=0, equal_nan=True), what       # fp64 sums in another order
            else:
                same_bits(a, b, what)
        else:
            for f in a.dtype.names:
                same(np.ascontiguousarray(a[f]), np.ascontiguousarray(b[f]), f)

    small = run()
    try:
        assert B._lib.disco_set_grid_divisor(2) == 0
        general = run()
    finally:
        assert B._lib.disco_set_grid_divisor(1) == 0
    for i, (a, b) in enumerate(zip(small, general)):
        same(a, b, f"result {i}")


# TBT order statistics: analytic timelines of a small trace are counted in device memory, those of one length once per wave;
# one more request than the small ones takes the counts in LDS; ranks that leave the window of keys start over on raw keys
@pytest.mark.parametrize("n_req,length,tau", [(1, 2, 0.2), (65, 37, 0.2), (1500, 1, 0.2), (2049, 4097, 0.2), (2049, 4096, 0.2), (3000, 0, 0.02), (32_769, 5, 0.2)])
def test_analytic_timelines_of_small_traces(B, oracle, n_req, length, tau):
    print(f"analytic timelines: n_req={n_req} length={length} tau={tau}", flush=True)
    tr = DI.handmade_trace(400 + n_req, n_req, tokens=False, max_out=60)
    if length:
        tr["output_len"][:] = length
        tr["output_len"][:: 7] = 3
        tr["tok_off"][1:] = np.cumsum(tr["output_len"])
        tr["n_tok"] = int(tr["tok_off"][-1])
    specs = [dict(mode=0, l_th=x, mig_mode=1) for x in (0, 400, 1500, 5000)] + [dict(mode=1, l_th=-1, w_tail=DI.f32(0.3), mig_mode=0)]
    check_stats(B, oracle, tr, specs, DI.COST_S, tau=DI.f32(tau), kappa=DI.KAPPA_LAG, quantiles=((1, 100), (50, 100), (99, 100)))


# token timelines of small traces: flags and exact walks in one launch, totals by column up to 16 384 requests and by workgroup
# beyond, every kind of hand-off; from 32 769 on the streaming walk
@pytest.mark.parametrize("n_req,max_out,tokens", [(0, 5, True), (1, 3, True), (3, 2100, True), (8195, 30, True), (16_384, 12, False), (16_385, 12, True),
                                                  (32_768, 6, False), (32_769, 6, True)])
def test_timelines_of_small_traces(B, oracle, n_req, max_out, tokens):
    print(f"timelines of small traces: n_req={n_req} max_out={max_out} tokens={tokens}", flush=True)
    tr = slow_prefill(DI.handmade_trace(500 + n_req, n_req, tokens=tokens, max_out=max_out, stall_p=0.05), 16.0)
    for mode in (0, 1):
        specs = [dict(mode=mode, l_th=x, w_tail=DI.f32(0.05 * j), mig_mode=j % 3) for j, x in enumerate((-1, 300, 900, 1500, 2900))]
        cost = DI.COST_D if mode else DI.COST_S
        check_migration(B, oracle, tr, specs, DI.TAU, DI.KAPPA_LAG, delivered_col=None, cost=cost)
        check_stats(B, oracle, tr, specs, cost, tau=DI.TAU, kappa=DI.KAPPA_LAG)


# small traces whose requests have more than 512 tokens on average: 1024 per iteration; lengths around its vectors and its ends, stalls
# (hand-offs) in every one of them
@pytest.mark.parametrize("n_req,stall_p", [(1, 0.0), (13, 0.004), (260, 0.001), (260, 0.05)])
def test_long_requests_of_small_traces(B, oracle, n_req, stall_p):
    print(f"long requests of small traces: n_req={n_req} stall_p={stall_p}", flush=True)
    tr = DI.handmade_trace(620 + n_req, n_req, tokens=False, max_out=3)
    n = np.array([1025, 255, 257, 513, 769, 1023, 1024, 2047, 2049, 3073, 4097, 1, 5000])[np.arange(n_req) % 13]
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    rng = np.random.default_rng(n_req)
    gap = rng.lognormal(-3.5, 0.6, int(off[-1])).astype(np.float32)
    stall = rng.random(len(gap)) < stall_p
    gap[stall] = rng.uniform(0.5, 400.0, int(stall.sum())).astype(np.float32)       # (some beyond what a reader of 5000 tokens has buffered)
    arr = np.zeros(len(gap), np.float32)
    for i in range(n_req):
        arr[off[i] + 1:off[i + 1]] = np.cumsum(gap[off[i] + 1:off[i + 1]], dtype=np.float32)
    assert off[-1] > 512 * n_req
    tr.update(n_tok=len(arr), output_len=n.astype(np.int32), tok_off=off, tok_arr=arr)
    tr = slow_prefill(tr, 16.0)
    for mode in (0, 1):
        specs = [dict(mode=mode, l_th=x, w_tail=DI.f32(0.05 * j), mig_mode=j % 3) for j, x in enumerate((-1, 300, 900, 1500, 2900))]
        cost = DI.COST_D if mode else DI.COST_S
        check_migration(B, oracle, tr, specs, DI.TAU, DI.KAPPA_LAG, delivered_col=None, cost=cost)
        check_stats(B, oracle, tr, specs, cost, tau=DI.TAU, kappa=DI.KAPPA_LAG)


# stretches of tokens that do not move the running maximum are counted by binade of the delivery: pacing intervals whose ratio to
# the spacing of the floats is an integer or not, maxima on and off half spacings, stretches over one to twenty binades, more
# of them in a request than wait together, stalls on both sides of a chunk's ends
@pytest.mark.parametrize("tau", [0.25, 0.2, 0.15, 0.1875, 3.0, 0.0009765625, 1.25e-4])
@pytest.mark.parametrize("every", [0, 255, 256, 512, 700])
def test_stretches_of_paced_tokens(B, oracle, tau, every):
    print(f"paced stretches: tau={tau} every={every}", flush=True)
    tau = DI.f32(tau)
    n = np.array([1, 2, 3, 255, 256, 257, 258, 511, 513, 1025, 3000, 5000, 17_001, 25_000])
    n_req = len(n)
    tr = DI.handmade_trace(600, n_req, tokens=True, max_out=2)
    tr["output_len"] = n.astype(np.int32)
    tr["prompt_len"][:] = 2000
    tr["srv_ttft"][:] = np.float32(0.1)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    arr = np.zeros(int(off[-1]), np.float32)
    for i in range(n_req):
        t = np.arange(n[i])
        late = 0.5 * tau * (1 + i) if i % 2 else 0.37 * tau + 0.01 * i          # a first move of the maximum, dyadic or not
        step = np.where(t >= 2, late, 0.0)
        if every:
            step = step + (t // every) * tau * every * (0.75 if i % 3 else 1.03) * (t >= every)
        arr[off[i]:off[i + 1]] = np.maximum.accumulate((t * (0.25 * tau) + step)).astype(np.float32)
        arr[off[i]] = 0.0
    tr.update(n_tok=len(arr), tok_off=off, tok_arr=arr)
    specs = [dict(mode=0, l_th=0, mig_mode=0), dict(mode=0, l_th=0, mig_mode=1), dict(mode=0, l_th=0, mig_mode=2), dict(mode=0, l_th=5000, mig_mode=0)]
    check_stats(B, oracle, tr, specs, DI.COST_S, tau=tau, kappa=1e6, quantiles=((1, 100), (50, 100), (90, 100), (999, 1000)))
    check_stats(B, oracle, tr, specs, DI.COST_S, tau=tau, kappa=DI.KAPPA_LAG, quantiles=((50, 100), (99, 100)))


# more gaps than the pools hold: timelines whose entries are taken back are walked in the passes, next to those that fit
def test_gaps_beyond_the_pools(B, oracle):
    print("gaps beyond the pools", flush=True)
    gen = dict(DI.config(4, n_req=600_000, seed=9)["gen"], out_mu=3.4, out_hi=60, gap_stall_p=0.3)
    tr = oracle.gen_trace(gen)
    assert tr["n_tok"] * 4 < 1 << 30
    specs = [dict(mode=0, l_th=0, mig_mode=0), dict(mode=0, l_th=0, mig_mode=1)]
    check_stats(B, oracle, tr, specs, DI.COST_S, tau=DI.TAU, kappa=DI.KAPPA_LAG)


# timelines of sources slower than the reader, which no pool holds: all of them walked in the passes, with every kind of hand-off,
# by more and fewer workgroups than there are classes, and (a few workgroups) by waves that stop trying to count their gaps
@pytest.mark.parametrize("n_req,max_out,tau,tokens,divisor", [(1, 40, 0.02, True, 1), (700, 300, 0.02, True, 1), (2500, 120, 0.05, False, 1),
                                                              (3100, 90, 0.01, True, 64), (33_001, 40, 0.03, True, 1), (33_001, 40, 0.03, True, 128)])
def test_sources_slower_than_the_reader(B, oracle, n_req, max_out, tau, tokens, divisor):
    print(f"slow sources: n_req={n_req} max_out={max_out} tau={tau} tokens={tokens} divisor={divisor}", flush=True)
    tr = slow_prefill(DI.handmade_trace(540 + n_req, n_req, tokens=tokens, max_out=max_out, stall_p=0.1), 16.0)
    if not tokens:
        tr["srv_tbt"] = (tr["srv_tbt"] * np.float32(4)).astype(np.float32)
    try:
        assert B._lib.disco_set_grid_divisor(divisor) == 0
        for mode in (0, 1):
            specs = [dict(mode=mode, l_th=x, w_tail=DI.f32(0.1 * j), mig_mode=(2, 1, 0, 2)[j]) for j, x in enumerate((-1, 16, 30, 40))]
            check_stats(B, oracle, tr, specs, DI.COST_D if mode else DI.COST_S, tau=DI.f32(tau), kappa=DI.KAPPA_LAG,
                        quantiles=((1, 100), (50, 100), (99, 100)))
    finally:
        assert B._lib.disco_set_grid_divisor(1) == 0


# the passes with two workgroups per CU begin at 2^18 requests: the gaps of as many and of one fewer, the last one of which has a
# single token and so no gap, have the same order statistics; sources slower and faster than the reader
@pytest.mark.parametrize("tau", [0.02, 0.1, 0.2])
def test_passes_of_many_requests(B, tau):
    print(f"passes of many requests: tau={tau}", flush=True)
    n = 1 << 18
    t = B.disco_gen_trace(dict(DI.config(4, n_req=n, seed=11)["gen"], out_hi=200))
    keep = int(t.tok_off[n - 1].item())
    t.output_len[n - 1] = 1
    t.tok_off[n] = keep + 1
    t.n_tok = keep + 1
    for table in ([dict(mode=0, l_th=x, mig_mode=m) for x, m in ((0, 1), (200, 2), (700, 0))],
                  [dict(mode=1, l_th=-1, w_tail=DI.f32(w), mig_mode=2) for w in (0.1, 0.4)]):
        pols = [B.Policy(**x) for x in table]
        P, got = len(pols), []
        for k in (n, n - 1):
            x = B.Trace(**{**{f: getattr(t, f) for f in ("prompt_len", "output_len", "srv_ttft", "srv_tbt", "dev_pre_spt", "dev_dec_spt", "tok_off", "tok_arr",
                                                        "dev_pre_spt_s", "dev_dec_spt_s", "dev_ttft_c")}, "n_req": k, "n_tok": keep + 1})
            ws = B.workspace(k, P)
            acc = B.disco_eval_dispatch(x, pols, ws=ws)["acc"]
            B.disco_eval_migration(x, DI.f32(tau), DI.KAPPA_LAG, pols, ws=ws, acc=acc, cost=DI.COST_D)
            got.append(B.stats_to_host(B.disco_reduce_stats(x, DI.COST_D, pols, acc, ((1, 100), (50, 100), (99, 100)), tau=DI.f32(tau), kappa=DI.KAPPA_LAG,
                                                            ws=ws, mig_cost=DI.COST_D, reuse_walk=True), P).copy())
        assert (got[0]["tbt_count"] == got[1]["tbt_count"]).all() and (got[0]["tbt_count"] > 0).all()
        for f in ("tbt_rank", "tbt_q"):
            same_bits(got[0][f], got[1][f], f)


# per-pair outputs: four requests per lane, rows that start anywhere, chunks of eight columns, next to the totals of small traces
# and of large ones
@pytest.mark.parametrize("n_req", [1, 2, 3, 5, 4095, 4097, 32_768, 32_769, 36_866])
@pytest.mark.parametrize("cols", [1, 8, 9, 17])
def test_per_pair_outputs(B, oracle, n_req, cols):
    print(f"per-pair outputs: n_req={n_req} cols={cols}", flush=True)
    tr = DI.handmade_trace(700 + n_req, n_req, tokens=False, ties=True)
    specs = [dict(mode=0, l_th=170 * j) if j % 4 < 2 else
             (dict(mode=1, l_th=100 * (j % 3), w_tail=DI.f32(0.07 * j)) if j % 4 == 2 else dict(mode=2 + j % 2, beta=DI.f32(0.1 + 0.05 * j), l_mid=j)) for j in range(cols)]
    check_dispatch(B, oracle, tr, specs)


# totals beside the per-pair outputs: by 96, 128 or 192 of their workgroups by the kind of the table, the others leave
@pytest.mark.parametrize("kind,cols", [("threshold", 1), ("threshold", 2), ("threshold", 5), ("wait", 3), ("stochastic", 1), ("stochastic", 3), ("all", 4)])
def test_totals_beside_per_pair_outputs(B, oracle, kind, cols):
    print(f"totals beside per-pair outputs: kind={kind} cols={cols}", flush=True)
    tr = DI.handmade_trace(720, 263_003, tokens=False, ties=True)
    of = {"threshold": lambda j: dict(mode=0, l_th=300 * j + 100), "wait": lambda j: dict(mode=1, l_th=100 * j, w_tail=DI.f32(0.2 * j)),
          "stochastic": lambda j: dict(mode=2 + j % 2, beta=DI.f32(0.2 + 0.2 * j), l_mid=j)}
    kinds = list(of) if kind == "all" else [kind]
    check_dispatch(B, oracle, tr, [of[kinds[j % len(kinds)]](j) for j in range(cols)])


# wait and slope searches behind their second pass: all steps in one launch (8192 requests, the last size, and one more), the rest
# from the list of the requests that still change (none, a few, some that all change at one wait) and further passes where that
# list is too long (all of them at one wait: already a workgroup's share); 16 000 of 40 003 at one wait: more than the walk holds in
# LDS, so that its rounds go over the list in device memory, and for a single search too long by its total alone; step counts
# at the ends of the passes
@pytest.mark.parametrize("n_req,same", [(8191, 0.4), (8192, 1.0), (8193, 0.0), (20_011, 0.4), (40_003, 1.0), (300_011, 0.0), (40_003, 0.4)])
@pytest.mark.parametrize("n_steps", [10, 11, 20, 21, 31, 64])
def test_searches_behind_the_second_pass(B, oracle, n_req, same, n_steps):
    print(f"searches behind the second pass: n_req={n_req} same={same} n_steps={n_steps}", flush=True)
    tr = DI.handmade_trace(700 + n_req, n_req, tokens=False, ties=False)
    at = np.arange(n_req) % 100 < 100 * same
    tr["srv_ttft"][at] = np.float32(0.7)
    total = float(tr["prompt_len"].sum(dtype=np.int64))
    below = float(tr["prompt_len"][tr["srv_ttft"] > np.float32(0.7)].sum(dtype=np.int64))
    middle = 0.5 * (below + float(tr["prompt_len"][tr["srv_ttft"] >= np.float32(0.7)].sum(dtype=np.int64)))
    searches = [  # template, parameter, accumulator, lo, hi, target
        (dict(mode=1, l_th=-1), B.PARAM_W_TAIL, "device_prefill_tok", 0.0, 4.0, middle),
        (dict(mode=1, l_th=60), B.PARAM_W_TAIL, "total_cost", 0.1, 3.0, 0.4 * DI.COST_D["cs_pre"] * total),
        (dict(mode=1, l_th=-1, w_tail=DI.f32(1.5)), B.PARAM_BETA, "device_prefill_tok", 0.0, 0.02, 0.3 * total),
    ]
    out = B.disco_budget_search(B.upload_trace(tr), DI.COST_D, [B.Policy(**s[0]) for s in searches],
                                [dict(which_param=p, which_acc=acc, n_steps=n_steps, lo=lo, hi=hi, target=target)
                                 for _, p, acc, lo, hi, target in searches])
    so = B.search_to_host(out["out"], len(searches))
    pol = B.policies_to_host(out["pol_out"], len(searches))
    alone = B.disco_budget_search(B.upload_trace(tr), DI.COST_D, [B.Policy(**searches[0][0])],       # (a shorter list)
                                  [dict(which_param=searches[0][1], which_acc=searches[0][2], n_steps=n_steps, lo=searches[0][3],
                                        hi=searches[0][4], target=searches[0][5])])
    same_bits(B.search_to_host(alone["out"], 1)["hist_acc"][0][:n_steps], so["hist_acc"][0][:n_steps], "one search")
    for j, (templ, p, acc, lo, hi, target) in enumerate(searches):
        find = oracle.search_wait if p == B.PARAM_W_TAIL else oracle.search_slope
        x, hp, ha = find(tr, oracle.Policy(**templ), lo, hi, n_steps, acc, DI.COST_D, target)
        same_bits(so["hist_param"][j][:n_steps].astype(np.float32), hp, f"hist_param {j}")
        same_bits(so["hist_acc"][j][:n_steps], ha, f"hist_acc {j}")
        got = pol[j].w_tail if p == B.PARAM_W_TAIL else pol[j].beta
        assert np.float32(got) == np.float32(x) == np.float32(so["param"][j]), j


# more than 2^32 requests: those that still change behind the second pass are the last ones.  All the others are over before the
# brackets begin and take no device, so that the histories are those of the same searches on the last ones alone
def test_searches_of_more_than_2_to_the_32_requests(B):
    n_req, tail, n_steps = (1 << 32) + 4099, 3001, 40
    print(f"searches of {n_req} requests", flush=True)
    rng = np.random.default_rng(32)
    few = dict(prompt_len=rng.integers(1, 4, tail).astype(np.int32), output_len=rng.integers(1, 300, tail).astype(np.int32),
               srv_ttft=rng.uniform(0.6, 7.4, tail).astype(np.float32))
    rest = dict(prompt_len=1, output_len=1, srv_ttft=0.25)

    def trace(n):
        arrays = {}
        for name, x in few.items():
            arrays[name] = torch.full((n,), rest[name], dtype=torch.float32 if name == "srv_ttft" else torch.int32, device="cuda")
            arrays[name][n - tail:] = torch.from_numpy(x).cuda()
        return B.Trace(n_req=n, n_tok=0, srv_tbt=None, dev_pre_spt=None, dev_dec_spt=None, tok_off=None, tok_arr=None,
                       dev_pre_spt_s=DI.f32(0.01), dev_dec_spt_s=DI.f32(0.05), dev_ttft_c=0.0, **arrays)

    templ = [dict(mode=1, l_th=-1), dict(mode=1, l_th=-1, w_tail=float("inf"))]
    specs = [dict(which_param=B.PARAM_W_TAIL, which_acc="device_prefill_tok", n_steps=n_steps, lo=0.5, hi=8.0, target=2500.0),
             dict(which_param=B.PARAM_BETA, which_acc="device_cost", n_steps=n_steps, lo=0.5, hi=8.0, target=1000 * DI.COST_D["lam"] * DI.COST_D["e_pre"])]
    res = []
    for n in (tail, n_req):
        t = trace(n)
        assert t.srv_ttft.numel() == n
        out = B.disco_budget_search(t, DI.COST_D, [B.Policy(**x) for x in templ], specs, ws=B.workspace(0, 2))
        res.append(B.search_to_host(out["out"], 2).copy())
        del t, out
    torch.cuda.empty_cache()
    alone, among = res
    for f in ("hist_param", "hist_acc", "param", "acc_at_param", "lo", "hi"):
        same_bits(among[f], alone[f], f)
    for f in ("d_pre", "d_dec", "n_dev_started", "n_dev_win"):
        assert (among["at_param"][f] == alone["at_param"][f]).all(), f
    assert (among["at_param"]["s_pre"] == int(few["prompt_len"].sum()) + n_req - tail).all()


# tables of threshold columns from their sorted thresholds (workgroups with more than one batch per wave: one workgroup here): the
# fewest and most columns of each width, thresholds below, between, at and above all lengths, equal ones, lengths and tokens
# beyond 2^24, server TTFTs of infinity, arrays on and off 16-byte boundaries, pairs beside the totals
@pytest.mark.parametrize("n_req,P,shift", [(1025, 64, 0), (1030, 33, 1), (5003, 64, 2), (2049, 16, 0), (4097, 5, 3), (20_011, 8, 0), (4098, 3, 0)])
@pytest.mark.parametrize("equal", [False, True])
def test_threshold_tables_by_bucket(B, oracle, n_req, P, shift, equal):
    print(f"threshold buckets: n_req={n_req} P={P} shift={shift} equal={equal}", flush=True)
    tr = DI.handmade_trace(800 + n_req, n_req, tokens=False, ties=True)
    tr["srv_ttft"][5] = np.inf
    tr["prompt_len"][7], tr["prompt_len"][n_req - 1] = (1 << 24) + 5, 2**31 - 1
    tr["output_len"][9] = (1 << 24) + 7
    at = np.sort(tr["prompt_len"])[np.arange(P) * n_req // P]
    th = np.full(P, at[P // 2]) if equal else np.random.default_rng(P).permutation(at + np.arange(P) % 2)
    th = [int(x) for x in th]
    if not equal:
        th[0], th[P - 1], th[P // 2] = -5, 2**31 - 1, 0
    specs = [dict(mode=0, l_th=x) for x in th]
    try:
        assert B._lib.disco_set_grid_divisor(64) == 0
        dt, acc = check_dispatch(B, oracle, tr, specs)
        check_dispatch(B, oracle, tr, specs, materialise=False)
        for name in ("prompt_len", "output_len", "srv_ttft", "dev_pre_spt"):
            x = getattr(dt, name)
            buf = torch.zeros(x.numel() + shift, dtype=x.dtype, device="cuda")[shift:]
            buf.copy_(x)
            setattr(dt, name, buf)
        moved = B.accum_to_host(B.disco_eval_dispatch(dt, [B.Policy(**s) for s in specs])["acc"], P)
        torch.cuda.synchronize()
    finally:
        assert B._lib.disco_set_grid_divisor(1) == 0
    for f in ("s_pre", "s_dec", "d_pre", "d_dec", "n_dev_started", "n_dev_win", "ttft_min_bits", "ttft_max_bits"):
        assert (moved[f] == acc[f]).all(), f
    assert np.allclose(moved["ttft_sum"], acc["ttft_sum"], rtol=1e-12, atol=0)       # fp64 sums in another order
