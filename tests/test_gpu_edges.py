"""Kernels whose work split depends on the size of their input, at the sizes where one form gives way to the next and
at the remainders of their tiles, against the CPU oracle (bit for bit unless a test says otherwise)."""
import numpy as np
import pytest
import torch

import disco_inputs as DI

pytestmark = pytest.mark.gpu


def same_bits(got, want, what):
    got, want = np.ascontiguousarray(got), np.ascontiguousarray(want)
    assert got.shape == want.shape, what
    bad = np.flatnonzero(got.view(np.uint8).ravel() != want.view(np.uint8).ravel())
    assert bad.size == 0, f"{what}: {bad.size} bytes differ, first at {bad[:5]}"


# requests per wave of the token generator: 1 below 8192 requests, 4 below 32768, then 16; pieces of 64, 256 and 1024
# tokens from multiples of 32 on; the stall test at both ends of its range
@pytest.mark.parametrize("n_req,out_mu,out_hi,stall_p", [
    (1, 6.0, 1100, 0.01), (15, 6.5, 2100, 0.5), (8191, 3.0, 70, 0.01), (8192, 4.5, 600, 0.0), (8195, 3.5, 300, 1.0),
    (32767, 3.0, 65, 0.01), (32768, 3.5, 130, 0.01), (32785, 3.5, 97, 0.25)])
def test_generated_tokens(B, oracle, n_req, out_mu, out_hi, stall_p):
    print(f"generated tokens: n_req={n_req} out_mu={out_mu} out_hi={out_hi} stall_p={stall_p}", flush=True)
    gen = dict(DI.config(4, n_req=n_req, seed=n_req)["gen"], out_mu=out_mu, out_hi=out_hi, gap_stall_p=stall_p)
    want = oracle.gen_trace(gen)
    got = B.disco_gen_trace(gen)
    assert got.n_tok == want["n_tok"]
    same_bits(got.tok_off.cpu().numpy(), want["tok_off"], "tok_off")
    same_bits(got.tok_arr.cpu().numpy(), want["tok_arr"], "tok_arr")
