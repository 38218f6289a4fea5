"""Batch formation where the KV budget stops a chunk of 64 candidates: parity
with the oracle around the rule that counts lanes instead of summing.

The rule holds up to the first candidate that computes more than a token, and
only where the sequence and the token budget do not end the batch before the
candidate that does not fit. The engines put each of those limits at and
around that candidate: whole prompts in one chunk (the candidate is the first
or a later one of several), chunks of one token (every lane counts), a token
budget that clips it, a sequence cap that it reaches, blocks of one token and
of sizes that are no power of two, and batches of several chunks. Results are
whole numbers: equality is exact.
"""
import numpy as np
import pytest

import oracle
from paper_2606_18431_amd import workloads as W
from test_gpu_parity import assert_parity, edge_workload, gpu_run, torch  # noqa: F401

pytestmark = pytest.mark.gpu

POLICIES = [W.setting(0, W.FCFS), W.setting(0, W.SRPT), W.setting(0, W.TRAIL),
            W.setting(0, W.BOOST, gamma=1e-3, **W.UNIBOOST),
            W.setting(0, W.BOOST, gamma=1e-3, **W.VANILLA)]
EXTENDED = POLICIES + [W.setting(0, W.SARATHI)]
ENGINES = {
    "prompt in one chunk": W.Engine(max_seqs=64, kv_blocks=90, chunk=4096, max_tokens=8192),
    "chunks of one token": W.Engine(max_seqs=64, kv_blocks=90, chunk=1, max_tokens=64),
    "one-token blocks": W.Engine(max_seqs=100, kv_blocks=1100, block_tokens=1, chunk=64,
                                 max_tokens=300),
    "24-token blocks": W.Engine(max_seqs=64, kv_blocks=60, block_tokens=24, chunk=100,
                                max_tokens=1000),
    "token budget clips": W.Engine(max_seqs=64, kv_blocks=90, chunk=60, max_tokens=61),
    "sequence cap": W.Engine(max_seqs=7, kv_blocks=60, chunk=512, max_tokens=600),
    "several chunks": W.Engine(max_seqs=256, kv_blocks=500, chunk=256, max_tokens=2048),
}


@pytest.mark.parametrize("policies", [POLICIES, EXTENDED], ids=["fixed", "extended"])
@pytest.mark.parametrize("p_med", [4, 40])
@pytest.mark.parametrize("name", list(ENGINES))
def test_kv_budget_stops_a_chunk(torch, name, p_med, policies):  # noqa: F811
    a, p, d = W.small_random(47, 300, rate_per_s=400.0, p_med=p_med, d_med=60, p_max=500,
                             d_max=400)
    w = edge_workload(a, p, d, ENGINES[name], policies)
    o = oracle.run(w)
    assert np.all(o["status"] == 0)
    assert np.any(o["counters"][:, 3:5] > 0)  # evictions: the budget binds
    assert_parity(w, gpu_run(w), o)
