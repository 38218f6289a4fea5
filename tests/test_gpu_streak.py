"""Runs of repeated iterations applied in one pass: parity with the oracle
where a run can end or must not start.

Each case puts one event on the edges of a run: completions, level crossings
(alone and together with a completion), arrivals at the very end of an
iteration, KV budgets that the next blocks just fill, iteration costs and
context sums past the pass's 32-bit range, the iteration limit, LTR+
promotions and demotions, and the grid changes of adaptive gamma. All results
are whole numbers (and gamma, compared by its bits): equality is exact.
"""
import numpy as np
import pytest

import oracle
from paper_2606_18431_amd import workloads as W
from test_gpu_parity import assert_parity, edge_workload, gpu_run, torch  # noqa: F401

pytestmark = pytest.mark.gpu

ADA = dict(W.ADA, window=16, min_samples=4, beta=0.3)
POLICIES = [W.setting(0, W.FCFS), W.setting(0, W.SRPT), W.setting(0, W.LAS), W.setting(0, W.TRAIL),
            W.setting(0, W.BOOST, gamma=1e-3, **W.UNIBOOST),
            W.setting(0, W.BOOST, gamma=1e-3, k=3, memguard=1, delta_us=5000),
            W.setting(0, W.BOOST, gamma=1e-3, **W.VANILLA),
            W.setting(0, W.DIST, gamma=1e-3), W.setting(0, W.SARATHI),
            W.setting(0, W.BOOST, gamma=1e-3, signal=1, **W.VANILLA),
            W.setting(0, W.BOOST, gamma=1e-3, signal=2, **W.VANILLA),
            W.setting(0, W.BOOST, gamma=1e-3, ada=ADA, **W.VANILLA)]
LTR = [W.setting(0, W.LTR, ltr=(5, 3)), W.setting(0, W.LTR, ltr=(1, 1)),
       W.setting(0, W.LTR, ltr=(200, 70))]

ENGINES = {
    # nothing waits: runs of 64, through completions and crossings
    "roomy": (W.Engine(), 8.0),
    # one step's cost takes all of the clock: every run ends at an arrival
    "slow steps": (W.Engine(iter_base_us=400_000, max_seqs=48), 4.0),
    # full batches: waiting requests behind the last member
    "sequence cap": (W.Engine(max_seqs=6), 60.0),
    # admissions closed by a waiting request that does not fit
    "kv": (W.Engine(max_seqs=24, kv_blocks=70, chunk=64, max_tokens=200), 60.0),
    "kv, one-token blocks": (W.Engine(max_seqs=24, kv_blocks=900, block_tokens=1, chunk=64,
                                      max_tokens=100), 60.0),
    "kv, 24-token blocks": (W.Engine(max_seqs=24, kv_blocks=50, block_tokens=24, chunk=50,
                                     max_tokens=128), 60.0),
    # the batch fills the token budget exactly
    "token budget": (W.Engine(max_seqs=8, max_tokens=8, chunk=8, kv_blocks=400), 30.0),
    # several chunks of members
    "wide": (W.Engine(max_seqs=200, kv_blocks=1500), 120.0),
    # the context sum itself in the cost
    "unit divisor": (W.Engine(iter_ctx_div=1, max_seqs=32, kv_blocks=300), 10.0),
}


@pytest.mark.parametrize("ltr", [False, True], ids=["policies", "ltr"])
@pytest.mark.parametrize("name", list(ENGINES))
def test_runs_end_where_they_must(torch, name, ltr):  # noqa: F811
    e, rate = ENGINES[name]
    a, p, d = W.small_random(31, 150, rate_per_s=rate, d_med=40, d_max=400)
    w = edge_workload(a, p, d, e, LTR if ltr else POLICIES)
    o = oracle.run(w)
    g = gpu_run(w)
    assert np.array_equal(g["status"], o["status"])
    assert_parity(w, g, o, inst=np.nonzero(o["status"] == 0)[0])
    assert np.array_equal(g["gamma"].view(np.int64), o["gamma"].view(np.int64))
    assert np.array_equal(g["switches"], o["switches"])


@pytest.mark.parametrize("base,P,div", [((1 << 24) - 33, 30, 1 << 20), ((1 << 24) + 5, 30, 7),
                                        (5000, 1_150_000, 1), (5000, 1_100_000, 1)])
def test_costs_past_the_pass(torch, base, P, div):  # noqa: F811
    """Iterations of 2^24 us and more, by the base cost or by a context sum
    in units of one token (15 contexts just above and just below 2^24 / 15),
    take the ordinary path."""
    n = 15
    e = W.Engine(iter_base_us=base, max_seqs=n, iter_tok_us=1 if P < 100 else 0, iter_ctx_div=div,
                 chunk=32767, max_tokens=n * 32767, kv_blocks=n * (P // 16 + 8))
    w = edge_workload(np.arange(n), np.full(n, P), 40 + np.arange(n), e, POLICIES)
    o = oracle.run(w)
    assert np.all(o["status"] == 0)
    assert_parity(w, gpu_run(w), o)


@pytest.mark.parametrize("shift", [-1, 0, 1])
@pytest.mark.parametrize("step", [1, 2, 63, 64, 65, 130])
def test_arrival_at_the_end_of_an_iteration(torch, step, shift):  # noqa: F811
    """Three requests decode alone (the cost of every iteration is known);
    a fourth arrives `shift` us from the end of the `step`-th repeated one."""
    e = W.Engine(max_seqs=8, iter_ctx_div=7)
    P, D = 32, 400
    t = e.iter_base_us + e.iter_tok_us * 3 * P + 3 * P // e.iter_ctx_div
    for j in range(1, step + 1):
        t += e.iter_base_us + e.iter_tok_us * 3 + 3 * (P + j) // e.iter_ctx_div
    w = edge_workload([0, 0, 0, t + shift], [P, P, P, 50], [D, D, D - 7, 30], e, POLICIES)
    o = oracle.run(w)
    assert_parity(w, gpu_run(w), o)


@pytest.mark.parametrize("limit", [40, 41, 104, 105, 168, 169, 400])
def test_iteration_limit_inside_a_run(torch, limit):  # noqa: F811
    """The limit ends an instance at the same iteration, run or not."""
    w = edge_workload([0, 0], [16, 40], [limit, limit - 3], W.Engine(max_iters=limit), POLICIES)
    o = oracle.run(w)
    assert np.all(o["status"] == 0)
    assert_parity(w, gpu_run(w), o)
    w = edge_workload([0, 0], [16, 40], [limit + 1, limit], W.Engine(max_iters=limit), POLICIES)
    assert np.array_equal(gpu_run(w)["status"], oracle.run(w)["status"])


@pytest.mark.parametrize("D", [3, 4, 5, 6, 7, 250, 251, 253, 254, 255, 509, 510, 511])
def test_crossing_beside_completion(torch, D):  # noqa: F811
    """Level thresholds k 2^j at and around the last token, and two requests
    that cross in the same iteration while a third waits."""
    e = W.Engine(max_seqs=3, kv_blocks=80)
    w = edge_workload([0, 0, 10, 20], [2, 2, 9, 3], [D, D + 1, D, 12], e, POLICIES)
    o = oracle.run(w)
    assert_parity(w, gpu_run(w), o)


def assert_gamma(g, o):
    assert np.array_equal(g["gamma"].view(np.int64), o["gamma"].view(np.int64)), (g["gamma"], o["gamma"])
    assert np.array_equal(g["switches"], o["switches"])


def crossing_before_completions(ahead):
    """Two requests complete in one iteration; the older one crossed a level
    `ahead` iterations before, which moved it behind the other in the batch."""
    e = W.Engine(iter_ctx_div=1_000_000, iter_tok_us=0)  # 5 ms an iteration
    DA, later = 200, 20
    arr, P, D = [0, later * 5000], [512 - (DA - ahead), 100], [DA, DA - later]
    for i in range(21):  # then one at a time; the last one decodes on as the window has dropped one
        arr.append(DA * 5000 + 1000 + 100_000 * i)
        P.append(16)
        D.append(90 if i == 20 else 2 + i % 3)
    ada = dict(W.ADA, window=21, min_samples=20, beta=0.3)
    return edge_workload(arr, P, D, e,
                         [W.setting(0, W.BOOST, gamma=1e-3, ada=dict(ada, window=n), **W.UNIBOOST)
                          for n in (20, 21, 22)])


@pytest.mark.parametrize("ahead", [0, 1, 2, 20, 63, 64, 65, 130])
def test_two_completions_after_a_crossing(torch, ahead):  # noqa: F811
    """Their latencies enter gamma's window in batch order, and a window that
    is full later drops the one that entered first: with 21 latencies the
    largest or the second largest, so that gamma differs by the order."""
    w = crossing_before_completions(ahead)
    o = oracle.run(w)
    done = w.arrival_us[0] + o["ttlt"]
    assert np.all(done[:, 0] == done[:, 1])
    g = gpu_run(w)
    assert_parity(w, g, o)
    assert_gamma(g, o)


def bursts(seed, burst, longest):
    """Bursts of requests that arrive apart and complete together, on every
    80th iteration, after level crossings in quiet stretches."""
    rng = np.random.default_rng(seed)
    n = 500
    m = np.sort(np.concatenate([400 * b + rng.integers(0, 60, burst) for b in range(n // burst)]))
    D = 80 * ((m + rng.integers(30, 300, n)) // 80 + 1) - m
    e = W.Engine(iter_ctx_div=1_000_000, iter_tok_us=0, max_seqs=300, kv_blocks=100_000)
    sets = [W.setting(0, W.BOOST, gamma=g0, ada=dict(W.ADA, window=k, min_samples=k // 2 + 1, beta=b),
                      **kw)
            for g0 in (1e-4, 1e-2) for k, b in ((21, 0.05), (33, 0.3), (100, 1.0))
            for kw in (W.UNIBOOST, W.VANILLA, dict(k=7, signal=1))]
    return edge_workload(m * 5000, rng.integers(1, longest, n), D, e, sets)


@pytest.mark.parametrize("seed,burst,longest", [(24, 25, 200), (12, 10, 600), (6, 50, 100)])
def test_many_completions_at_once(torch, seed, burst, longest):  # noqa: F811
    """Several latencies enter small windows at once, all the time."""
    w = bursts(seed, burst, longest)
    o = oracle.run(w)
    assert np.all(o["status"] == 0) and np.all(o["switches"] > 0)
    g = gpu_run(w)
    assert_parity(w, g, o)
    assert_gamma(g, o)


@pytest.mark.parametrize("engine", [
    W.Engine(max_seqs=64, max_tokens=65, chunk=65, kv_blocks=26),
    W.Engine(max_seqs=64, max_tokens=66, chunk=66, kv_blocks=26),
    W.Engine(max_seqs=64, max_tokens=67, chunk=66, kv_blocks=26),
])
def test_protected_member_passes_a_clipped_prefill(torch, engine):  # noqa: F811
    """TRAIL: a waiting prefill that takes the whole token budget does not
    fit; the only resident, which its progress protects, ranks behind it.
    Once the resident has fewer tokens left it ranks before the prefill and
    takes a token of the budget: the prefill's chunk shrinks by one, where
    that crosses a block boundary it fits."""
    w = edge_workload([0, 1_621_098], [16, 66], [400, 5], engine,
                      [W.setting(0, W.TRAIL), W.setting(0, W.SRPT), W.setting(0, W.LAS)])
    o = oracle.run(w)
    assert_parity(w, gpu_run(w), o)


def tight_budgets(tokens, bs, sets):
    """The token budget clips the prefill at which the KV budget closes
    admissions, all the time."""
    a, p, d = W.small_random(61, 300, rate_per_s=60.0, p_med=90, d_med=60, p_max=700, d_max=400)
    e = W.Engine(max_seqs=32, max_tokens=tokens, chunk=tokens, block_tokens=bs, max_iters=20_000,
                 kv_blocks=1200 // bs)
    return edge_workload(a, p, d, e, sets)


@pytest.mark.parametrize("extended", [False, True], ids=["fixed", "extended"])
@pytest.mark.parametrize("bs", [1, 16, 24])
@pytest.mark.parametrize("tokens", [40, 64, 200])
def test_token_and_kv_budget_bind(torch, tokens, bs, extended):  # noqa: F811
    w = tight_budgets(tokens, bs, POLICIES + LTR if extended else POLICIES[:7])
    o = oracle.run(w)
    assert np.any(o["counters"][:, 3:5] > 0)  # evictions: the KV budget binds
    g = gpu_run(w)
    assert np.array_equal(g["status"], o["status"])
    assert_parity(w, g, o, inst=np.nonzero(o["status"] == 0)[0])


@pytest.mark.parametrize("n", [127, 130, 260])
@pytest.mark.parametrize("D", [1, 3])
def test_contexts_released_together_past_31_bits(torch, D, n):  # noqa: F811
    """n requests of nearly 2^24 tokens complete in one iteration (D = 1: at
    their first token, D = 3: at the end of a run): the context they release
    passes 2^31, or 2^32. A small one decodes on, at the context's cost."""
    P = (1 << 24) - 8
    e = W.Engine(iter_base_us=1000, iter_tok_us=0, iter_ctx_div=1 << 20, max_seqs=n + 1,
                 chunk=32767, max_tokens=(n + 1) * 32767, kv_blocks=(n + 1) << 20)
    w = edge_workload(np.zeros(n + 1), [P] * n + [40], [D] * n + [700], e, POLICIES)
    o = oracle.run(w)
    assert np.all(o["status"] == 0)
    assert len(set(o["ttlt"][0][:n])) == 1
    g = gpu_run(w)
    assert_parity(w, g, o)
