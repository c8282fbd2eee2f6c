"""Parity of the scheduler's pool pass (one queued call per lane) with the oracle at the
edges of its capacities: 64 calls, 64 users, spilled first calls up to millions of one user,
chains whose next call waits, ties of zero-cost calls, keys too far apart for one order word,
and the hand-over to the slot pass and back; in one call and in slices."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_15997_amd as fs
from gpu_common import compare_sim, gpu_schedule, say
from tiny import random_trace
import tracegen as tg

pytestmark = pytest.mark.gpu


def _check(tr, cost, reason, step, cap, theta, chunks):
    o = oracle.simulate(tr, cost, reason, step, cap, theta)
    compare_sim(gpu_schedule(tr, cost, reason, step, cap, theta), o)
    compare_sim(gpu_schedule(tr, cost, reason, step, cap, theta, chunks=chunks), o)


@pytest.mark.parametrize("multi", [False, True])
@pytest.mark.parametrize("users,cap,theta", [(3, 20, 10 ** 9), (40, 25, 300), (63, 60, 10 ** 9),
                                             (64, 30, 500), (66, 45, 10 ** 9), (130, 25, 10 ** 9),
                                             (200_000, 30, 400)])
def test_pool_edges(users, cap, theta, multi):
    """Backlogs of a few users with long queues up to more users than lanes."""
    rng = np.random.default_rng(users * 2 + multi)
    say("pool edges", users, cap, theta, multi)
    tr = tg.concat([random_trace(rng, 1500, users, 2, 4000, multi=multi, max_tok=8) for _ in range(3)])
    for most in (2, 5000, 1 << 39):   # ties, plain, far-apart keys
        cost = rng.integers(0, most, tr.n).astype(np.int64)
        reason = rng.integers(0, 3, tr.n).astype(np.uint8)
        _check(tr, cost, reason, 50, cap, theta, 23)


@pytest.mark.parametrize("multi", [False, True])
@pytest.mark.parametrize("replicas,n", [(1, 20_000), (800, 60), (1, 300)])
def test_pool_spilled_calls(replicas, n, multi):
    """A queue longer than the pool: its tail is spilled, up to thousands of calls of a user."""
    rng = np.random.default_rng(n + multi)
    say("pool spill", replicas, n, multi)
    tr = tg.concat([random_trace(rng, n, 2, 2, n // 2 + 1, multi=multi, max_tok=8)
                    for _ in range(replicas)])
    cost = rng.integers(0, 4000, tr.n).astype(np.int64)
    reason = np.zeros(tr.n, np.uint8)
    _check(tr, cost, reason, 10, 30, 10 ** 9, 400)


def test_pool_outgrown_and_taken_back():
    """Bursts of more users than lanes between quiet stretches: the replica changes passes
    and comes back; users are lifted, throttled and chained across the changes."""
    rng = np.random.default_rng(9)
    tr = random_trace(rng, 6000, 150, 2, 100, multi=True, max_tok=6)
    tr.ts_us = np.sort(np.concatenate([np.full(120, b * 40_000) + rng.integers(0, 600, 120)
                                       for b in range(50)])).astype(np.int64)
    cost = rng.integers(0, 900, tr.n).astype(np.int64)
    reason = rng.integers(0, 3, tr.n).astype(np.uint8)
    for theta in (10 ** 9, 200, -1):
        say("pool taken back", theta)
        _check(tr, cost, reason, 100, 12, theta, 301)


@pytest.mark.parametrize("length", [20, 80])
def test_pool_long_drain_of_chains(length):
    """More than 2^32 tokens admitted between two rankings of the pool, while some of its
    calls are outside the ranking: 12 chains whose calls have all arrived (each admitted call
    makes the next one ready, which takes its rank in place) over 41 queued first calls.  A
    step admits one or two calls of up to 2^24 - 1 tokens; the second ranking, after a full one
    and new arrivals, leaves the first calls out."""
    rng = np.random.default_rng(length)
    chains, plain, C = 12, 41, 3 << 22
    rows = [(0, u, 0, 10) for u in range(chains)]  # (step, user, call, tokens); admitted in step 0
    rows += [(1, chains + k, 0, 1000 + k) for k in range(plain - 1)]
    rows += [(1, u, 1, int(rng.integers(1 << 23, 1 << 24))) for u in range(chains)]
    rows += [(2, chains + plain - 1, 0, 1000)]
    rows += [(2, u, c, int(rng.integers(1 << 23, 1 << 24))) for c in range(2, length) for u in range(chains)]
    at = {}
    n = len(rows)
    user, call, tok, ts = (np.zeros(n, np.int32) for _ in range(4))
    head, prev = np.arange(n, dtype=np.int32), np.full(n, -1, np.int32)
    for i, (step, u, c, t) in enumerate(rows):
        user[i], call[i], tok[i], ts[i] = u, c, t, step * 10
        if c > 0:
            head[i], prev[i] = at[u, 0], at[u, c - 1]
        at[u, c] = i
    z = np.zeros(n, np.int32)
    tr = tg.Trace(1, chains + plain, 1, np.array([0, n], np.int64), ts.astype(np.int64), user, z.copy(),
                  call, head, prev, tok, None, z.copy())
    cost = rng.integers(1, 900, n).astype(np.int64)
    say("pool long drain", length)
    _check(tr, cost, np.zeros(n, np.uint8), 10, C, 10 ** 12, 301)


def _burst(queued):
    """Every request arrives at once: `queued` calls of user 0, four calls each of 60 others
    (they fill the pool, so that user 0's pooled calls are spilled as well), 50 of user 0."""
    rng = np.random.default_rng(queued)
    user = np.concatenate([np.zeros(queued, np.int32), np.tile(np.arange(1, 61, dtype=np.int32), 4),
                           np.zeros(50, np.int32)])
    n = user.size
    z = np.zeros(n, np.int32)
    tr = tg.Trace(1, 61, 1, np.array([0, n], np.int64), np.zeros(n, np.int64), user, z, None, None, None,
                  rng.integers(0, 8, n).astype(np.int32), None, z)
    return tr, rng.integers(0, 4000, n).astype(np.int64)


def _burst_reference(tr, cost, cap):
    """Admission order, step and counter after each call of such a burst in closed form: the
    least counter is always served next, so the order is that of (counter before the call,
    user, position), and the call with t tokens admitted before it is admitted in step t // cap
    (overshoot is carried as debt).  (The oracle takes 25 s for 2^24 queued calls of one user.)"""
    n = tr.n
    after = np.zeros(n, np.int64)
    for u in range(tr.n_users):
        m = tr.user == u
        after[m] = np.cumsum(cost[m])
    order = np.lexsort((tr.user, after - cost))  # (stable: a user's calls stay in order)
    seq, step = np.zeros(n, np.int32), np.zeros(n, np.int32)
    seq[order] = np.arange(n)
    before = np.cumsum(tr.len_in[order].astype(np.int64)) - tr.len_in[order]
    step[order] = before // cap
    return seq, step, after


@pytest.mark.parametrize("queued,sliced", [(3000, True), ((1 << 23) + 100, True), ((1 << 24) + 100, False)])
def test_pool_many_spilled_calls_of_one_user(queued, sliced):
    """2^23 and 2^24 queued calls of one user: their order holds while the queue grows, while it
    is rebuilt by a second call, and while it drains."""
    tr, cost = _burst(queued)
    cap = 4096 if queued < 10_000 else 1 << 20
    seq, step, after = _burst_reference(tr, cost, cap)
    if queued < 10_000:  # the closed form is the oracle's schedule
        o = oracle.simulate(tr, cost, None, 10, cap, 10 ** 12)
        assert (o.admit_seq == seq).all() and (o.admit_step == step).all() and (o.counter_after == after).all()
    say("pool many spilled", queued, sliced)
    dt = fs.DeviceTrace(tr)
    c, eng, out, st = torch.as_tensor(cost).cuda(), fs.make_engine(10, cap, 10 ** 12), fs.Outputs(dt), fs.fs_state_init(dt)
    for n_steps in ((1, -1) if sliced else (-1,)):
        fs.fs_schedule_step(dt, st, c, None, eng, out, n_steps)
        say("steps so far", int(out.steps[0]))
    h = out.host()
    assert (h["status"] == 0).all()
    for k, want in (("admit_seq", seq), ("admit_step", step), ("counter_after", after)):
        bad = np.nonzero(h[k] != want)[0]
        assert bad.size == 0, (k, bad.size, bad[:5], h[k][bad[:5]], want[bad[:5]])


@pytest.mark.parametrize("users,cap", [(20, 12), (45, 20), (90, 14)])
def test_pool_deep_queues_of_chains(users, cap):
    """Overloads long enough that a replica's queue of chained calls is handed to the slot pass,
    and quiet stretches in which the pool takes it back; with more users than lanes as well."""
    rng = np.random.default_rng(users)
    say("pool deep chains", users, cap)
    trs = []
    for _ in range(3):
        tr = random_trace(rng, 9000, users, 2, 100, multi=True, max_tok=6)
        tr.ts_us = np.sort(np.concatenate([b * 600_000 + rng.integers(0, 40_000, 3000) for b in range(3)])).astype(np.int64)
        trs.append(tr)
    tr = tg.concat(trs)
    cost = rng.integers(0, 900, tr.n).astype(np.int64)
    reason = rng.integers(0, 3, tr.n).astype(np.uint8)
    for theta in (10 ** 9, 3000):
        _check(tr, cost, reason, 100, cap, theta, 2500)
