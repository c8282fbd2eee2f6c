"""Metrics and workload analysis where a work-group's users go through an LDS hash table:
just above the directly indexed sizes, the application counts at which a table no longer
fits, replicas shorter than a chunk, and more distinct keys in a chunk than the table
holds (the rest go to global memory one by one).  Exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_15997_amd as fs
from gpu_common import say
import tracegen as tg

pytestmark = pytest.mark.gpu


def _trace(rng, n, U, A, links=True):
    """Uniform users and apps (most of a chunk's keys distinct), a heavy user, and calls whose
    first call is a few records back."""
    user = np.where(rng.random(n) < 0.2, min(7, U - 1), rng.integers(0, U, n)).astype(np.int32)
    app = rng.integers(0, A, n).astype(np.int32)
    i = np.arange(n, dtype=np.int32)
    back = np.minimum(rng.integers(1, 300, n), i).astype(np.int32)
    first = (rng.random(n) < 0.7) | (i == 0)
    head = np.where(first, i, i - back).astype(np.int32)
    # a later call's first call is a first call
    first |= ~first[head]
    head = np.where(first, i, head).astype(np.int32)
    first = head == i
    user = user[head]
    L = lambda: rng.integers(0, 5000, n).astype(np.int32)  # noqa: E731
    ts = np.sort(rng.integers(0, 10 ** 9, n)).astype(np.int64)
    call = np.where(first, 0, 1).astype(np.int32)
    prev = np.where(first, -1, head).astype(np.int32)
    if not links:
        call = head = prev = None
    return tg.Trace(1, U, A, np.array([0, n], np.int64), ts, user, app, call, head, prev, L(), L(), L())


def _metrics(tr, rng):
    n, step = tr.n, 50_000
    cost = rng.integers(0, 10 ** 6, n).astype(np.int64)
    status = rng.choice(np.array([0, 0, 0, 1, 2, 3], np.int8), n)
    astep = np.where(status == 0, tr.ts_us // step + rng.integers(0, 3, n), -1).astype(np.int32)
    gap = rng.integers(0, 2 ** 40, tr.n_replicas).astype(np.int64)
    dt = fs.DeviceTrace(tr)
    out = fs.Outputs(dt, parity=False)
    out.status[:n].copy_(torch.as_tensor(status))
    out.admit_step[:n].copy_(torch.as_tensor(astep))
    out.max_gap.copy_(torch.as_tensor(gap))
    m = fs.fs_fairness_metrics(dt, torch.as_tensor(cost).cuda(), out, fs.make_engine(step, 1000, 1000)).host()
    o = oracle.fairness_metrics(tr, cost, status, astep, gap, step, 0)
    for k in ("throttled", "aborted_midway", "wasted_tokens"):
        assert (m[k] == getattr(o, k)).all(), k
    for k in ("jain", "svc_req_pct", "svc_int_pct", "served_users_pct", "delayed_users_pct"):
        # both are one rounding of the same exact integers: a few units in the last place
        np.testing.assert_allclose(m[k], getattr(o, k), rtol=1e-14, atol=0, err_msg=k)


@pytest.mark.parametrize("links", [True, False])
@pytest.mark.parametrize("sizes,U,A", [([5000, 0, 1, 900], 4097, 3), ([40_000], 200_000, 2),
                                       ([2047, 2049, 4096], 8191, 5), ([4_600_000], 1_000_000, 2)])
def test_metrics_many_users(sizes, U, A, links):
    rng = np.random.default_rng(U + links)
    say("metrics many users", sizes, U, links)
    _metrics(tg.concat([_trace(rng, n, U, A, links) for n in sizes]), rng)


@pytest.mark.parametrize("sizes,U,A", [([3000, 0, 1, 900], 300, 31), ([30_000], 5000, 32), ([30_000], 5000, 33),
                                       ([20_000], 3000, 64), ([20_000], 3000, 65),
                                       ([2047, 2049, 4096], 257, 7), ([2_300_000], 400_000, 3)])
def test_workload_many_keys(sizes, U, A):
    rng = np.random.default_rng(U + A)
    say("workload many keys", sizes, U, A)
    tr = tg.concat([_trace(rng, n, U, A) for n in sizes])
    got = fs.fs_workload_stats(fs.DeviceTrace(tr), 60_000_000).host()
    want = oracle.workload_stats(tr, 60_000_000)
    for k, v in got.items():
        w = getattr(want, k)
        assert (v.reshape(w.shape) == w).all(), k


@pytest.mark.parametrize("U,A", [((1 << 26) + 1, 64), ((1 << 32) // 33, 33), (1 << 27, 32)])
def test_workload_more_keys_than_32_bits(U, A):
    """(replica, user, app) keys just below and beyond 2^32 (64 GiB of workspace; the histograms
    are those of the same requests with the users numbered densely)."""
    rng = np.random.default_rng(A)
    say("workload wide keys", U, A)
    tr = _trace(rng, 30_000, U, A)
    ids, dense = np.unique(tr.user, return_inverse=True)
    d = tg.Trace(1, ids.size, A, tr.rep_off, tr.ts_us, dense.astype(np.int32), tr.app, tr.call, tr.head, tr.prev,
                 tr.len_in, tr.len_sys, tr.len_out)
    want = oracle.workload_stats(d, 60_000_000)
    got = fs.fs_workload_stats(fs.DeviceTrace(tr), 60_000_000, per_app=False)
    at = torch.as_tensor(ids.astype(np.int64)).cuda()
    for k in ("user_req", "user_tok"):
        v = getattr(got, k)
        assert (v[0, at].cpu().numpy() == getattr(want, k)[0]).all(), k
        assert int(v.sum()) == int(getattr(want, k).sum()), k
    for k in ("minutes", "rate_hist", "len_hist", "len_sum", "size_hist", "graph"):
        w = getattr(want, k)
        assert (getattr(got, k).cpu().numpy().reshape(w.shape) == w).all(), k
    del got, v
    torch.cuda.empty_cache()


def test_workload_two_to_the_31_users():
    """2 x 2^30 users, the most a trace may have (64 GiB of workspace and outputs)."""
    U, n = 1 << 30, 3000
    rng = np.random.default_rng(31)
    say("workload 2^31 users")
    tr = tg.concat([_trace(rng, n, U, 1) for _ in range(2)])
    got = fs.fs_workload_stats(fs.DeviceTrace(tr), 60_000_000, per_app=False)
    for r in range(2):
        m = slice(r * n, (r + 1) * n)
        ids, dense = np.unique(tr.user[m], return_inverse=True)
        d = tg.Trace(1, ids.size, 1, np.array([0, n], np.int64), tr.ts_us[m], dense.astype(np.int32), tr.app[m],
                     tr.call[m], tr.head[m], tr.prev[m], tr.len_in[m], tr.len_sys[m], tr.len_out[m])
        want = oracle.workload_stats(d, 60_000_000)
        at = torch.as_tensor(ids.astype(np.int64)).cuda()
        for k in ("user_req", "user_tok"):
            v = getattr(got, k)[r]
            assert (v[at].cpu().numpy() == getattr(want, k)[0]).all(), (r, k)
            assert int(v.sum()) == int(getattr(want, k).sum()), (r, k)
        for k in ("minutes", "rate_hist", "len_hist", "len_sum", "size_hist", "graph"):
            assert (getattr(got, k)[r].cpu().numpy() == getattr(want, k)[0]).all(), (r, k)
    del got, v
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [900, 5000])
def test_metrics_two_to_the_31_users(n):
    """One replica of 2^31 - 1 users, the last of them with requests: the finish pass in one
    work-group and in parts (40 GiB; the metrics are those of the users numbered densely)."""
    U = (1 << 31) - 1
    rng = np.random.default_rng(n)
    say("metrics 2^31 users", n)
    tr = _trace(rng, n, U - 600, 2)
    tr.n_users = U
    tr.user = np.where(tr.user % 3 == 0, U - 1 - tr.user % 599, tr.user).astype(np.int32)
    ids, dense = np.unique(tr.user, return_inverse=True)
    step = 50_000
    cost = rng.integers(0, 10 ** 6, n).astype(np.int64)
    status = rng.choice(np.array([0, 0, 0, 1, 2, 3], np.int8), n)
    astep = np.where(status == 0, tr.ts_us // step + rng.integers(0, 3, n), -1).astype(np.int32)
    gap = np.array([123], np.int64)
    dt = fs.DeviceTrace(tr)
    out = fs.Outputs(dt, parity=False)
    out.status[:n].copy_(torch.as_tensor(status))
    out.admit_step[:n].copy_(torch.as_tensor(astep))
    out.max_gap.copy_(torch.as_tensor(gap))
    m = fs.fs_fairness_metrics(dt, torch.as_tensor(cost).cuda(), out, fs.make_engine(step, 1000, 1000)).host()
    d = tg.Trace(1, ids.size, 2, tr.rep_off, tr.ts_us, dense.astype(np.int32), tr.app, tr.call, tr.head, tr.prev,
                 tr.len_in, tr.len_sys, tr.len_out)
    o = oracle.fairness_metrics(d, cost, status, astep, gap, step, 0)
    for k in ("throttled", "aborted_midway", "wasted_tokens"):
        assert (m[k] == getattr(o, k)).all(), k
    for k in ("jain", "svc_req_pct", "svc_int_pct", "served_users_pct", "delayed_users_pct"):
        np.testing.assert_allclose(m[k], getattr(o, k), rtol=1e-14, atol=0, err_msg=k)
    del dt, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("links", [True, False])
@pytest.mark.parametrize("sizes,U", [([262_145], 4096), ([524_289, 1, 0, 700], 100), ([5] * 40 + [300_001], 1024)])
def test_metrics_chunks(sizes, U, links):
    """Directly indexed users: chunks that follow from the largest replica, not from the total."""
    rng = np.random.default_rng(U + links)
    say("metrics chunks", sizes[-1], U, links)
    _metrics(tg.concat([_trace(rng, n, U, 3, links) for n in sizes]), rng)


@pytest.mark.parametrize("links", [True, False])
@pytest.mark.parametrize("sizes", [[37] * 300, [511, 0, 0, 513, 1, 2047] * 3, [40, 0] * 60 + [2048], [300] * 70])
def test_metrics_short_replicas(sizes, links):
    """Replicas of few requests and many users (taken by single waves), on both sides of the
    sizes where the whole work-group takes a replica; more replicas in a chunk than waves, and
    replicas cut by the end of a chunk."""
    rng = np.random.default_rng(len(sizes) + links)
    say("metrics short replicas", len(sizes), links)
    _metrics(tg.concat([_trace(rng, n, 4100, 3, links) for n in sizes]), rng)
