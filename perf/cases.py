"""Timed cases of the policy hot path, each through the package's public entry points.

A case is one call (or one step) of a user's program on one MI355X: the whole path over
a batch of trace replicas (cost, window test, schedule, metrics), a scheduler advanced
in slices of time, the window test on its own over a request stream, and the offline
passes (metrics, workload analysis, weights from a history, cost).  The traces are
seeded synthetic ones with the shapes the repository's workloads have: Zipf users with
a few abusive ones, a home app per user, chained calls a second apart, lognormal tokens.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2411_15997_amd as fs

NO_LIMIT = 2 ** 31 - 1
Q16 = 1 << 16
SECOND_US = 1_000_000
K = 1024                       # scale of the Eq. 1 weights

# Request mixes: rate (requests/s of a replica), users' Zipf exponent, share of abusive
# users and their multiple, chained calls, token spread, limits and engine step.
MIXES = {
    # a few users of two apps, one of them heavy; direct weights, an app limit only
    "small": dict(rate=33.3, zipf=0.0, abusive=0.125, mult=40.0, calls="one", sigma=1.0,
                  window_s=10, t_user=NO_LIMIT, t_app=30, step_us=250_000, cap=4096),
    # a weight sweep: single-call requests, each replica with weights of its own
    "sweep": dict(rate=33.3, zipf=1.1, abusive=0.05, mult=10.0, calls="one", sigma=1.0,
                  window_s=60, t_user=120, t_app=30, step_us=200_000, cap=16384),
    # replicas of a service with chained calls
    "replicas": dict(rate=27.8, zipf=1.1, abusive=0.05, mult=10.0, calls="geom", sigma=1.0,
                     window_s=60, t_user=240, t_app=60, step_us=250_000, cap=16384),
    # one large tenant over a day: diurnal, interaction sizes of the paper's Table 2,
    # system prompts, weights per stage
    "tenant": dict(rate=115.7, zipf=1.2, abusive=0.01, mult=50.0, calls="table2", sigma=0.5,
                   window_s=60, t_user=300, t_app=38, step_us=160_000, cap=65536),
    # a request stream in front of the engine: window tests only, no tokens
    "stream": dict(rate=13_900.0, zipf=1.1, abusive=0.05, mult=10.0, calls="geom3", sigma=None,
                   window_s=60, t_user=300, t_app=100, step_us=250_000, cap=16384),
}
GEOM_P = (1.0, 1.0, 0.7, 0.5, 0.5, 0.3, 0.3, 0.2)
TENANT_STAGES = 20


def _case(name, kind, mix, R, U, A, n, **more):
    c = {"name": name, "kind": kind, "mix": mix, "replicas": R, "users": U, "apps": A,
         "requests": n, "ragged": False}
    c.update(more)
    return c


def listed():
    return [
        # the smallest whole run: a minute of one service, every per-request output asked for
        _case("run_small", "run", "small", 1, 8, 2, 2_000, policy="fs", literal=False,
              parity=True, slices=0),
        # the benchmark's default: a weight sweep over 1,024 replicas
        _case("run_sweep", "run", "sweep", 1024, 1024, 8, 20_000, policy="fs", literal=False,
              parity=False, slices=0),
        # an hour of 64 replicas with chained calls
        _case("run_replicas", "run", "replicas", 64, 256, 8, 100_000, policy="fs", literal=False,
              parity=False, slices=0),
        # three quarters of an hour of one large tenant: a single long decision chain
        _case("run_tenant", "run", "tenant", 1, 100_000, 32, 300_000, policy="fs", literal=False,
              parity=False, slices=0),
        # the execution stream as the paper writes it (decode steps, KV capacity), odd sizes
        _case("run_literal_ragged", "run", "replicas", 41, 251, 7, 20_000, ragged=True, policy="fs",
              literal=True, parity=False, slices=0),
        # a serving loop: the same replicas advanced in slices of time, state kept between
        _case("run_slices", "run", "replicas", 64, 256, 8, 10_000, policy="fs", literal=False,
              parity=True, slices=12),
        # the window test on the largest stream, gated by interaction
        _case("throttle_stream", "throttle", "stream", 1, 10_000, 16, 50_000_000, raw=False,
              app_scope=0, counts=False),
        # an app-level rate limit (every user of an app together) on a shorter, odd stream
        _case("throttle_app_level", "throttle", "stream", 3, 2_501, 13, 1_000_003, ragged=True,
              raw=True, app_scope=1, counts=False),
        # served-experience metrics of the large tenant's whole day
        _case("metrics_tenant", "metrics", "tenant", 1, 100_000, 32, 10_000_000, blind=False),
        # workload analysis of the large tenant's whole day
        _case("workload_tenant", "workload", "tenant", 1, 100_000, 32, 10_000_000),
        # weights and app limits from the large tenant's day as the history
        _case("history_tenant", "history", "tenant", 1, 100_000, 32, 10_000_000),
        # Eq. 2 over the sweep with a priority per user
        _case("cost_priorities", "cost", "sweep", 1024, 1024, 8, 20_000, prio=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed kinds: sizes over their whole ranges, odd ones, other policies,
    modes and options among them."""
    kind = rng.choice(("run", "run", "run", "run", "throttle", "throttle", "metrics", "workload",
                       "history", "cost"))
    if kind == "throttle":
        n = _log_int(rng, 1_000, 30_000_000)
        R = rng.choice((1, 1, 1, _log_int(rng, 2, 40)))
        counts = rng.random() < 0.2
        return _case("", kind, "stream", R, _log_int(rng, 50, 20_000), rng.randint(2, 32),
                     max(1, n // R), ragged=rng.random() < 0.5, raw=rng.random() < 0.5,
                     app_scope=int(rng.random() < 0.25), counts=counts)
    mix = rng.choice(("sweep", "replicas", "tenant"))
    if kind == "run":
        policy = rng.choice(("fs", "fs", "fs", "wsc_only", "vtc", "rpm"))
        literal = rng.random() < 0.2
        most = 5_000 if policy == "rpm" else 15_000 if literal or policy != "fs" else \
            {"sweep": 20_000, "replicas": 100_000, "tenant": 200_000}[mix]
        R = {"sweep": _log_int(rng, 1, 1024), "replicas": _log_int(rng, 1, 128),
             "tenant": rng.choice((1, 1, 2, 3))}[mix]
        U = {"sweep": _log_int(rng, 16, 1200), "replicas": _log_int(rng, 16, 1000),
             "tenant": _log_int(rng, 1_000, 100_000)}[mix]
        n = _log_int(rng, 500, most)
        slices = rng.randint(2, 12) if rng.random() < 0.25 else 0
        return _case("", kind, mix, R, U, rng.randint(2, 16), n, ragged=rng.random() < 0.5,
                     policy=policy, literal=literal, parity=rng.random() < 0.3, slices=slices)
    total = _log_int(rng, 2_000, 10_000_000)
    R = {"sweep": _log_int(rng, 1, 1024), "replicas": _log_int(rng, 1, 128), "tenant": 1}[mix]
    U = {"sweep": _log_int(rng, 16, 1200), "replicas": _log_int(rng, 16, 5_000),
         "tenant": _log_int(rng, 1_000, 100_000)}[mix]
    A = rng.randint(2, 32 if mix == "tenant" else 12)
    c = _case("", kind, mix, R, U, A, max(1, total // R), ragged=rng.random() < 0.5)
    if kind == "metrics":
        c["blind"] = rng.random() < 0.3
    if kind == "cost":
        c["prio"] = rng.random() < 0.5
    return c


# ------------------------------------------------------------------------- inputs

def _lengths(c):
    """Requests of each replica; ragged replicas differ by up to a half."""
    n = c["requests"]
    return [n - (r * 7919) % (n // 2 + 1) if c["ragged"] else n for r in range(c["replicas"])]


def _means(c):
    """Mean input, system and output tokens per app: input-heavy to output-heavy apps."""
    A = c["apps"]
    x = np.arange(A) / max(1, A - 1)
    if c["mix"] == "tenant":
        return 200 * 32.0 ** x, 50 * 40.0 ** x, 30 * 20.0 ** ((13 * np.arange(A)) % A / max(1, A - 1))
    if c["mix"] == "small":
        return np.full(A, 665.0), np.zeros(A), np.full(A, 245.0)
    return 200 * 20.0 ** x, np.zeros(A), 200 * 20.0 ** (1 - x)


def _interaction_sizes(c, apps, u):
    """Calls of each interaction from uniform draws `u`."""
    kind = MIXES[c["mix"]]["calls"]
    if kind == "one":
        return torch.ones_like(apps)
    if kind == "table2":   # request shares 73.22 : 26.09 : 0.50 for sizes 1, 2-10, 11-20
        w = np.array([73.22] + [26.09 / 9 / s for s in range(2, 11)] + [0.05 / s for s in range(11, 21)])
        cdf = torch.from_numpy(np.cumsum(w / w.sum())).to(u)
        return torch.searchsorted(cdf, u, right=True).clamp_(max=19) + 1
    p = torch.tensor([0.3 if kind == "geom3" else GEOM_P[a % 8] for a in range(c["apps"])], dtype=u.dtype,
                     device=u.device)[apps]
    m = torch.floor(torch.log1p(-u) / torch.log1p(-p.clamp(max=1 - 1e-9))).long() + 1
    return torch.where(p >= 1, torch.ones_like(m), m.clamp_(1, 20))


def _trace(c, seed):
    """A seeded trace made on the GPU, as host arrays (what a user's program reads in)."""
    mix, dev = MIXES[c["mix"]], "cuda"
    R, U, A, n = c["replicas"], c["users"], c["apps"], c["requests"]
    gen = torch.Generator(dev).manual_seed(seed)
    rand = lambda *s: torch.rand(s, generator=gen, device=dev, dtype=torch.float64)  # noqa: E731
    rank = rand(R, U).argsort(1).double() + 1
    w = rank ** (-mix["zipf"])
    abusive = rand(R, U).argsort(1) < max(1, round(mix["abusive"] * U))
    w = torch.where(abusive, w * mix["mult"], w)
    cdf = ((w * 2.0 ** 30).long() + 1).cumsum(1)
    home = (rand(R, U) * A).long()
    # interactions, more than enough for n requests
    I = n if mix["calls"] != "geom3" else min(n, int(n * 0.31) + 64)
    user = torch.searchsorted(cdf, (rand(R, I) * cdf[:, -1:]).long(), right=True).clamp_(max=U - 1)
    app = torch.where(rand(R, I) < 0.8, home.gather(1, user), (rand(R, I) * A).long())
    m = _interaction_sizes(c, app, rand(R, I))
    t0 = rand(R, I).sort(1)[0]
    cm = m.cumsum(1)
    at = torch.arange(n, device=dev).expand(R, n).contiguous()
    inter = torch.searchsorted(cm, at, right=True).clamp_(max=I - 1)
    first = (cm - m).gather(1, inter)
    stage = at - first
    if mix["calls"] == "table2":   # a day's rise and fall
        x = np.linspace(0, 1, 1 << 16)
        day = torch.from_numpy(x - np.sin(2 * np.pi * x) / (4 * np.pi)).to(dev)
        k = torch.searchsorted(day, t0).clamp_(1, (1 << 16) - 1)
        t0 = (k - (day[k] - t0) / (day[k] - day[k - 1])) / ((1 << 16) - 1)
    # the interactions that are used span the horizon
    span = t0.gather(1, inter[:, -1:]).clamp(min=1e-9)
    per_user = 50_000_000 / 3600 / 10_000    # a stream's rate grows with its users
    rate = per_user * U if c["mix"] == "stream" else mix["rate"]
    horizon = max(2.0, n / rate) * SECOND_US
    ts = (t0.gather(1, inter) / span * horizon).long() + stage * SECOND_US
    del span, t0, cm, m
    ts, order = ts.sort(dim=1, stable=True)
    out = SimpleNamespace(n_replicas=R, n_users=U, n_apps=A)
    ns = _lengths(c)
    out.rep_off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int64)
    keep = None
    if c["ragged"]:
        keep = at < torch.tensor(ns, device=dev)[:, None]

    def host(x, dt):
        x = x.to(dt)
        return (x.reshape(-1) if keep is None else x[keep]).cpu().numpy()

    out.ts_us = host(ts, torch.int64)
    del ts
    chosen = inter.gather(1, order)
    out.user = host(user.gather(1, chosen), torch.int32)
    ap = app.gather(1, chosen)
    out.app = host(ap, torch.int32)
    st = stage.gather(1, order)
    out.call = out.head = out.prev = None
    if mix["calls"] != "one":
        pos = torch.empty_like(order).scatter_(1, order, at)
        out.call = host(st, torch.int32)
        out.head = host(pos.gather(1, first.gather(1, order)), torch.int32)
        before = pos.gather(1, (order - 1).clamp_(min=0))
        out.prev = host(torch.where(st > 0, before, torch.full_like(st, -1)), torch.int32)
        del pos, before
    out.len_in = out.len_sys = out.len_out = None
    if mix["sigma"] is not None:
        slope = 0.25 if c["mix"] == "tenant" else 0.0
        for k, mean, sl in zip(("len_in", "len_sys", "len_out"), _means(c), (slope, 0.0, 0.0)):
            if not mean.any():
                continue
            mu = torch.from_numpy(np.log(mean)).to(dev)[ap] + torch.log1p(st * sl)
            z = torch.randn(mu.shape, generator=gen, device=dev, dtype=torch.float64)
            x = torch.exp(mu - mix["sigma"] ** 2 / 2 + mix["sigma"] * z).round().clamp_(1, 65_536)
            setattr(out, k, host(x, torch.int32))
    return out


def _coef(c, seed):
    """Q16 weights: drawn per replica (sweep), fixed (small), else Eq. 1 per app and stage."""
    R, A = c["replicas"], c["apps"]
    if c.get("policy") == "vtc":
        return np.full((1, A, 1, 3), Q16, np.int64)
    if c["mix"] == "sweep":
        g = np.random.RandomState(seed % 2 ** 32).randint(0, 113, (R, 2)) * (Q16 // 16) + Q16
        t = np.full((R, A, 1, 3), 2 * Q16, np.int64)
        t[:, :, 0, 0], t[:, :, 0, 2] = g[:, :1], g[:, 1:]
        return t
    if c["mix"] == "small":
        return np.array([[[[Q16, 2 * Q16, (2 + 2 * a) * Q16]] for a in range(A)]], np.int64)
    J = TENANT_STAGES if c["mix"] == "tenant" else 1
    mi, ms, mo = _means(c)
    e_in = mi[:, None] * (1 + (0.25 * np.arange(J) if J > 1 else 0))
    w = e_in + 2 * ms[:, None] + mo[:, None]
    return np.rint(np.array([1.0, 2.0, 1.0]) * Q16 * K / w[..., None]).astype(np.int64)[None]


def _policy(c):
    """(user limit, app limits, overload threshold, first come first served, interaction-blind)"""
    mix, A = MIXES[c["mix"]], c["apps"]
    p = c.get("policy", "fs")
    if p in ("wsc_only", "vtc"):
        return NO_LIMIT, [NO_LIMIT] * A, mix["cap"], False, False
    if p == "rpm":
        return mix["t_user"], [NO_LIMIT] * A, -1, True, True
    return mix["t_user"], [mix["t_app"]] * A, mix["cap"], False, False


def prepare(case, seed):
    c, dev = case, "cuda"
    mix = MIXES[c["mix"]]
    s = SimpleNamespace(case=c, kind=c["kind"])
    s.dt = dt = fs.DeviceTrace(_trace(c, seed), device=dev)
    s.err = torch.zeros(1, dtype=torch.int32, device=dev)
    t_user, t_app, theta, fcfs, blind = _policy(c)
    s.limits = fs.make_limits(mix["window_s"] * SECOND_US, t_user, t_app, c.get("app_scope", 0))
    buf = lambda nb: torch.empty(max(nb, 1), dtype=torch.uint8, device=dev)  # noqa: E731
    gen = torch.Generator(dev).manual_seed(seed + 1)
    prio = None
    if c.get("prio"):
        prio = torch.randint(64, 1024, (dt.n_users,), generator=gen, device=dev).cpu().numpy()
    if s.kind in ("run", "cost", "metrics"):
        coef = _coef(c, seed)
        s.weights, s.tables = fs.make_weights(dt, coef, prio, per_replica=coef.shape[0] > 1)
    if s.kind == "run":
        step, cap = mix["step_us"], mix["cap"]
        if c["literal"]:       # decode iterations of 20 ms, 4M KV-cache tokens
            step, cap = 20_000, 1 << 22
        s.engine = fs.make_engine(step, cap, theta, fcfs=fcfs, blind=blind, literal=c["literal"])
        s.out = fs.Outputs(dt, parity=c["parity"])
        s.metrics, s.metrics_ws = fs.Metrics(dt), buf(fs.fs_metrics_workspace(dt))
        if c["slices"]:
            s.cost = torch.empty(dt.n, dtype=torch.int64, device=dev)
            s.reason = torch.empty(dt.n, dtype=torch.uint8, device=dev)
            s.bitmap = torch.zeros((dt.n + 31) // 32, dtype=torch.int32, device=dev)
            s.throttle_ws, s.state = buf(fs.fs_throttle_workspace(dt)), buf(fs.fs_state_bytes(dt))
            # slices of equal time over the trace's horizon; the last one drains the queue
            s.slice_steps = max(1, int(dt.ts_us.max()) // step // c["slices"])
        else:
            s.ws, s.cost, s.reason = fs.run_trace_buffers(dt)
    elif s.kind == "throttle":
        s.ws = buf(fs.fs_throttle_workspace(dt))
        s.bitmap = torch.zeros((dt.n + 31) // 32, dtype=torch.int32, device=dev)
        s.reason = torch.empty(dt.n, dtype=torch.uint8, device=dev)
    elif s.kind == "metrics":
        s.engine = fs.make_engine(mix["step_us"], mix["cap"], theta)
        s.cost = fs.fs_cost(dt, s.weights)
        s.out = fs.Outputs(dt, parity=False)
        _outcome(s, c, gen)
        s.metrics, s.ws = fs.Metrics(dt), buf(fs.fs_metrics_workspace(dt))
    elif s.kind == "workload":
        s.out, s.ws = fs.WorkloadStats(dt), buf(fs.fs_workload_workspace(dt))
    elif s.kind == "cost":
        s.cost = torch.empty(dt.n, dtype=torch.int64, device=dev)
    return s


def _outcome(s, c, gen):
    """A finished run's outcome: a fifth of the interactions throttled (or, blind to them, of
    the calls, with every later call of the interaction dropped), waits of a few steps."""
    dt, tau = s.dt, MIXES[c["mix"]]["step_us"]
    rep = _replica(dt)
    at = torch.arange(dt.n, device=dt.device)
    head = at if dt.head is None else dt.rep_off[rep] + dt.head
    over = torch.rand(dt.n, generator=gen, device=dt.device) < 0.2
    why = torch.where(torch.rand(dt.n, generator=gen, device=dt.device) < 0.5, 1, 2)
    first = at == head
    if c["blind"] and dt.head is not None:
        call = dt.call.long()
        drop = torch.full_like(at, 1 << 20).scatter_reduce_(0, head[over], call[over], "amin")[head]
        st = torch.where(call == drop, why, torch.where(call > drop, 3, 0))
    else:
        st = torch.where(over[head], torch.where(first, why[head], 3), 0)
    s.out.status.copy_(st)
    wait = (torch.rand(dt.n, generator=gen, device=dt.device) ** 8 * 40).long()
    s.out.admit_step.copy_(torch.where(st == 0, dt.ts_us // tau + wait, -1))
    s.out.max_gap.copy_((torch.rand(dt.n_replicas, generator=gen, device=dt.device) * 2 ** 40).long())


# ------------------------------------------------------------------------- one pass

def run(s):
    dt, c = s.dt, s.case
    if s.kind == "run":
        if c["slices"]:
            fs.fs_cost(dt, s.weights, cost=s.cost, err=s.err, check=False)
            fs.fs_throttle(dt, s.limits, raw=True, ws=s.throttle_ws, err=s.err, check=False,
                           bitmap=s.bitmap, reason=s.reason)
            fs.fs_state_init(dt, state=s.state)
            for k in range(c["slices"]):
                steps = s.slice_steps if k + 1 < c["slices"] else -1
                fs.fs_schedule_step(dt, s.state, s.cost, s.reason, s.engine, s.out, steps, check=False)
        else:
            fs.fs_run_trace(dt, s.weights, s.limits, s.engine, s.out, s.ws, check=False)
        fs.fs_fairness_metrics(dt, s.cost, s.out, s.engine, m=s.metrics, ws=s.metrics_ws, check=False)
        r = {k: getattr(s.out, k) for k in ("status", "admit_step", "admit_seq", "counter_after",
                                            "counter_on_arrival", "counter", "steps", "decisions",
                                            "max_gap", "err")}
        return {**r, **_values(s.metrics), "cost": s.cost, "reason": s.reason}
    if s.kind == "throttle":
        o = fs.fs_throttle(dt, s.limits, raw=c["raw"], want_counts=c["counts"], ws=s.ws, err=s.err,
                           check=False, bitmap=s.bitmap, reason=s.reason)
        return {"bitmap": o.bitmap, "reason": o.reason, "cnt_user": o.cnt_user, "cnt_app": o.cnt_app,
                "err": s.err}
    if s.kind == "metrics":
        fs.fs_fairness_metrics(dt, s.cost, s.out, s.engine, m=s.metrics, ws=s.ws, check=False)
        return {**_values(s.metrics), "err": s.out.err}
    if s.kind == "workload":
        fs.fs_workload_stats(dt, 60 * SECOND_US, out=s.out, ws=s.ws, err=s.err, check=False)
        return {**{k: getattr(s.out, k) for k in s.out.FIELDS}, "err": s.err}
    if s.kind == "history":
        J = TENANT_STAGES if c["mix"] == "tenant" else 1
        stats, coef, t_app = fs.fs_weights_from_history(dt, J, K=K, base_limit=30, err=s.err, check=False)
        return {"stats": stats, "coef": coef, "t_app": t_app, "err": s.err}
    fs.fs_cost(dt, s.weights, cost=s.cost, err=s.err, check=False)
    return {"cost": s.cost, "err": s.err}


def _values(m):
    return {k: getattr(m, k) for k in (
        "jain", "max_gap_tokens", "svc_req_pct", "svc_int_pct", "served_users_pct",
        "delayed_users_pct", "throttled", "aborted_midway", "wasted_tokens")}


# ------------------------------------------------------------------------- what a pass needs

def work(case):
    """Every input that the method reads once, every output written once; the operations are
    the integer ones of the cost, the window tests and the sums."""
    c = case
    N, R, U, A = sum(_lengths(c)), c["replicas"], c["users"], c["apps"]
    links = MIXES[c["mix"]]["calls"] != "one"
    lens = 12 if c["mix"] == "tenant" else 8
    if c["kind"] == "run":      # ts, user, app, lengths, links in; status, step, cost, reason out
        b = N * (8 + 4 + 4 + lens + (12 if links else 0) + 1 + 4 + 8 + 1 + (20 if c["parity"] else 0))
        return {"bytes": b + R * U * 8 + R * 96, "flops": 40 * N}
    if c["kind"] == "throttle":
        b = 8 + 4 + 4 + (0 if c["raw"] else 4) + 1 + 0.125 + (8 if c["counts"] else 0)
        return {"bytes": N * b, "flops": 8 * N}
    if c["kind"] == "metrics":  # ts, user, app, status, admission step, cost, call and first call
        return {"bytes": N * (8 + 4 + 4 + 1 + 4 + 8 + (8 if links else 0)) + R * 72, "flops": 10 * N}
    if c["kind"] == "workload":
        out = R * (8 + U * 16 + U * A * 16 + (A + 1) * 2 * 128 * 8 + A * (3 * 32 + 3 + 64) * 8 + 280)
        return {"bytes": N * (8 + 4 + 4 + lens + (8 if links else 0)) + out, "flops": 20 * N}
    if c["kind"] == "history":
        J = TENANT_STAGES if c["mix"] == "tenant" else 1
        return {"bytes": N * (4 + lens + (4 if links else 0)) + A * J * 64 + A * 4, "flops": 6 * N}
    return {"bytes": N * (4 + lens + (4 if links else 0) + (4 if c["prio"] else 0) + 8), "flops": 7 * N}


def tolerance(case):
    """Integer arithmetic throughout, and percentages and Jain's index from exact integers:
    the same bits on every run."""
    return "exact"


# ------------------------------------------------------------------------- plain torch, 64 bits

def _replica(dt):
    n = dt.rep_off[1:] - dt.rep_off[:-1]
    return torch.repeat_interleave(torch.arange(dt.n_replicas, device=dt.device), n, output_size=dt.n)


def _counts(key, ts, W):
    """Requests of the same key in (ts - W, ts] up to each request, in stream order."""
    order = torch.sort(key, stable=True)[1]
    wide = int(ts.max()) + W + 2
    x = key[order] * wide + ts[order] + W + 1
    k = torch.arange(1, x.numel() + 1, device=x.device) - torch.searchsorted(x, x - W, right=True)
    return torch.empty_like(k).scatter_(0, order, k)


def _lengths_of(dt):
    zero = torch.zeros_like(dt.len_in)
    return [x.long() for x in (dt.len_in, zero if dt.len_sys is None else dt.len_sys, dt.len_out)]


def exact(case, seed):
    c = case
    if c["kind"] == "run":     # a sequential simulation: no closed form in array operations
        return None
    s = prepare(c, seed)
    dt = s.dt
    rep, user, app = _replica(dt), dt.user.long(), dt.app.long()
    U, A, R = dt.n_users, dt.n_apps, dt.n_replicas
    at = torch.arange(dt.n, device=dt.device)
    head = at if dt.head is None else dt.rep_off[rep] + dt.head
    first = at == head
    err = torch.zeros(1, dtype=torch.int32, device=dt.device)
    total = lambda idx, v, n: torch.zeros(n, dtype=torch.int64, device=dt.device).index_add_(0, idx, v)  # noqa: E731
    if c["kind"] == "throttle":
        lim, t_app = s.limits
        cu = _counts(rep * U + user, dt.ts_us, lim.window_us)
        ca = _counts((rep if lim.app_scope else rep * U + user) * A + app, dt.ts_us, lim.window_us)
        raw = torch.where(cu > lim.t_user, 1, torch.where(ca > torch.from_numpy(t_app).to(ca)[app], 2, 0))
        if not c["raw"]:
            raw = torch.where(first, raw, torch.where(raw[head] != 0, 3, 0))
        bits = torch.nn.functional.pad(raw != 0, (0, -dt.n % 32)).reshape(-1, 32).long()
        words = (bits << torch.arange(32, device=bits.device)).sum(1)
        words = torch.where(words >= 2 ** 31, words - 2 ** 32, words).int()
        return {"bitmap": words, "reason": raw.to(torch.uint8), "cnt_user": cu.int() if c["counts"] else None,
                "cnt_app": ca.int() if c["counts"] else None, "err": err}
    L = _lengths_of(dt)
    if c["kind"] == "cost":
        coef, prio = s.tables
        k = coef[rep if coef.shape[0] > 1 else torch.zeros_like(rep), app, torch.zeros_like(app) if dt.call is None
                 else dt.call.long().clamp(max=coef.shape[2] - 1)]
        E = 256 if prio is None else prio.long()[user]
        return {"cost": E * (k * torch.stack(L, 1)).sum(1) >> 8, "err": err}
    if c["kind"] == "history":
        J = TENANT_STAGES if c["mix"] == "tenant" else 1
        j = torch.zeros_like(app) if dt.call is None else dt.call.long().clamp(max=J - 1)
        one = torch.ones_like(app)
        first_call = one if dt.call is None else (dt.call == 0).long()
        st = torch.stack([total(app * J + j, v, A * J) for v in (one, first_call, *L)], 1).reshape(A, J, 5)
        h = st.cpu().numpy()
        coef, lim = np.zeros((A, J, 3), np.int64), np.zeros(A, np.int32)
        for a in range(A):
            for k in range(J):
                for g in (h[a, k], h[a].sum(0), h.sum((0, 1)), None):   # group, app, history, none
                    n, D = (1, K) if g is None else (int(g[0]), int(g[2] + 2 * g[3] + g[4]))
                    if n and D:
                        break
                for x, weight in enumerate((1, 2, 1)):
                    q, r = divmod(Q16 * K * weight * n, D)
                    coef[a, k, x] = q + (2 * r > D or (2 * r == D and q % 2))
            n, f = int(h[a, :, 0].sum()), int(h[a, :, 1].sum())
            lim[a] = -(-30 * n // f) if f else 30
        return {"stats": st, "coef": torch.from_numpy(coef), "t_app": torch.from_numpy(lim), "err": err}
    if c["kind"] == "metrics":
        return {**_exact_metrics(s, rep, user, head, first, sum(L), total), "err": err}
    return {**_exact_workload(dt, rep, user, app, head, first, L, total), "err": err}


def _exact_metrics(s, rep, user, head, first, tokens, total):
    dt, tau = s.dt, s.engine.step_us
    R, U = dt.n_replicas, dt.n_users
    status = s.out.status[:dt.n].long()
    served = status == 0
    one = torch.ones_like(rep)
    n_served, n_calls = total(head[served], one[served], dt.n), total(head, one, dt.n)
    full = first & (n_served == n_calls)
    aborted = (n_served > 0) & (n_served < n_calls)
    delayed = served & (s.out.admit_step[:dt.n] - dt.ts_us // tau > 0)
    ru = rep * U + user
    any_of = lambda m: (total(ru[m], one[m], R * U) > 0).reshape(R, U)  # noqa: E731
    has = any_of(torch.ones_like(served))
    x = total(ru[served], s.cost[:dt.n][served], R * U).reshape(R, U).cpu().numpy()
    jain = []
    for r in range(R):
        v = [int(k) for k in x[r] if k]
        jain.append(sum(v) ** 2 / (int(has[r].sum()) * sum(k * k for k in v)) if v else 1.0)
    sums = lambda m, v: total(rep[m], v[m], R)  # noqa: E731
    pct = lambda a, b: torch.where(b > 0, 100.0 * a.double() / b.clamp(min=1).double(), 0.0)  # noqa: E731
    users = has.sum(1)
    return {"jain": torch.tensor(jain, dtype=torch.float64), "max_gap_tokens": s.out.max_gap.double() / Q16,
            "svc_req_pct": pct(sums(served, one), total(rep, one, R)),
            "svc_int_pct": pct(sums(full, one), sums(first, one)),
            "served_users_pct": pct(any_of(full).sum(1), users),
            "delayed_users_pct": pct(any_of(delayed).sum(1), users),
            "throttled": sums(status > 0, one), "aborted_midway": sums(first & aborted, one),
            "wasted_tokens": sums(served & aborted[head], tokens)}


def _log2_floor(x):
    """floor(log2 x) of whole x >= 1 (frexp is exact below 2^53)."""
    return torch.frexp(x.double())[1].long() - 1


def _exact_workload(dt, rep, user, app, head, first, L, total):
    R, U, A = dt.n_replicas, dt.n_users, dt.n_apps
    one, tok = torch.ones_like(rep), sum(L)
    last = torch.full((R,), -1, dtype=torch.int64, device=dt.device).scatter_reduce_(0, rep, dt.ts_us, "amax")
    M = torch.where(last >= 0, last // (60 * SECOND_US) + 1, 0)
    rua = (rep * U + user) * A + app
    ua = [total(rua, v, R * U * A).reshape(R, U, A) for v in (one, tok)]
    u = [x.sum(2) for x in ua]

    def rate_bin(x):
        m = M.clamp(min=1).reshape(R, *[1] * (x.dim() - 1)).expand_as(x)
        d = _log2_floor(x.clamp(min=1)) - _log2_floor(m)
        less = torch.where(d >= 0, x < (m << d.clamp(min=0)), (x << (-d).clamp(min=0)) < m)
        return torch.where(x == 0, 0, 64 + d - less.long())

    rate = torch.zeros((R, A + 1, 2, 128), dtype=torch.int64, device=dt.device)
    for q in range(2):
        for rows, x, has in ((slice(0, A), ua[q].transpose(1, 2), ua[0].transpose(1, 2) > 0),
                             (slice(A, A + 1), u[q][:, None], u[0][:, None] > 0)):
            rate[:, rows, q].scatter_add_(2, rate_bin(x), has.long())
    ra = rep * A + app
    len_hist, len_sum = [], []
    for v in L:
        b = torch.where(v == 0, 0, 1 + _log2_floor(v.clamp(min=1)))
        len_hist.append(total(ra * 32 + b, one, R * A * 32).reshape(R, A, 32))
        len_sum.append(total(ra, v, R * A).reshape(R, A))
    size = total(head, one, dt.n)
    size_hist = total((ra * 64 + size.clamp(max=64) - 1)[first], one[first], R * A * 64).reshape(R, A, 64)
    edges = torch.tensor([1, 10, 20, 30, 40, 50], device=dt.device)
    g = rep * 7 + torch.searchsorted(edges, size[head])
    graph = torch.stack([total(g, v, R * 7) for v in (first.long(), one, L[0], L[2], L[1])], 1)
    return {"minutes": M, "user_req": u[0], "user_tok": u[1], "user_app_req": ua[0], "user_app_tok": ua[1],
            "rate_hist": rate, "len_hist": torch.stack(len_hist, 2), "len_sum": torch.stack(len_sum, 2),
            "size_hist": size_hist, "graph": graph.reshape(R, 7, 5)}
