"""The scheduler's optional per-request outputs (admission order, counter after, counter on
arrival) are each optional on its own: every subset of the three against the oracle, with and
without interactions, in one call and in slices, for the paper's policy and for the flags."""
import itertools

import numpy as np
import pytest
import torch

import oracle
import paper_2411_15997_amd as fs
from gpu_common import compare_sim, say
from tiny import random_trace
import tracegen as tg

pytestmark = pytest.mark.gpu

OPTIONAL = ("admit_seq", "counter_after", "counter_on_arrival")
SUBSETS = [s for k in range(len(OPTIONAL) + 1) for s in itertools.combinations(OPTIONAL, k)]


def _schedule(tr, cost, reason, engine, keep, chunks):
    dt = fs.DeviceTrace(tr)
    out = fs.Outputs(dt)
    for k in OPTIONAL:
        if k not in keep:
            setattr(out, k, None)
            setattr(out.s, k, None)
    c, rz = torch.as_tensor(cost).cuda(), torch.as_tensor(reason).cuda()
    st = fs.fs_state_init(dt)
    done, most = 0, -1 if chunks is None else chunks
    while True:
        fs.fs_schedule_step(dt, st, c, rz, engine, out, most)
        done += max(most, 0)
        if most < 0 or (out.steps.cpu().numpy() < done).all():
            break
    return out.host()


@pytest.mark.parametrize("multi", [False, True])
@pytest.mark.parametrize("keep", SUBSETS, ids=lambda s: "+".join(s) or "none")
def test_each_optional_output_alone(keep, multi):
    rng = np.random.default_rng(40 + multi)
    # queues of a few calls (a user is often in Q when its next request arrives), queues
    # longer than a user's share on chip, and more users than a wave has lanes
    for users, cap, theta in ((5, 25, 200), (40, 40, 10 ** 9), (150, 30, 400)):
        say("optional outputs", keep, multi, users)
        tr = tg.concat([random_trace(rng, 900, users, 2, 5000, multi=multi, max_tok=8) for _ in range(3)])
        cost = rng.integers(0, 3000, tr.n).astype(np.int64)
        reason = rng.integers(0, 3, tr.n).astype(np.uint8)
        for flags, kw in ((0, {}), (oracle.FSO_FCFS, dict(fcfs=True)), (oracle.FSO_LITERAL, dict(literal=True))):
            room = cap * 8 if flags == oracle.FSO_LITERAL else cap
            o = oracle.simulate(tr, cost, reason, 50, room, theta, flags=flags)
            eng = fs.make_engine(50, room, theta, **kw)
            for chunks in (None, 17):
                g = _schedule(tr, cost, reason, eng, keep, chunks)
                compare_sim(g, o)
