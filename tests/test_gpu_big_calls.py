"""Calls that do not fit the on-chip passes' packed word: three lengths of up to 2^24 - 1 that
sum to more than 24 bits, and costs of 2^40 and more, among ordinary calls.  Every policy and
engine mode, in one call and in slices (a slice resumes with such calls queued or running),
bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_common import compare_sim, gpu_schedule, say
from tiny import random_trace
import tracegen as tg

pytestmark = pytest.mark.gpu

TOP = (1 << 24) - 1


def _trace(rng, users, multi, what, share, literal):
    tr = tg.concat([random_trace(rng, 700, users, 2, 6000, multi=multi, max_tok=30) for _ in range(3)])
    big = rng.random(tr.n) < share
    cost = rng.integers(0, 5000, tr.n).astype(np.int64)
    if what == "tokens":
        # sums on both sides of 2^24, and close to 3 * 2^24 (the literal engine decodes len_out
        # steps, so there only the prompt is long)
        top = np.where(rng.random(tr.n) < 0.5, TOP, TOP // 2 + rng.integers(-2, 3, tr.n)).astype(np.int32)
        tr.len_in = np.where(big, top, tr.len_in)
        tr.len_sys = np.where(big & (rng.random(tr.n) < 0.7), top, tr.len_sys)
        if not literal:
            tr.len_out = np.where(big & (rng.random(tr.n) < 0.7), top, tr.len_out)
        tr.len_in, tr.len_sys, tr.len_out = (x.astype(np.int32) for x in (tr.len_in, tr.len_sys, tr.len_out))
    else:
        cost = np.where(big, rng.integers((1 << 40) - 3, 1 << 44, tr.n), cost)
    return tr, cost


@pytest.mark.parametrize("fcfs,blind,literal", [(False, False, False), (True, False, False), (False, True, False),
                                                (True, True, False), (False, False, True), (True, True, True)])
@pytest.mark.parametrize("multi", [False, True])
@pytest.mark.parametrize("what,share", [("tokens", 0.003), ("tokens", 0.2), ("cost", 0.01)])
def test_calls_beyond_the_packed_word(what, share, multi, fcfs, blind, literal):
    rng = np.random.default_rng([multi, fcfs, blind, literal, int(share * 1000)])
    flags = ((oracle.FSO_FCFS if fcfs else 0) | (oracle.FSO_BLIND if blind else 0) |
             (oracle.FSO_LITERAL if literal else 0))
    for users in (6, 70):
        tr, cost = _trace(rng, users, multi, what, share, literal)
        reason = rng.integers(0, 3, tr.n).astype(np.uint8)
        cap = (1 << 26 if what == "tokens" else 600) if literal else (1 << 22 if what == "tokens" else 60)
        for theta in (10 ** 12, 1 << 25 if what == "tokens" else 400):
            say("big calls", what, share, multi, fcfs, blind, literal, users, theta)
            o = oracle.simulate(tr, cost, reason, 50, cap, theta, flags=flags)
            for chunks in (None, 29):
                g = gpu_schedule(tr, cost, reason, 50, cap, theta, chunks=chunks, fcfs=fcfs, blind=blind,
                                 literal=literal)
                compare_sim(g, o)
