"""Served requests that change their launches under way: as others are
admitted and retire, a request's chunks move between a launch of its own
and the shared ones (batched and column-split table launches).  Every
request, whatever ran beside it, ends like the same anneal alone."""
import time

import numpy as np
import pytest

from paper_2407_10205_amd import instances as inst

pytestmark = pytest.mark.gpu

SCHED = dict(eps=0.2, gamma=1.0, beta0=0.1, beta1=2.0, refresh_L=20)


def make(kind, N, seed):
    if kind == "i8":
        return inst.er_maxcut(N, 0.1, seed, signed=True)
    if kind == "i8wide":
        return inst.sk_gauss_fixed(N, seed, frac_bits=5, bits=8)
    return inst.sk_gauss_fixed(N, seed, frac_bits=9, bits=16)


def check(specs, slots):
    """specs: (kind, N, replicas, steps, accept/reject) in order of arrival."""
    from paper_2407_10205_amd import phia as P
    srv = P.Server(1 << 36, max_slots=slots, chunk_steps=30)
    probs, tickets = [], []
    for i, (kind, N, R, T, mh) in enumerate(specs):
        p = P.Problem(*make(kind, N, i % 3))
        probs.append(p)
        tickets.append(srv.submit(p, R, T, -(1 << 60), seed=i + 1, mh=mh, **SCHED))
    res = [srv.wait(t, 60.0) for t in tickets]
    spins = [srv.spins(t) for t in tickets]
    srv.close()
    for i, (kind, N, R, T, mh) in enumerate(specs):
        print("request", i, specs[i], flush=True)
        with P.Problem(*make(kind, N, i % 3)) as q:
            q.anneal(R, T, seed=i + 1, mh=mh, **SCHED)
            e, _, r = q.best_exact()
            s = q.replica_best()[1][r]
        assert (res[i]["state"], res[i]["energy_units"], res[i]["replica"], res[i]["steps_used"]) == (P.REQ_DONE, e, r, T)
        assert np.array_equal(spins[i], s), specs[i]
        probs[i].close()


def test_large_requests_move_between_split_and_table():
    """Twenty requests of 897 to 1100 columns, in shared launches while they
    are many and in launches of their own as the last ones remain, int8 and
    16-bit, one and two row tiles in the table, several chunks in either."""
    check([("i8wide", 900 + 20 * (i % 4), (5, 16, 40)[i % 3], 60 + 35 * (i % 8), None) for i in range(14)] +
          [("bf16hilo", 550 + 50 * (i % 6), (16, 33)[i % 2], 45 + 50 * (i % 5), None) for i in range(12)], 26)
    # admitted one after the other: alone first, then among many
    check([("i8wide", 900, 16, 400, None)] + [("i8wide", 950, 16, 90, None)] * 12, 32)


def test_large_requests_share_launches():
    """Many requests with few replicas each do not pay a step chain of their
    own each: 32 take less than 0.7 times as long as one after the other."""
    from paper_2407_10205_amd import phia as P
    J, h = make("i8wide", 900, 1)
    probs = [P.Problem(J, h) for _ in range(32)]
    t = {}
    for n in (1, 32):
        srv = P.Server(1 << 36, max_slots=64, chunk_steps=100)
        t[n] = []
        for _ in range(4):
            t0 = time.perf_counter()
            for k in [srv.submit(p, 16, 500, -(1 << 60), seed=1, **SCHED) for p in probs[:n]]:
                assert srv.wait(k, 60.0)["steps_used"] == 500
            t[n].append(time.perf_counter() - t0)
        srv.close()
    for p in probs:
        p.close()
    print("one", min(t[1]), "thirty-two", min(t[32]), flush=True)
    assert min(t[32]) < 0.7 * 32 * min(t[1])


@pytest.mark.parametrize("N,R,want", [(520, 32, 0), (520, 33, 5), (700, 63, 5), (864, 33, 5)])
def test_served_requests_that_one_cu_holds(N, R, want):
    """Served requests past the batch sizes run resident from 33 replicas."""
    from paper_2407_10205_amd import phia as P
    J, h = make("i8", N, 1)
    with P.Server(1 << 36, max_slots=4, chunk_steps=30) as srv, P.Problem(J, h) as p, P.Problem(J, h) as q:
        t = srv.submit(p, R, 70, -(1 << 60), seed=5, **SCHED)
        r = srv.wait(t, 60.0)
        s = srv.spins(t)
        assert p.info()["sweep_kernel"] == want
        q.anneal(R, 70, seed=5, **SCHED)
        e, _, k = q.best_exact()
        assert (r["energy_units"], r["replica"]) == (e, k) and np.array_equal(s, q.replica_best()[1][k])


def test_batch_sized_requests_move_between_own_and_batched_launches():
    """Batch-sized requests whose number crosses the line both ways, with and
    without the accept/reject step (its state passes from sweep to sweep),
    chunk ends within and at the ends of trajectories."""
    check([("i8", 60 + 28 * i, (8, 21, 64)[i % 3], 50 + 40 * (i % 9), ((1.1, 0.9), None, (1.0, 1.0))[i % 3]) for i in range(16)] +
          [("i8wide", 200 + 20 * i, 12, 300 - 20 * i, ((1.05, 0.95), None)[i % 2]) for i in range(6)], 22)
    check([("bf16hilo", 130 + 40 * i, (5, 40)[i % 2], 45 + 60 * (i % 4), None) for i in range(9)], 9)
    # admitted as others retire
    check([("i8", 100 + 13 * i, 16, 75 + 30 * (i % 4), (1.1, 0.9) if i % 2 else None) for i in range(24)], 12)


@pytest.mark.parametrize("n,N,R,most", [(4, 130, 16, 3.2), (12, 130, 64, 7.0)])
def test_few_small_16_bit_requests_share_launches(n, N, R, most):
    """16-bit requests of few columns are batched from a few on: n of them end
    before the launches of their own, one after the other, would."""
    from paper_2407_10205_amd import phia as P
    probs = [P.Problem(*make("bf16hilo", N, i % 3)) for i in range(n)]
    t = {}
    for m in (1, n):
        srv = P.Server(1 << 36, max_slots=64, chunk_steps=100)
        t[m] = []
        for _ in range(4):
            t0 = time.perf_counter()
            for k in [srv.submit(p, R, 1500, -(1 << 60), seed=1, **SCHED) for p in probs[:m]]:
                assert srv.wait(k, 60.0)["steps_used"] == 1500
            t[m].append(time.perf_counter() - t0)
        srv.close()
    for p in probs:
        p.close()
    print(n, N, R, "one", min(t[1]), "all", min(t[n]), "ratio", min(t[n]) / min(t[1]), flush=True)
    assert min(t[n]) < most * min(t[1])
