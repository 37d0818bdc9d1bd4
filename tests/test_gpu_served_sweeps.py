"""Served requests on the resident and split sweeps: few batch-sized requests
in launches of their own and more of them in the batched launch give the same
results, as do sizes on either side of every rule that picks a served
request's sweep."""
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
    if kind == "bf16hilo":
        return inst.sk_gauss_fixed(N, seed, frac_bits=9, bits=16)
    return inst.regular3_pm1(N, seed)


def serve(specs, slots):
    from paper_2407_10205_amd import phia as P
    srv = P.Server(1 << 36, max_slots=slots, chunk_steps=30)
    probs, tickets = [], []
    for i, (kind, N, R, mh) in enumerate(specs):
        J, h = make(kind, N, i)
        p = P.Problem(J, h)
        probs.append(p)
        tickets.append(srv.submit(p, R, 70, -(1 << 60), seed=i + 1, mh=mh, **SCHED))
    res = [srv.wait(t, 120.0) for t in tickets]
    spins = [srv.spins(t) for t in tickets]
    kinds = [p.info()["sweep_kernel"] for p in probs]
    srv.close()
    for p in probs:
        p.close()
    return [(r["state"], r["energy_units"], r["replica"], r["steps_used"]) for r in res], spins, kinds


def direct(spec, i):
    from paper_2407_10205_amd import phia as P
    kind, N, R, mh = spec
    J, h = make(kind, N, i)
    with P.Problem(J, h) as p:
        p.anneal(R, 70, seed=i + 1, mh=mh, **SCHED)
        e, s, r = p.best_exact()
        return e, r, p.replica_best()[1][r]


def check(specs, slots=32):
    from paper_2407_10205_amd import phia as P
    res, spins, kinds = serve(specs, slots)
    for i, spec in enumerate(specs):
        e, r, s = direct(spec, i)
        assert res[i] == (P.REQ_DONE, e, r, 70), spec
        assert np.array_equal(spins[i], s), spec
    return kinds


def test_few_and_many_batch_sized_requests():
    few = [("i8", 60 + 40 * i, 9 + i, None) for i in range(4)] + [("bf16hilo", 130 + 60 * i, 20, None) for i in range(4)]
    assert check(few) == [5] * 4 + [6] * 4
    check([("i8", 30 + 20 * i, 8, None) for i in range(12)] + [("bf16hilo", 129 + 20 * i, 5, None) for i in range(10)])


def test_rules_of_the_served_sweeps():
    specs = [("i8", 512, 8, None), ("i8", 520, 64, None), ("i8", 520, 32, None), ("i8", 832, 64, None), ("i8wide", 833, 16, None),
             ("i8wide", 700, 64, None), ("bf16hilo", 128, 8, None), ("bf16hilo", 700, 8, None), ("ell", 900, 8, None),
             ("i8", 300, 7, (1.1, 0.9)), ("i8", 700, 64, (1.1, 0.9)), ("bf16hilo", 300, 7, (1.1, 0.9))]
    assert check(specs) == [5, 5, 0, 5, 6, 0, 0, 6, 4, 5, 5, 0]
