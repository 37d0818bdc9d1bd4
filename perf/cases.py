"""Timed cases of the annealer: what a user's program has it do.

Every case is one whole call sequence through the Python binding: an anneal
of one instance read out by `best` and `replica_best`, the allocation-free
anneal on the caller's device buffers, one launch of a batch plan with its
instances' best states, or a handful of requests through the server.  The
instances are those of `paper_2407_10205_amd.instances`, with the schedules
the benchmark uses (eps 0.2, gamma 1, beta up to 3 divided by the size of the
couplings).

A case's fields: kind ("anneal", "noalloc", "batch", "serve"), family (the
generator below), N, R replicas, T steps, L steps between momentum draws,
deriv ("tanh" or "poly2"), mh ("off", "fixed" or "adaptive": the accept/reject
step), ikick (the initial-kick variant), gamma, table (an explicit beta table
in place of the linear one); batches and servers add count and nmin, with N
the largest instance.
"""
import math

import numpy as np
import torch

from paper_2407_10205_amd import instances, phia


def _case(name, kind, family, N, R, T, L=25, deriv="tanh", mh="off", ikick=False, gamma=1.0, table=False, count=1,
          nmin=0):
    c = dict(kind=kind, family=family, N=N, R=R, T=T, L=L, deriv=deriv, mh=mh, ikick=ikick, gamma=gamma, table=table,
             count=count, nmin=nmin)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a tiny spin glass, where the latency of a step is all there is
        _case("sk16", "anneal", "sk", 16, 64, 1000, L=50),
        # one mid-size graph annealed by a few chains, as an interactive program does
        _case("maxcut256_r16", "anneal", "signed_cut", 256, 16, 1000),
        # an odd size with fractional couplings and fields, and the quadratic kick factor
        _case("spin437_poly2", "anneal", "fixed6", 437, 100, 1000, deriv="poly2"),
        # max-cut with many chains, on buffers that the caller keeps on the device
        _case("maxcut800", "noalloc", "cut", 800, 1024, 2000),
        # the same graph with the accept/reject step and an adaptive temperature
        _case("maxcut800_mh", "anneal", "cut", 800, 256, 1000, mh="adaptive"),
        # the large dense spin glass in 8-bit fixed point, many chains and few
        _case("sk2000", "anneal", "fixed8", 2000, 512, 1000),
        _case("sk2000_r16", "anneal", "fixed8", 2000, 16, 1000),
        # 16-bit fixed-point couplings
        _case("sk1000_16bit", "anneal", "fixed16", 1000, 128, 1000),
        # couplings beyond 16 bits
        _case("sk500_wide", "anneal", "wide", 500, 128, 400, table=True),
        # a large sparse graph
        _case("reg3_4000", "anneal", "reg3", 4000, 64, 1000),
        # many instances of uneven size annealed together by a plan that is kept
        _case("batch512", "batch", "mixed", 512, 32, 5000, count=512, nmin=32),
        # requests of uneven size and precision that arrive at a server together
        _case("serve20", "serve", "mixed", 2000, 64, 500, count=20, nmin=100),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# largest N of each family's draws
_NMAX = {"sk": 1000, "cut": 1000, "signed_cut": 1000, "fixed6": 2000, "fixed8": 2000, "fixed16": 2000, "wide": 1000,
         "reg3": 4000, "nae3sat": 400}


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choices(["anneal", "noalloc", "batch", "serve"], [10, 5, 3, 2])[0]
    L = rng.choice([10, 25, 25, 50, 100])
    deriv = rng.choices(["tanh", "poly2"], [4, 1])[0]
    gamma = rng.choices([1.0, round(rng.uniform(0.5, 2.0), 3)], [3, 1])[0]
    if kind == "batch":
        nmin = rng.choice([8, 32, 100])
        return _case(None, kind, rng.choice(["mixed", "mixed", "sk", "fixed6"]), rng.randint(nmin + 20, 512),
                     rng.choice([16, 32, 32, 50, 64]), rng.choice([500, 1000, 2000]), L, deriv, gamma=gamma,
                     count=_log_uniform(rng, 16, 384), nmin=nmin)
    if kind == "serve":
        return _case(None, kind, "mixed", _log_uniform(rng, 400, 2000), rng.choice([16, 32, 64]),
                     rng.choice([200, 300, 500]), L, deriv, count=rng.randint(4, 16), nmin=50)
    family = rng.choice(list(_NMAX))
    N = _log_uniform(rng, 8 if family not in ("reg3", "nae3sat") else 16, _NMAX[family])
    N += N % 2 if family == "reg3" else 0
    R = _log_uniform(rng, 1, 1024)
    mh, ikick = "off", False
    if kind == "anneal" and rng.random() < 0.15:
        mh = rng.choice(["fixed", "adaptive"])
    elif family in ("wide", "sk") and N <= 512 and rng.random() < 0.25:
        ikick = True
    # no more spin-updates and products than the largest listed cases
    cap = min(8e8 / (N * R), 1.5e12 / (N * N * max(R, 16)))
    if family == "wide" or ikick:
        cap = min(cap, 6e9 / (N * N * max(R, 16)))
    T = int(max(20, min(_log_uniform(rng, 200, 2000), cap)))
    return _case(None, kind, family, N, R, T, L, deriv, mh, ikick, gamma, table=rng.random() < 0.2)


def _instance(family, N, seed):
    """(J, h, size of the couplings) of one instance."""
    if family == "sk":
        return (*instances.sk_pm1(N, seed), 1.0)
    if family == "cut":
        return (*instances.er_maxcut(N, 0.06, seed), 1.0)
    if family == "signed_cut":
        return (*instances.er_maxcut(N, 0.06, seed, signed=True), 1.0)
    if family == "fixed6":
        return (*instances.uniform_fixed(N, seed, frac_bits=6), 1.0)
    if family == "fixed8":
        return (*instances.sk_gauss_fixed(N, seed, frac_bits=5, bits=8), 5.0)
    if family == "fixed16":
        return (*instances.sk_gauss_fixed(N, seed, frac_bits=12, bits=16), 5.0)
    if family == "wide":
        return (*instances.sk_gauss_fixed(N, seed, frac_bits=14, bits=17), 5.0)
    if family == "reg3":
        return (*instances.regular3_pm1(N, seed), 1.0)
    if family == "nae3sat":
        return (*instances.nae_3_sat(N, seed)[:2], 1.0)
    raise ValueError(family)


def _schedule(case, size):
    s = dict(eps=0.2, gamma=case["gamma"], refresh_L=case["L"], deriv=case["deriv"])
    b0, b1 = 0.1 / size, 3.0 / size
    if case["table"]:
        s["betas"] = np.geomspace(b0, b1, case["T"]).astype(np.float32)
    else:
        s["beta0"], s["beta1"] = b0, b1
    if case["mh"] != "off":
        s["mh"] = (1.0, 1.0) if case["mh"] == "fixed" else (1.02, 0.98)
    if case["ikick"]:
        s["ikick"] = True
    return s


def _members(case):
    """Family and size of every instance of a batch or a server's queue (the
    same for every seed: the outputs of two passes have one shape)."""
    g = instances.rng(case["N"] * 1000 + case["nmin"])
    out = []
    for i in range(case["count"]):
        if case["kind"] == "batch":
            N = int(g.integers(case["nmin"], case["N"] + 1))
            family = ("sk", "reg3")[i % 2] if case["family"] == "mixed" else case["family"]
        else:
            N = int(round(math.exp(g.uniform(math.log(case["nmin"]), math.log(case["N"])))))
            family = ("cut", "reg3", "fixed8", "fixed16")[i % 4]
        out.append((family, N + (N % 2 if family == "reg3" else 0)))
    return out


class State:
    """What the program keeps between passes; device objects go with it."""

    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        for name in ("server", "plan"):
            if hasattr(self, name):
                getattr(self, name).close()
        for p in getattr(self, "problems", ()):
            p.close()


def prepare(case, seed):
    kind, R, T = case["kind"], case["R"], case["T"]
    # chains of another seed, and another instance of the same family
    chain_seed = (seed * 0x9E3779B1 + 17) & 0xFFFFFFFF
    if kind in ("anneal", "noalloc"):
        J, h, size = _instance(case["family"], case["N"], seed)
        # |J| past 16 bits for certain, so that every seed takes the same arithmetic
        if case["family"] == "wide" and case["N"] > 1:
            J[0, 1] = J[1, 0] = 2.5
        p = phia.Problem(J, h)
        st = State(kind=kind, problems=[p], R=R, T=T, seed=chain_seed, sched=_schedule(case, size))
        if kind == "noalloc":
            Np = p.info()["Np"]
            st.x = torch.empty((R, Np), dtype=torch.float32, device="cuda")
            st.v = torch.empty_like(st.x)
            st.E = torch.empty(R, dtype=torch.int64, device="cuda")
            st.S = torch.empty((R, Np), dtype=torch.int8, device="cuda")
            st.K = torch.empty(R, dtype=torch.int64, device="cuda")
        return st
    problems, scheds = [], []
    for i, (family, N) in enumerate(_members(case)):
        J, h, size = _instance(family, N, seed * 4096 + i)
        problems.append(phia.Problem(J, h, defer_upload=(kind == "serve")))
        scheds.append(_schedule(case, size))
    st = State(kind=kind, problems=problems, R=R, T=T, scheds=scheds,
               seeds=[chain_seed + i for i in range(len(problems))])
    if kind == "batch":
        st.plan = phia.Batch(problems, [R] * len(problems), [T] * len(problems), scheds)
    else:
        st.server = phia.Server(8 << 30, max_slots=64, chunk_steps=100)
    return st


def run(st):
    if st.kind == "anneal":
        p = st.problems[0]
        p.anneal(st.R, st.T, seed=st.seed, **st.sched)
        energy, spins = p.best()
        E, S, K = p.replica_best()
        return {"energy": energy, "spins": spins, "E": E, "S": S, "K": K}
    if st.kind == "noalloc":
        e, r = st.problems[0].anneal_noalloc(st.R, st.T, x=st.x.data_ptr(), v=st.v.data_ptr(),
                                             bestE=st.E.data_ptr(), bestS=st.S.data_ptr(),
                                             bestStep=st.K.data_ptr(), seed=st.seed, **st.sched)
        return {"energy": e, "replica": r, "x": st.x, "v": st.v, "E": st.E, "S": st.S, "K": st.K}
    if st.kind == "batch":
        st.plan.launch(st.seeds)
        st.plan.sync()
        best = [p.best() for p in st.problems]
        return {"energy": np.array([e for e, _ in best]), "spins": np.concatenate([s for _, s in best])}
    # targets below any energy: every request uses its whole budget of steps
    tickets = [st.server.submit(p, st.R, st.T, -(1 << 60), seed=sd, **sc)
               for p, sd, sc in zip(st.problems, st.seeds, st.scheds)]
    res = [st.server.wait(t) for t in tickets]
    return {"energy": np.array([r["energy_units"] for r in res], dtype=np.int64),
            "steps": np.array([r["steps_used"] for r in res], dtype=np.int64),
            "spins": np.concatenate([st.server.spins(t) for t in tickets])}


def work(case):
    """Couplings and fields read once, states and records written once; per
    spin-update two operations per coupling and the 33 (tanh; 14 for the
    quadratic) of the drift, the readout, the energy and the kick."""
    def one(family, N):
        deg = {"cut": 0.06 * N, "signed_cut": 0.06 * N, "reg3": 3.0, "nae3sat": min(N - 1.0, 12.0)}.get(family, N - 1.0)
        width = {"fixed16": 2, "wide": 4}.get(family, 1)
        per = 2.0 * deg + (33 if case["deriv"] == "tanh" else 14)
        return case["R"] * case["T"] * N * per, N * deg * width + 4 * N + case["R"] * (N * 9 + 16)

    if case["kind"] in ("anneal", "noalloc"):
        flops, nbytes = one(case["family"], case["N"])
    else:
        parts = [one(*m) for m in _members(case)]
        flops, nbytes = sum(p[0] for p in parts), sum(p[1] for p in parts)
    return {"bytes": float(nbytes), "flops": float(flops)}


def exact(case, seed):
    """None: a chain of hundreds of binary32 steps is chaotic, so its end
    point and its integer records have no value in 64 bits to compare with."""
    return None
