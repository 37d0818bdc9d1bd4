"""The split sweep (k_sweep_split) against the oracle, bit for bit: one, two
and three int8 planes and sparse rows at the edges of its variants (k blocks, waves, members
of a group), four and sixteen replicas per group, ragged replica counts and
several passes over the replica blocks, launches that begin and end between
momentum draws and past the wrap of the tags, both kick factors, the
allocation-free call, and the rules that choose it."""
import os

import numpy as np
import pytest

from paper_2407_10205_amd import instances as inst

pytestmark = pytest.mark.gpu

FRAC = {"i8": (5, 8), "bf16hilo": (9, 16), "fp32": (12, 20), "ell": (6, 16)}


@pytest.fixture
def geometry(monkeypatch):
    return lambda spec: monkeypatch.setenv("PHIA_GEOMETRY", spec)


def instance(path, N, seed):
    """Fixed-point couplings that use the path's whole width."""
    f, bits = FRAC[path]
    if path == "ell":  # uneven rows of 0 to about a dozen couplings
        rs = np.random.default_rng(seed)
        A = np.triu((rs.random((N, N)) < min(1.0, 4.0 / N)) * rs.integers(-2**15 + 1, 2**15, (N, N)), 1)
        return (A + A.T) / 2.0**f, rs.integers(-300, 300, N) / 2.0**f, f
    J, h = inst.sk_gauss_fixed(N, seed, frac_bits=f, bits=bits)
    if path != "i8" and N > 3:  # the planes' extreme values
        top = {"bf16hilo": 32639, "fp32": 8355711}[path] / 2.0**f
        if path == "bf16hilo" or N < 500:  # row sums below 2^24
            J[0, 3] = J[3, 0] = top
            J[1, 2] = J[2, 1] = -top
    return J, h, f


def check(O, J, h, f, sched, T, rows, E, S, K, x, v):
    Ji, hi = np.rint(J * 2**f).astype(np.int32), np.rint(h * 2**f).astype(np.int32)
    for r in rows:
        o = O.anneal(Ji, hi, f, 1, O.beta_linear(sched["beta0"], sched["beta1"], T), sched["eps"], sched["gamma"],
                     sched["refresh_L"], sched["seed"], r0=r, deriv=sched["deriv"])
        assert E[r] == o.bestE[0] and K[r] == o.bestStep[0], r
        assert np.array_equal(S[r], o.bestS[0]), r
        assert np.array_equal(x[r].view(np.uint32), o.x[0].view(np.uint32)), r
        assert np.array_equal(v[r].view(np.uint32), o.v[0].view(np.uint32)), r


# path, N, replicas, replicas per group, members (0: as chosen)
CASES = [("i8", 5, 3, 4, 2), ("i8", 200, 7, 4, 0), ("i8", 300, 19, 16, 7), ("i8", 1024, 5, 4, 8), ("i8", 1025, 17, 16, 0),
         ("i8", 1536, 3, 4, 0), ("i8", 1537, 16, 16, 13), ("i8", 2048, 5, 16, 0), ("i8", 300, 4100, 4, 3),
         ("bf16hilo", 17, 6, 4, 4), ("bf16hilo", 256, 18, 16, 0), ("bf16hilo", 257, 5, 4, 0), ("bf16hilo", 512, 33, 16, 5),
         ("bf16hilo", 1000, 7, 4, 8), ("bf16hilo", 1025, 4, 4, 0), ("bf16hilo", 1537, 17, 16, 0),
         ("bf16hilo", 2048, 3, 4, 32), ("fp32", 2, 1, 4, 2), ("fp32", 33, 20, 16, 0), ("fp32", 256, 5, 4, 0),
         ("fp32", 257, 17, 16, 0), ("fp32", 512, 6, 4, 32), ("fp32", 768, 4, 4, 0), ("fp32", 769, 18, 16, 0),
         ("fp32", 1025, 3, 4, 0), ("fp32", 1537, 17, 16, 0), ("fp32", 2000, 2, 4, 0), ("fp32", 40, 2100, 16, 2),
         ("ell", 20, 3, 4, 2), ("ell", 300, 9, 4, 0), ("ell", 700, 6, 4, 11), ("ell", 1030, 5, 4, 5), ("ell", 4000, 3, 4, 0),
         ("ell", 2000, 140, 4, 0), ("ell", 100, 700, 4, 5)]


@pytest.mark.parametrize("path,N,R,rows,G", CASES)
def test_split_matches_oracle(geometry, path, N, R, rows, G):
    from oracle import oracle as O
    from paper_2407_10205_amd import phia as P
    J, h, f = instance(path, N, N + R)
    T = 23 + N % 3
    sched = dict(eps=0.2, gamma=0.8, beta0=0.01, beta1=0.3, refresh_L=(1, 7, 40)[N % 3], seed=N + 3,
                 deriv="poly2" if N % 4 == 1 else "tanh")
    geometry(f"split,{rows},{G}")
    print("split", path, N, R, rows, G, flush=True)
    with P.Problem(J, h, frac_bits=f, path=path) as p:
        p.start(R, T, **sched)
        info = p.info()
        assert info["sweep_kernel"] == 6 and info["rows_per_block"] == rows and (G == 0 or info["group"] == G)
        for k in (1, 8, T - 2, T):
            p.run(k)
        E, S, K = p.replica_best()
        x, v, _ = p.get_state()
    check(O, J, h, f, sched, T, sorted({0, 1 % R, min(R - 1, 16), R // 2, R - 1}), E, S, K, x, v)


@pytest.mark.parametrize("R,seq", [(40, 65520), (2100, 65500)])
def test_split_tags_past_their_wrap(geometry, R, seq):
    """Sequence numbers that pass 2^16 between and within launches, with one
    pass over the replica blocks and with several uneven ones (whose idle
    groups' words the host clears): the run of a fresh problem."""
    from paper_2407_10205_amd import phia as P
    J, h, f = instance("bf16hilo", 70, 3)
    T = 90
    sched = dict(eps=0.2, gamma=1.0, beta0=0.01, beta1=0.3, refresh_L=11, seed=5)
    geometry("split,4,2")
    out = []
    for s in (None, seq):
        with P.Problem(J, h, frac_bits=f, path="bf16hilo") as p:
            p.start(R, T, **sched)
            if s is not None:
                p.set_exchange_seq(s)
                with pytest.raises(P.PhiaError):
                    p.set_exchange_seq(65521)
            for k in (5, 6, 40, T):
                p.run(k)
            out.append(p.replica_best() + p.get_state()[:2])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("path", ["i8", "bf16hilo", "fp32", "ell"])
def test_split_noalloc(geometry, path):
    """The allocation-free call equals phia_anneal."""
    import torch
    from paper_2407_10205_amd import phia as P
    J, h, f = instance(path, 600, 4)
    sched = dict(eps=0.2, gamma=1.0, beta0=0.01, beta1=0.3, refresh_L=9, seed=2)

    def bufs(R, Np):
        x, v = (torch.full((R, Np), 7.0, device="cuda") for _ in range(2))
        return x, v, torch.zeros(R, dtype=torch.int64, device="cuda"), torch.zeros((R, Np), dtype=torch.int8, device="cuda"), \
            torch.zeros(R, dtype=torch.int64, device="cuda")

    geometry("split,4" if path == "ell" else "split,16")
    with P.Problem(J, h, frac_bits=f, path=path) as p:
        p.anneal(50, 60, **sched)
        assert p.info()["sweep_kernel"] == 6
        E, S, K = p.replica_best()
        for _ in range(2):
            b = bufs(50, p.info()["Np"])
            p.anneal_noalloc(50, 60, **sched, **dict(zip(("x", "v", "bestE", "bestS", "bestStep"), (t.data_ptr() for t in b))))
            assert np.array_equal(b[2].cpu().numpy(), E) and np.array_equal(b[4].cpu().numpy(), K)
            assert np.array_equal(b[3].cpu().numpy()[:, :600], S)


def test_split_under_stream_capture():
    """An FP32 run recorded into a graph records the sweep without an
    exchange; state and records equal an eager run's."""
    import torch
    from paper_2407_10205_amd import phia as P
    J, h, f = instance("fp32", 150, 4)
    sched = dict(eps=0.2, gamma=1.0, beta0=0.01, beta1=0.3, refresh_L=9, seed=2)
    with P.Problem(J, h, frac_bits=f, path="fp32") as q:
        q.anneal(10, 40, **sched)
        assert q.info()["sweep_kernel"] == 6
        ref = q.replica_best() + q.get_state()[:2]
    st = torch.cuda.Stream()
    with P.Problem(J, h, frac_bits=f, path="fp32", stream=st.cuda_stream) as p:
        p.start(10, 40, **sched)
        p.run(25)
        p.sync()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            p.run(40)
        g.replay()
        torch.cuda.synchronize()
        got = p.replica_best() + p.get_state()[:2]
        assert p.info()["sweep_kernel"] == 6
    for a, b in zip(ref, got):
        assert np.array_equal(a, b)


def test_split_wait_that_gives_up(geometry):
    """The device error word raised from the host: phia_sync reports it, a
    fresh handle works."""
    from paper_2407_10205_amd import phia as P
    J, h, f = instance("bf16hilo", 300, 4)
    sched = dict(eps=0.2, gamma=1.0, beta0=0.01, beta1=0.3, refresh_L=9, seed=2)
    geometry("split")
    p = P.Problem(J, h, frac_bits=f, path="bf16hilo")
    p.start(64, 200, **sched)
    p.raise_error_word()
    p.run(200)
    with pytest.raises(P.PhiaError) as e:
        p.sync()
    assert e.value.code == -6
    p.close()
    with P.Problem(J, h, frac_bits=f, path="bf16hilo") as q:
        q.anneal(64, 50, **sched)
        q.sync()


def test_split_is_the_default_where_it_applies():
    """Default geometry: FP32 and BF16 hi/lo past 128 columns, int8 past the
    resident sweep, up to Np = 2048; not with traces or the accept/reject
    step, nor where a coupling or a row sum is too large for the planes."""
    from paper_2407_10205_amd import phia as P

    def kind(J, h=None, path="auto", trace=False, R=8, **kw):
        with P.Problem(J, h, path=path) as p:
            p.set_trace(trace)
            p.anneal(R, 4, 0.2, 1.0, beta0=0.01, beta1=0.02, **kw)
            return p.info()["sweep_kernel"]

    Jw = instance("fp32", 100, 1)[0]
    assert kind(Jw) == 6 and kind(Jw, trace=True) == 4 and kind(Jw, mh=(1.0, 1.0)) == 4 and kind(Jw, ikick=True) == 4
    Jb = instance("bf16hilo", 129, 1)[0]
    assert kind(Jb) == 6 and kind(Jb, trace=True) == 0 and kind(Jb, mh=(1.0, 1.0)) == 0
    assert kind(instance("bf16hilo", 128, 1)[0]) == 0
    Jb[0, 5] = Jb[5, 0] = 32640 / 512.0  # past two planes
    assert kind(Jb) == 0
    Jw = inst.sk_gauss_fixed(100, 1, frac_bits=12, bits=16)[0]
    Jw[0, 5] = Jw[5, 0] = 8355712 / 4096.0  # past three
    assert kind(Jw) == 4
    assert kind(inst.sk_gauss_fixed(513, 1)[0]) == 6
    assert kind(inst.sk_pm1(897, 1)[0]) == 6
    assert kind(inst.sk_gauss_fixed(2049, 1)[0]) != 6
    J, h = inst.regular3_pm1(600, 1)
    assert kind(J, h) == 6 and kind(J, h, trace=True) == 4 and kind(J, h, mh=(1.0, 1.0)) == 4
    assert kind(J, h, R=256) == 4  # more than eight column blocks to a member
    J, h = inst.regular3_pm1(4000, 1)
    assert kind(J, h, R=64) == 6 and kind(J, h, R=65) == 4  # more blocks than run at once
    J, h = inst.regular3_pm1(500, 1)
    assert kind(J, h, path="ell") == 4
