"""Which sweep an anneal takes by default, beside the rules that the tests of
the single sweeps check: streams, replica counts, settings and files that
have a say in it, on both sides of each line."""
import numpy as np
import pytest

from paper_2407_10205_amd import instances as inst

pytestmark = pytest.mark.gpu

SCHED = dict(eps=0.2, gamma=1.0, beta0=0.01, beta1=0.02, refresh_L=25)


def couplings(path, N):
    """Couplings that the path holds and no narrower one does."""
    if path == "ell":
        return inst.regular3_pm1(N, 1)
    f, bits = {"i8": (5, 8), "bf16hilo": (9, 16), "fp32": (12, 20)}[path]
    return inst.sk_gauss_fixed(N, 1, frac_bits=f, bits=bits)


def kind(path, N, R, stream=None, setup=None, **kw):
    from paper_2407_10205_amd import phia as P
    with P.Problem(*couplings(path, N), path=path, stream=stream) as p:
        if setup:
            setup(p)
        p.anneal(R, 4, **SCHED, **kw)
        return p.info()["sweep_kernel"]


@pytest.mark.parametrize("path,N,R,alone,beside", [
    ("ell", 1000, 64, 6, 4), ("ell", 4000, 16, 6, 4), ("bf16hilo", 192, 1024, 6, 0), ("bf16hilo", 192, 1025, 6, 6),
    ("bf16hilo", 193, 16, 6, 6), ("fp32", 48, 1024, 6, 4), ("fp32", 48, 1025, 6, 6), ("fp32", 49, 16, 6, 6),
    ("i8", 900, 16, 6, 6), ("i8", 300, 16, 5, 5)])
def test_anneals_on_streams_of_their_own(path, N, R, alone, beside):
    """On a stream of its own an anneal keeps the sweep without an exchange
    where several side by side finish sooner by it."""
    import torch
    print("stream", path, N, R, flush=True)
    assert kind(path, N, R) == alone
    assert kind(path, N, R, stream=torch.cuda.Stream().cuda_stream) == beside


@pytest.mark.parametrize("path,N,R,want", [
    ("bf16hilo", 129, 2048, 6), ("bf16hilo", 129, 2049, 0), ("bf16hilo", 192, 4096, 0), ("bf16hilo", 193, 4096, 6),
    ("fp32", 16, 20000, 6), ("fp32", 200, 4100, 6), ("i8", 640, 2100, 6)])
def test_split_past_one_pass(path, N, R, want):
    """More replicas than one pass of the split sweep holds."""
    print("passes", path, N, R, flush=True)
    assert kind(path, N, R) == want


@pytest.mark.parametrize("path,N,R", [("bf16hilo", 1000, 128), ("bf16hilo", 1500, 40)])
def test_incremental_product_on_request(path, N, R):
    """phia_set_incremental(1) takes a sweep with the flip-incremental product
    where there is one; the results are those of the default choice."""
    from paper_2407_10205_amd import phia as P
    out = []
    for on in (None, True):
        print("incremental", path, N, R, on, flush=True)
        with P.Problem(*couplings(path, N), path=path) as p:
            if on:
                p.set_incremental(True)
            p.anneal(R, 60, **dict(SCHED, beta1=3.0))
            i, st = p.info(), p.incremental_stats()
            assert (i["sweep_kernel"], i["incremental"]) == ((0, 1) if on else (6, 0))
            assert (st[0] + st[1] > 0) == bool(on)
            out.append(p.replica_best() + p.get_state()[:2])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("path,N,R,kw,want", [
    ("fp32", 300, 16, {}, 6), ("fp32", 300, 500, {}, 6), ("i8", 300, 64, {}, 5), ("i8", 300, 64, dict(ikick=True), 5),
    ("i8", 900, 16, dict(ikick=True), 6)])
def test_autotune_times_every_sweep(path, N, R, kw, want):
    """The autotuner finds the sweep that is fastest by far (FP32: split
    against VALU; also after an anneal with the initial kick, whose only sweep
    is the VALU one), and later anneals take it."""
    from paper_2407_10205_amd import phia as P
    print("autotune", path, N, R, kw, flush=True)
    with P.Problem(*couplings(path, N), path=path) as p:
        p.anneal(R, 4, **SCHED, **kw)
        assert p.autotune(R, 100) > 0
        p.anneal(R, 40, **SCHED)
        assert p.info()["sweep_kernel"] == want
        a = p.replica_best()
    with P.Problem(*couplings(path, N), path=path) as p:
        p.anneal(R, 40, **SCHED)
        for x, y in zip(a, p.replica_best()):
            assert np.array_equal(x, y)


def test_tune_cache_of_older_sweeps_is_skipped(monkeypatch, tmp_path):
    """A cache line written before the split sweep does not pin the sweep that
    it took the place of, but holds where neither it nor the resident sweep
    applies; one written now is used."""
    from paper_2407_10205_amd import phia as P
    f = tmp_path / "tune"
    monkeypatch.setenv("PHIA_TUNE_CACHE", str(f))
    Np = 960
    f.write_text(f"phia-tune4 2 {Np} 16 1 2 1 60 1 0 2.6\n")
    assert kind("i8", 900, 16) == 6
    with P.Problem(*couplings("i8", 900), path="i8") as p:
        assert p.info()["Np"] == Np and p.autotune(16, 50) > 0
        tuned = p.info()["sweep_kernel"]
    tag, path, np_, r, k, rows = f.read_text().split("\n")[1].split()[:6]
    assert (int(path), int(np_), int(r), int(k)) == (2, Np, 16, tuned)
    f.write_text(f"{tag} 2 {Np} 16 6 16 1 12 1 1 2.0\n")
    with P.Problem(*couplings("i8", 900), path="i8") as p:
        p.anneal(16, 4, **SCHED)
        i = p.info()
        assert (i["sweep_kernel"], i["rows_per_block"], i["group"]) == (6, 16, 12)
    f.write_text("phia-tune4 2 2112 16 0 1 2 44 0 0 9.0\n")
    with P.Problem(*couplings("i8", 2100), path="i8") as p:
        p.anneal(16, 4, **SCHED)
        assert (p.info()["sweep_kernel"], p.info()["group"]) == (0, 44)


@pytest.mark.parametrize("N,most", [(40, 1024), (64, 1024), (65, 512), (256, 512), (257, 256), (384, 256), (385, 0)])
def test_row_sums_past_the_resident_sweep(N, most):
    """Row sums past 2^31 / (2 N): few replicas take the VALU sweep, from one
    more on a matrix-core one, and both give the oracle's results."""
    from oracle import oracle as O
    from paper_2407_10205_amd import phia as P
    J, h = inst.sk_pm1(N, 1)
    h = h.copy()
    h[3] = float(1 << 28)
    o = O.anneal(J.astype(np.int32), h.astype(np.int32), 0, 1, O.beta_linear(0.01, 0.02, 4), 0.2, 1.0, 25, 0)
    for R in sorted({1, most, most + 1} - {0}):
        print("row sums", N, R, flush=True)
        with P.Problem(J, h, path="i8") as p:
            p.anneal(R, 4, **SCHED)
            assert (p.info()["sweep_kernel"] == 4) == (R <= most), (R, p.info())
            E, S, K = p.replica_best()
        assert E[0] == o.bestE[0] and K[0] == o.bestStep[0] and np.array_equal(S[0], o.bestS[0])
