"""Recorded sweeps: steps of an anneal recorded by a stream capture and
replayed several times, with eager launches of the same state and unrelated
work between the replays, equal the same steps run eagerly, on every sweep
whose workgroups exchange their spins through tagged words."""
import numpy as np
import pytest

from paper_2407_10205_amd import instances as inst

pytestmark = pytest.mark.gpu

# sweep, path, N, replicas, recorded steps.  The words' tags repeat after 2^16
# steps in the split sweep; one and two steps leave the tags that a replay
# waits for in the words; 4100 replicas run in several uneven passes.
CASES = [("split,16", "i8", 600, 20, 1), ("split,4", "bf16hilo", 300, 9, 2), ("split,16", "i8", 600, 20, 65536),
         ("split,16", "i8", 600, 20, 65537), ("split,4,3", "i8", 300, 4100, 30), ("split,4", "i8", 900, 6, 40),
         ("pp,4", "i8", 300, 40, 1), ("pp,4", "i8", 300, 40, 25), ("1,8,0", "i8", 400, 33, 1)]


@pytest.mark.parametrize("spec,path,N,R,n", CASES)
def test_replays_equal_eager_runs(monkeypatch, spec, path, N, R, n):
    import torch
    from paper_2407_10205_amd import phia as P
    f, bits = {"i8": (5, 8), "bf16hilo": (9, 16)}[path]
    J, h = inst.sk_gauss_fixed(N, 3, frac_bits=f, bits=bits)
    sched = dict(eps=0.2, gamma=1.0, beta0=0.01, beta1=0.3, refresh_L=9, seed=2)
    k0, k1 = 5, 5 + n
    monkeypatch.setenv("PHIA_GEOMETRY", spec)
    print("replays", spec, path, N, R, n, flush=True)

    def state(p):
        return p.replica_best() + p.get_state()[:2]

    ref = []
    with P.Problem(J, h, frac_bits=f, path=path) as q:
        q.start(R, k1, **sched)
        assert q.info()["group"] > 1
        q.run(k0)
        for i in range(4):
            if i:
                q.set_state(ref[-1][3], ref[-1][4], k0)
            q.run(k1)
            ref.append(state(q))
    st = torch.cuda.Stream()
    with P.Problem(J, h, frac_bits=f, path=path, stream=st.cuda_stream) as p:
        p.start(R, k1, **sched)
        p.run(k0)
        p.sync()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            p.run(k1)
        for i in range(4):
            if i == 2:  # an eager run between replays
                p.set_state(ref[1][3], ref[1][4], k0)
                p.run(k1)
            else:
                g.replay()
            torch.cuda.synchronize()
            for a, b in zip(ref[i], state(p)):
                assert np.array_equal(a, b), i
            torch.randn(512, 512, device="cuda").matmul(torch.randn(512, 512, device="cuda")).sum().item()


def test_error_word_of_a_replay_is_reported(monkeypatch):
    """A wait that gives up in a replay (the error word raised from the host's
    hook, recorded with the sweep) is reported by the next synchronisation,
    also when an earlier one has found the word clear."""
    import torch
    from paper_2407_10205_amd import phia as P
    J, h = inst.sk_gauss_fixed(600, 3, frac_bits=5, bits=8)
    monkeypatch.setenv("PHIA_GEOMETRY", "split,16")
    st = torch.cuda.Stream()
    with P.Problem(J, h, frac_bits=5, path="i8", stream=st.cuda_stream) as p:
        p.start(20, 30, eps=0.2, gamma=1.0, beta0=0.01, beta1=0.3, refresh_L=9, seed=2)
        p.run(5)
        p.sync()
        p.raise_error_word()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            p.run(30)
        p.sync()
        g.replay()
        torch.cuda.synchronize()
        with pytest.raises(P.PhiaError) as e:
            p.best()
        assert e.value.code == -6
