"""The two forms of the persistent batch sweep against the oracle, bit for
bit: whole workgroups (a plan of few instances) and squads of eight waves (a
plan of more small instances than the CUs hold in a round of pairs), at the
edges of their column blocks (64 and 128 columns), of the two 16-replica
halves and of the momentum rounds."""
import numpy as np
import pytest

from paper_2407_10205_amd import instances as inst

pytestmark = pytest.mark.gpu

TEAM = [(1, 33), (64, 16), (65, 17), (128, 32), (129, 1), (256, 31), (257, 33), (320, 5), (384, 32), (385, 18),
        (448, 16), (449, 33), (512, 32)]
SQUAD = [(1, 1), (2, 33), (63, 16), (64, 17), (65, 32), (127, 15), (128, 33), (129, 32), (191, 1), (192, 20), (193, 48),
         (255, 16), (256, 33)]


@pytest.mark.parametrize("sizes,count", [(TEAM, len(TEAM)), (SQUAD, 800)], ids=["teams", "squads"])
def test_batch_forms_match_oracle(sizes, count):
    from oracle import oracle as O
    from paper_2407_10205_amd import phia as P
    specs, insts, probs, scheds = [], [], [], []
    for i in range(count):
        N, R = sizes[i % len(sizes)]
        T, L = 13 + i % 4, (1, 5, 6, 100)[(i // len(sizes)) % 4]
        J, h = inst.sk_pm1(N, 900 + i % len(sizes))
        h = inst.random_field_pm1(N, 70 + i % len(sizes)) if i % 2 else h
        specs.append((N, R, T))
        insts.append((J, h))
        probs.append(P.Problem(J, h, path="i8"))
        scheds.append(dict(eps=0.2, gamma=1.0 if i % 3 else 0.7, beta0=0.1, beta1=2.5, refresh_L=L,
                           deriv="poly2" if i % 5 == 4 else "tanh"))
    plan = P.Batch(probs, [s[1] for s in specs], [s[2] for s in specs], scheds)
    assert {p.info()["sweep_kernel"] for p in probs} == {3}
    for launch in range(2):  # the queue starts over at every launch
        seeds = [4000 * launch + i for i in range(count)]
        plan.launch(seeds)
        plan.sync()
        step = max(1, count // 130)
        for i in range(0, count, step):
            (N, R, T), (J, h), sc = specs[i], insts[i], scheds[i]
            E, S, K = probs[i].replica_best()
            x, v, _ = probs[i].get_state()
            print("instance", i, specs[i], flush=True)
            for r in {0, R // 2, R - 1}:
                o = O.anneal(J.astype(np.int32), h.astype(np.int32), 0, 1, O.beta_linear(0.1, 2.5, T), sc["eps"],
                             sc["gamma"], sc["refresh_L"], seeds[i], r0=r, deriv=sc["deriv"])
                assert E[r] == o.bestE[0] and K[r] == o.bestStep[0], (specs[i], r)
                assert np.array_equal(S[r], o.bestS[0]), (specs[i], r)
                assert np.array_equal(x[r].view(np.uint32), o.x[0].view(np.uint32)), (specs[i], r)
                assert np.array_equal(v[r].view(np.uint32), o.v[0].view(np.uint32)), (specs[i], r)
    plan.close()
    for p in probs:
        p.close()
