"""The resident sweep (k_sweep_res) against the oracle, bit for bit: int8 and
FP4 operands at the edges of its variants (columns per wave, k blocks, blocks
in LDS), ragged replica counts, launches that begin and end between momentum
draws, both kick factors, with and without the energy trace, and the
allocation-free call."""
import os

import numpy as np
import pytest

from paper_2407_10205_amd import instances as inst

pytestmark = pytest.mark.gpu

# (N, FP4 couplings, replicas)
SIZES = [(1, True, 1), (2, True, 9), (16, True, 5), (17, True, 4), (128, True, 3), (129, True, 6), (256, True, 4),
         (257, True, 5), (384, True, 2), (385, True, 3), (512, True, 4), (513, True, 3), (640, True, 5), (641, True, 2),
         (768, True, 4), (769, True, 3), (800, True, 6), (832, True, 3),
         (64, False, 5), (65, False, 4), (128, False, 3), (129, False, 2), (256, False, 5), (257, False, 3),
         (384, False, 4), (385, False, 2), (448, False, 3), (449, False, 5), (512, False, 2)]


@pytest.mark.parametrize("N,fp4,R", SIZES)
def test_resident_matches_oracle(N, fp4, R):
    import torch
    from oracle import oracle as O
    from paper_2407_10205_amd import phia as P
    if fp4:
        J, f = inst.sk_pm1(N, N)[0], 0
        h = inst.random_field_pm1(N, N + 1)
    else:
        (J, h), f = inst.uniform_fixed(N, N, frac_bits=6), 6
    T, L, deriv = 23 + N % 3, (1, 7, 40)[N % 3], "poly2" if N % 4 == 1 else "tanh"
    sched = dict(eps=0.2, gamma=1.0 if N % 2 else 0.8, beta0=0.1, beta1=2.5, refresh_L=L, seed=N + 3, deriv=deriv)
    os.environ["PHIA_GEOMETRY"] = "res"
    try:
        with P.Problem(J, h, frac_bits=f, path="i8") as p:
            print("resident", N, fp4, R, flush=True)
            p.set_trace(N % 2 == 0)
            p.start(R, T, **sched)
            assert p.info()["sweep_kernel"] == 5
            for k in (1, 8, T - 2, T):
                p.run(k)
            E, S, K = p.replica_best()
            x, v, _ = p.get_state()
            tr = p.trace(T) if N % 2 == 0 else None
            p.set_trace(False)
            Np = p.info()["Np"]
            bx, bv = (torch.full((R, Np), 7.0, device="cuda") for _ in range(2))
            bE, bK = (torch.zeros(R, dtype=torch.int64, device="cuda") for _ in range(2))
            bS = torch.zeros((R, Np), dtype=torch.int8, device="cuda")
            p.anneal_noalloc(R, T, x=bx.data_ptr(), v=bv.data_ptr(), bestE=bE.data_ptr(), bestS=bS.data_ptr(),
                             bestStep=bK.data_ptr(), **sched)
            assert np.array_equal(bE.cpu().numpy(), E) and np.array_equal(bK.cpu().numpy(), K)
            assert np.array_equal(bS.cpu().numpy()[:, :N], S) and not bS[:, N:].any()
            assert np.array_equal(bx.cpu().numpy()[:, :N].view(np.uint32), x.view(np.uint32)) and not bx[:, N:].any()
            assert np.array_equal(bv.cpu().numpy()[:, :N].view(np.uint32), v.view(np.uint32)) and not bv[:, N:].any()
    finally:
        del os.environ["PHIA_GEOMETRY"]
    Ji, hi = np.rint(J * 2**f).astype(np.int32), np.rint(h * 2**f).astype(np.int32)
    for r in range(R):
        o = O.anneal(Ji, hi, f, 1, O.beta_linear(0.1, 2.5, T), 0.2, sched["gamma"], L, N + 3, r0=r, deriv=deriv,
                     trace=True)
        assert E[r] == o.bestE[0] and K[r] == o.bestStep[0]
        assert np.array_equal(S[r], o.bestS[0])
        assert np.array_equal(x[r].view(np.uint32), o.x[0].view(np.uint32))
        assert np.array_equal(v[r].view(np.uint32), o.v[0].view(np.uint32))
        assert tr is None or np.array_equal(tr[r], o.Etrace[0])


@pytest.mark.parametrize("N,fp4,R", [(16, True, 5), (130, True, 4), (385, True, 6), (600, True, 3), (800, True, 4),
                                     (64, False, 3), (250, False, 5), (437, False, 4), (512, False, 2)])
def test_resident_accept_reject_matches_oracle(N, fp4, R):
    """The accept/reject step of the resident sweep: decisions, multipliers and
    rejected end points with launches that begin and end within trajectories
    and at their ends, traces on and off."""
    from oracle import oracle as O
    from paper_2407_10205_amd import phia as P
    if fp4:
        J, f = inst.er_maxcut(N, min(1.0, 8 / N), 3, signed=True)[0], 0
        h = inst.random_field_pm1(N, N + 1)
    else:
        (J, h), f = inst.uniform_fixed(N, N, frac_bits=6), 6
    T, L = 61, (7, 20)[N % 2]
    mh = (1.25, 0.8) if N % 3 else (1.0, 1.0)
    sched = dict(eps=0.25, gamma=1.0, beta0=0.05, beta1=1.5, refresh_L=L, seed=N + 3, deriv="poly2" if N % 4 == 1 else "tanh")
    os.environ["PHIA_GEOMETRY"] = "res"
    try:
        with P.Problem(J, h, frac_bits=f, path="i8") as p:
            print("accept/reject", N, fp4, R, flush=True)
            for _ in range(2):  # the second anneal starts on the first one's buffers
                p.set_trace(N % 2 == 0)
                p.start(R, T, mh=mh, **sched)
                assert p.info()["sweep_kernel"] == 5
                for k in (1, L, L + 1, 2 * L - 1, 2 * L, T):
                    p.run(k)
                E, S, K = p.replica_best()
                x, v, _ = p.get_state()
                acc, dec, lam = p.replica_mh()
                tr = p.trace(T) if N % 2 == 0 else None
    finally:
        del os.environ["PHIA_GEOMETRY"]
    Ji, hi = np.rint(J * 2**f).astype(np.int32), np.rint(h * 2**f).astype(np.int32)
    for r in range(R):
        o = O.anneal(Ji, hi, f, 1, O.beta_linear(0.05, 1.5, T), 0.25, 1.0, L, N + 3, r0=r, deriv=sched["deriv"], trace=True,
                     mh=mh)
        assert E[r] == o.bestE[0] and K[r] == o.bestStep[0] and np.array_equal(S[r], o.bestS[0])
        assert np.array_equal(x[r].view(np.uint32), o.x[0].view(np.uint32))
        assert np.array_equal(v[r].view(np.uint32), o.v[0].view(np.uint32))
        assert acc[r] == o.acc[0] and dec[r] == o.dec[0] and lam[r] == o.lam[0]
        assert tr is None or np.array_equal(tr[r], o.Etrace[0])


def test_resident_is_the_default_where_it_fits():
    """Default geometry: the resident sweep up to Np = 832 with FP4 couplings
    and 512 with int8 ones, between 65 and 256 columns up to a replica count;
    row sums past the exact range of its sums and larger instances take the
    other sweeps."""
    from paper_2407_10205_amd import phia as P

    def kind(J, h=None, R=8, **kw):
        with P.Problem(J, h, path="i8") as p:
            p.anneal(R, 4, 0.2, 1.0, beta0=0.1, beta1=1.0, **kw)
            return p.info()["sweep_kernel"]

    assert kind(inst.sk_pm1(832, 1)[0]) == 5
    assert kind(inst.sk_pm1(897, 1)[0]) != 5
    J8 = inst.uniform_fixed(512, 1, frac_bits=6)[0] * 64
    assert kind(J8) == 5
    assert kind(inst.uniform_fixed(513, 1, frac_bits=6)[0] * 64) != 5
    assert kind(J8, mh=(1.0, 1.0)) == 5
    for N, R in ((128, 4096), (129, 3072)):
        J = inst.sk_pm1(N, 1)[0]
        assert kind(J, R=R) == 5 and kind(J, R=R + 1) == 0
    J, h = inst.sk_pm1(40, 1)
    h = h.copy()
    h[3] = float(1 << 28)  # 2 N max_i(sum |J| + |h|) past 2^31
    assert kind(J, h) == 4
