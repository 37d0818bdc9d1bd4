"""Anneals at the sizes that programs run, on the sweep that they take by
default, against the oracle in sampled replicas: the resident sweep with more
replicas than the CUs hold at once and at the last columns that one CU holds,
and the paired-wave form of the split sweep in two passes over its groups."""
import numpy as np
import pytest

from paper_2407_10205_amd import instances as inst

pytestmark = pytest.mark.gpu

# couplings, N, replicas, sweep, replicas per workgroup or group, compared replicas
CASES = [
    ("cut", 800, 1024, 5, 4, (0, 3, 4, 511, 512, 1020, 1023)),
    ("cut", 800, 1027, 5, 4, (0, 1, 513, 1023, 1024, 1026)),
    ("cut", 800, 4098, 5, 4, (0, 2047, 2048, 4095, 4096, 4097)),
    ("pm1", 833, 9, 5, 4, (0, 5, 8)),
    ("pm1", 848, 6, 5, 4, (0, 5)),
    ("pm1", 849, 6, 5, 4, (0, 5)),
    ("pm1", 864, 1030, 5, 4, (0, 3, 1023, 1029)),
    ("pm1", 865, 9, 6, 4, (0, 8)),
    ("fixed8", 512, 2050, 5, 4, (0, 1023, 1024, 2049)),
    # 25 groups of blocks in passes of sixteen; one block's last rows are padding
    ("fixed8", 2000, 397, 6, 16, (0, 15, 16, 255, 256, 271, 383, 384, 396)),
    ("fixed8", 1700, 512, 6, 16, (0, 7, 255, 256, 511)),
]


@pytest.mark.parametrize("family,N,R,kind,rows,sample", CASES)
def test_default_sweep_matches_oracle(family, N, R, kind, rows, sample):
    from oracle import oracle as O
    from paper_2407_10205_amd import phia as P
    f = 0
    if family == "cut":
        J, h = inst.er_maxcut(N, 0.06, 0)
    elif family == "pm1":
        J, h = inst.sk_pm1(N, N)[0], inst.random_field_pm1(N, N + 1)
    else:
        (J, h), f = inst.sk_gauss_fixed(N, 3, frac_bits=5, bits=8), 5
    size = 5.0 if f else 1.0
    T, L, b0, b1 = 40, 12, 0.02 / size, 0.6 / size
    print("default", family, N, R, flush=True)
    with P.Problem(J, h, frac_bits=f, path="i8") as p:
        p.start(R, T, 0.2, 1.0, beta0=b0, beta1=b1, refresh_L=L, seed=N + R)
        i = p.info()
        assert (i["sweep_kernel"], i["rows_per_block"]) == (kind, rows)
        for k in (17, T):
            p.run(k)
        E, S, K = p.replica_best()
        x, v, _ = p.get_state()
    Ji, hi = np.rint(J * 2**f).astype(np.int32), np.rint(h * 2**f).astype(np.int32)
    for r in sample:
        o = O.anneal(Ji, hi, f, 1, O.beta_linear(b0, b1, T), 0.2, 1.0, L, N + R, r0=r)
        assert E[r] == o.bestE[0] and K[r] == o.bestStep[0], r
        assert np.array_equal(S[r], o.bestS[0]), r
        assert np.array_equal(x[r].view(np.uint32), o.x[0].view(np.uint32)), r
        assert np.array_equal(v[r].view(np.uint32), o.v[0].view(np.uint32)), r
