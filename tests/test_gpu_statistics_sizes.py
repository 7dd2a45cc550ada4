"""Measurement statistics around the sizes where their kernels change: one workgroup up to 13 qubits, several
above; one chunk of 2^12 outcomes or many; up to 16384 shots in one workgroup; results of up to 2^17
shots in the handle's buffer.  Expected values from the gathered elements in numpy (FP64 sums of at most 2^15
terms of size 2^-n: relative 1e-12 leaves three orders of magnitude)."""
import sys

import numpy as np
import pytest

from paper_2404_13184_amd import tanq as T
from paper_2404_13184_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def through_readout(p, p01, p10):
    for t in range(len(p01)):
        v = p.reshape(-1, 2, 1 << t)
        p = np.stack([(1 - p10[t]) * v[:, 0] + p01[t] * v[:, 1], p10[t] * v[:, 0] + (1 - p01[t]) * v[:, 1]], 1).reshape(-1)
    return p


@pytest.mark.parametrize("n,prec", [(1, "f64"), (2, "f32"), (5, "f64"), (10, "f32"), (11, "f64"), (12, "f32"),
                                    (13, "f64"), (13, "f32"), (14, "f32"), (15, "f32")])
def test_statistics(oracle_mod, n, prec):
    say("statistics n=%d %s" % (n, prec))
    rng = np.random.default_rng(n)
    d = T.simulate(n, W.random_u3_cx(n, 2, 60 + n, 1e-2, 2e-2, gamma=1e-2), 2, prec)
    dim = 1 << n
    s = np.arange(dim, dtype=np.uint64)
    raw = d.gather(s * np.uint64(dim + 1)).real.astype(np.float64)
    p, tr = d.probs()
    assert abs(tr - raw.sum()) <= 1e-12
    assert np.abs(p - raw / raw.sum()).max() <= 1e-12 * p.max()
    q, _ = d.probs(renormalize=False)
    assert np.array_equal(q, raw)
    p01, p10 = rng.uniform(0, 0.05, n), rng.uniform(0, 0.03, n)
    want = through_readout(raw / raw.sum(), p01, p10)
    assert np.abs(d.probs_readout(p01, p10) - want).max() <= 1e-12 * want.max()
    for shots in (1, 1000, 16384, 16385, (1 << 17) + 5):
        got = d.sample(shots, 9, p01, p10)
        ref, _, _ = oracle_mod.sample(want, shots, 9)
        assert got.size == shots and got.max() < dim
        assert np.count_nonzero(got.astype(np.int64) != ref) <= 2  # draws at a CDF edge
    assert np.array_equal(d.sample(5000, 3), T.tanq_sample_noalloc(d.h, 5000, 3))
    strings = ["".join(rng.choice(list("IXYZ"), size=n)) for _ in range(70)]
    got = d.expect_paulis(strings)
    for st, v in zip(strings, got):
        xm = sum(1 << t for t, c in enumerate(st) if c in "XY")
        zm = sum(1 << t for t, c in enumerate(st) if c in "YZ")
        e = d.gather(s + ((s ^ np.uint64(xm)) << np.uint64(n))).astype(np.complex128)
        sign = np.array([1 - 2 * (bin(int(x) & zm).count("1") & 1) for x in s])
        assert abs(v - (1j ** st.count("Y")) * (sign * e).sum()) <= 1e-12
    assert np.array_equal(d.expect_paulis(strings[:1]), got[:1]) or n > 11  # more workgroups per string when few
    for k in range(1, min(4, n) + 1):
        keep = [int(x) for x in rng.permutation(n)[:k]]
        red = d.reduced(keep)
        free = s[(s & np.uint64(sum(1 << x for x in keep))) == 0]
        dep = [np.uint64(sum(((a >> t) & 1) << x for t, x in enumerate(keep))) for a in range(1 << k)]
        for a in range(1 << k):
            b = (a * 5 + 1) % (1 << k)
            e = d.gather((free | dep[a]) + ((free | dep[b]) << np.uint64(n))).astype(np.complex128)
            assert abs(red[a, b] - e.sum()) <= 1e-12
    d.free()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_superoperator_slots(oracle_mod, prec):
    """Twenty queued superoperators of each width reuse the handle's slots (and travel with the launch at width
    1): every one of them is the one that was passed."""
    n = 6
    rng = np.random.default_rng(8)
    for k in (1, 2, 3):
        say("slots k=%d %s" % (k, prec))
        ops = [W.gate(W.random_unitary(rng, 1 << k), [int(q) for q in rng.permutation(n)[:k]]) for _ in range(20)]
        with T.DM(n, prec) as d:
            for op in ops:
                u = op.mats[0]
                s = np.kron(u.conj(), u)
                d.apply_superop(op.qubits, s)
                s[:] = np.nan  # the caller's array is its own again
            got = oracle_mod.vec_to_matrix(d.read().astype(np.complex128), n)
        assert np.abs(got - oracle_mod.run(n, ops)).max() <= (1e-12 if prec == "f64" else 1e-5)
