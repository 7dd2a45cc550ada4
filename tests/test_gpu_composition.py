"""Composition of fused blocks on the GPU: operations of one, two and three qubits in every order of their
qubits, in blocks of every width within one list, against the product of their superoperators in NumPy."""
import numpy as np
import pytest

from paper_2404_13184_amd import tanq as T
from paper_2404_13184_amd import workloads as W

pytestmark = pytest.mark.gpu


def superop(op, pos, k):
    """S = sum conj(K) x K of an operation on the qubits pos of k (the first is the least significant)."""
    D, d = 1 << k, 1 << len(pos)
    S = np.zeros((D * D, D * D), dtype=np.complex128)
    for K in op.mats:
        F = np.zeros((D, D), dtype=np.complex128)
        for x in range(D):
            lx = sum(((x >> p) & 1) << t for t, p in enumerate(pos))
            rest = x & ~sum(1 << p for p in pos)
            for ly in range(d):
                F[rest | sum(((ly >> t) & 1) << p for t, p in enumerate(pos)), x] = np.asarray(K)[ly, lx]
        S += np.kron(F.conj(), F)
    return S


@pytest.mark.parametrize("seed,n,count", [(1, 3, 1), (2, 3, 90), (3, 4, 70), (4, 5, 40)])
def test_composition_of_mixed_operations(seed, n, count):
    print("[gpu-case] composition n=%d operations=%d" % (n, count), flush=True)
    rng = np.random.default_rng(seed)
    ops = []
    for _ in range(count):
        j = int(rng.choice([1, 2, 2, 3]))
        qs = [int(q) for q in rng.permutation(n)[:j]]
        if j < 3 and rng.random() < 0.3:
            ops.append(W.channel(W.depolarizing(0.05, j), qs))
        else:
            ops.append(W.gate(W.random_unitary(rng, 1 << j), qs))
    c = T.Circuit(n, ops)
    block, nb = c.plan(3)
    f = c.fuse(3, "f64")
    assert f.count == nb
    for b in range(nb):
        k, Q, S = f.get(b)
        loc = {q: i for i, q in enumerate(Q)}
        want = np.eye(1 << (2 * k), dtype=np.complex128)
        for op, ob in zip(ops, block):
            if ob == b:
                want = superop(op, [loc[q] for q in op.qubits], k) @ want
        # at most 90 operations of at most 64 products an entry, entries at most 1: 90 * 64 * 1.1e-16
        assert np.abs(S - want).max() <= 1e-12, b
    f.free()
    c.free()
