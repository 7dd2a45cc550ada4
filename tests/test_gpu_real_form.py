"""FP64 states in real (Pauli) form: the server's kernels at the edges of their tiles.

A full tile holds 2^12 elements (6 qubits): below it tiles are partial (2-5 qubits, with fewer than
16 groups per column block), above it a state has several tiles.  The output kernel has two LDS
sizes (up to 12 qubits, up to 14).  Circuits mix one-, two- and three-qubit operations on
unordered qubits, complex amplitudes, a non-unitary gate and a projector, and ask for strings with
Y.  FP64 composition and products of at most 64 terms over at most 40 operations: relative errors
of a few 1e-15 per entry of w, so 1e-12 leaves two orders of magnitude."""
import sys

import numpy as np
import pytest

from paper_2404_13184_amd import tanq as T
from paper_2404_13184_amd import workloads as W

pytestmark = pytest.mark.gpu

MiB = 1 << 20


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def mixed_ops(n, seed, width):
    rng = np.random.default_rng(seed)
    ops = []
    for _ in range(8):
        for q in rng.permutation(n):
            ops.append(W.gate(W.random_unitary(rng, 2), (int(q),)))
            ops.append(W.channel(W.amplitude_damping(0.05), (int(q),)))
        perm = [int(q) for q in rng.permutation(n)]
        ops.append(W.gate(W.random_unitary(rng, 4), perm[:2]))
        ops.append(W.channel(W.depolarizing(0.02, 2), perm[1::-1]))
        if n >= 3 and width == 3:
            ops.append(W.gate(W.random_unitary(rng, 8), perm[:3]))
    ops.append(W.gate(np.array([[0.9, 0.1j], [0.2, 0.8]]), (0,)))  # not unitary
    ops.append(W.channel([np.diag([1.0, 0, 0, 1.0])], (n - 1, 0)))  # lowers the trace
    return ops


@pytest.mark.parametrize("width", [2, 3])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 8])
def test_server_real_form_matches_oracle(oracle_mod, n, width):
    if n < width:
        pytest.skip("narrower than the fusion width")
    say("real form n=%d width=%d" % (n, width))
    ops = mixed_ops(n, 10 * n + width, width)
    rng = np.random.default_rng(n)
    strings = ["".join(rng.choice(list("IXYZ"), size=n)) for _ in range(20)] + ["Y" * n, "I" * n]
    with T.Server(64 * MiB, max_slots=2, prec="f64", width=width, steps_per_launch=4) as srv:
        res = srv.wait(srv.submit(n, ops, probs=True, paulis=strings))
    want = oracle_mod.run(n, ops)
    p, tr = oracle_mod.diag(want)
    assert abs(res["trace"] - tr) <= 1e-12
    assert np.abs(res["probs"] - p / tr).max() <= 1e-12
    for s, v in zip(strings, res["pauli"]):
        assert abs(v - oracle_mod.expect_pauli(want, s).real) <= 1e-12


@pytest.mark.parametrize("n", [12, 13])
def test_server_outputs_of_large_states(n):
    """Both LDS sizes of the output kernel, against the single-state path."""
    say("real form outputs n=%d" % n)
    ops = mixed_ops(n, n, 2)[:60]
    strings = W.z_paulis(n) + ["Y" * n, "XY" + "Z" * (n - 2)]
    with T.Server(2048 * MiB, max_slots=2, prec="f64", width=2, steps_per_launch=4) as srv:
        res = srv.wait(srv.submit(n, ops, probs=True, paulis=strings))
    d = T.simulate(n, ops, 2, "f64")
    p, tr = d.probs()
    e = d.expect_paulis(strings).real
    d.free()
    assert abs(res["trace"] - tr) <= 1e-12
    assert np.abs(res["probs"] - p).max() <= 1e-12
    assert np.abs(res["pauli"] - e).max() <= 1e-12
