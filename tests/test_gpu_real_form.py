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


# ---- long lists on single states (11 qubits and up, at least 12 launches) --------------------------


def hermitian_vec(n, seed):
    """vec of a random Hermitian matrix, exactly Hermitian in FP64 (not positive: linearity is enough)."""
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((1 << n, 1 << n)) + 1j * rng.standard_normal((1 << n, 1 << n))
    h = np.tril(a, -1)
    return (h + h.conj().T + np.diag(a.diagonal().real)).T.reshape(-1) / (1 << n)


def long_ops(n, seed):
    """Every width, with and without the top qubit, neighbours and distant pairs, unordered."""
    rng = np.random.default_rng(seed)
    ops = []
    for layer in range(6):
        perm = [int(q) for q in rng.permutation(n)]
        for q in perm:
            ops.append(W.gate(W.random_unitary(rng, 2), (q,)))
        ops.append(W.channel(W.amplitude_damping(0.1), (n - 1,)))
        for i in range(0, n - 1, 2):
            ops.append(W.gate(W.random_unitary(rng, 4), perm[i:i + 2]))
            ops.append(W.channel(W.depolarizing(0.01, 2), perm[i + 1:None if i == 0 else i - 1:-1]))
        ops.append(W.gate(W.random_unitary(rng, 8), perm[:3]))
    return ops


def apply_list(n, ops, mode, vec, limit, pieces=False):
    old = T.tanq_get_pass_limit()
    try:
        c = T.Circuit(n, ops)
        f = c.fuse(mode, "f64")
        T.tanq_set_pass_limit(limit)
        d = T.DM(n, "f64")
        if vec is not None:
            d.write(vec)
        runs = f.launches()
        if pieces:
            pos = 0
            for r in runs:
                d.apply_fused(f, pos, pos + r)
                pos += r
        else:
            d.apply_fused(f)
        out = d.read()
        d.free()
        f.free()
        c.free()
        return out, len(runs)
    finally:
        T.tanq_set_pass_limit(old)


# sums of at most 64 products per operation, some 100 operations and 2 n butterflies: a few 1e-14 of the
# largest entry at worst
LIST_TOL = 1e-12


@pytest.mark.parametrize("mode", [T.TANQ_FUSE_NONE, T.TANQ_FUSE_PAPER, 1, 2, 3])
@pytest.mark.parametrize("n", [11, 12, 13])
def test_long_list_on_hermitian_state(n, mode):
    """Real form against the blocks applied one by one (passes off, which keeps the complex form);
    the result is exactly Hermitian.  11, 12 and 13 qubits: one, two and two uneven steps of the
    transform beside its first."""
    say("real-form list n=%d mode=%d" % (n, mode))
    ops = long_ops(n, 100 * n + mode)
    vec = hermitian_vec(n, n)
    want, _ = apply_list(n, ops, mode, vec, 1)
    got, launches = apply_list(n, ops, mode, vec, 8)
    assert launches >= 12
    assert np.abs(got - want).max() <= LIST_TOL * np.abs(want).max()
    m = got.reshape(1 << n, 1 << n)
    assert np.array_equal(m, m.conj().T)


@pytest.mark.parametrize("limit", [2, 3, 8])
def test_long_list_pass_limits(limit):
    n = 11
    say("real-form list limit=%d" % limit)
    ops = W.random_u3_cx(n, 12, 5, 1e-3, 1e-2)
    want, _ = apply_list(n, ops, 2, None, 1)
    got, launches = apply_list(n, ops, 2, None, limit)
    assert launches >= 12
    assert np.abs(got - want).max() <= LIST_TOL * np.abs(want).max()


def test_list_of_eight_launches():
    """From 13 qubits on, lists of 8 launches are long enough."""
    n = 13
    say("real-form list of 8 launches")
    ops = W.random_u3_cx(n, 4, 3, 1e-3, 1e-2)
    vec = hermitian_vec(n, 4)
    want, _ = apply_list(n, ops, 2, vec, 1)
    got, launches = apply_list(n, ops, 2, vec, 8)
    assert 8 <= launches < 12
    assert np.abs(got - want).max() <= LIST_TOL * np.abs(want).max()
    m = got.reshape(1 << n, 1 << n)
    assert np.array_equal(m, m.conj().T)


@pytest.mark.parametrize("mode", [2, 3])
def test_long_list_whole_and_in_ranges(mode):
    """The whole list has an order of its own in the real form; ranges keep the list's."""
    n = 11
    say("real-form list in ranges, mode=%d" % mode)
    ops = long_ops(n, 17 + mode) + long_ops(n, 27 + mode)
    vec = hermitian_vec(n, 9)
    want, _ = apply_list(n, ops, mode, vec, 8)
    c = T.Circuit(n, ops)
    f = c.fuse(mode, "f64")
    runs = f.launches()
    cut = sum(runs[:len(runs) // 2])
    assert len(runs) // 2 >= 12
    d = T.DM(n, "f64")
    d.write(vec)
    d.apply_fused(f, 0, cut)
    d.apply_fused(f, cut, sum(runs))
    got = d.read()
    d.free()
    f.free()
    c.free()
    assert np.abs(got - want).max() <= LIST_TOL * np.abs(want).max()


def test_long_list_on_contiguous_tiles():
    """From 14 qubits on a workgroup's tiles follow one another."""
    n = 14
    say("real-form list n=14")
    ops = W.random_u3_cx(n, 6, 31, 1e-3, 1e-2)
    idx = np.random.default_rng(1).integers(0, 4 ** n, 5000).astype(np.uint64)
    old = T.tanq_get_pass_limit()
    out = []
    try:
        c = T.Circuit(n, ops)
        f = c.fuse(2, "f64")
        assert len(f.launches()) >= 12
        for limit in (1, 8):
            T.tanq_set_pass_limit(limit)
            d = T.DM(n, "f64")
            d.apply_fused(f)
            out.append((d.probs()[0], d.gather(idx)))
            d.free()
        f.free()
        c.free()
    finally:
        T.tanq_set_pass_limit(old)
    for want, got in zip(*out):
        assert np.abs(got - want).max() <= LIST_TOL * np.abs(want).max()


@pytest.mark.parametrize("spoil", ["all", "one", "diagonal", "huge", "nan"])
def test_long_list_on_other_states(spoil):
    """A state that is not Hermitian in a single element, or out of range, is applied in the complex form:
    bit for bit what the launches one by one give."""
    n = 11
    say("complex list, spoil=%s" % spoil)
    ops = W.random_u3_cx(n, 12, 6, 1e-3, 1e-2)
    vec = hermitian_vec(n, 3)
    if spoil == "all":
        vec = vec * (1 + 0.5j)
    elif spoil == "one":
        vec[(1 << n) * 777 + 1234] += 1e-17j * abs(vec[(1 << n) * 777 + 1234]) + 1e-18
    elif spoil == "diagonal":
        vec[((1 << n) + 1) * ((1 << n) - 1)] += 1e-300j
    elif spoil == "huge":
        vec[0] = 1e290
    else:
        vec[((1 << n) + 1) * 5] = np.nan
    got, launches = apply_list(n, ops, 2, vec, 8)
    want, _ = apply_list(n, ops, 2, vec, 8, pieces=True)
    assert launches >= 12
    assert np.array_equal(got.view(np.uint8), want.view(np.uint8))
