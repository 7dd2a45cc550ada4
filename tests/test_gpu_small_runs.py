"""Runs of superoperators on small states: one launch per run must give the bits of the blocks applied
one by one (passes and runs switched off).  Sizes: from one qubit (a tile of four elements) over partial
tiles (up to 5 qubits in FP64), one full tile, to the largest state that uses runs (9 qubits in FP64, 10
in FP32); modes with blocks of one, two and three qubits, mixed, in any qubit order; lists longer than
the 32 blocks of one launch."""
import sys

import numpy as np
import pytest

from paper_2404_13184_amd import tanq as T
from paper_2404_13184_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def ops_for(n, seed):
    rng = np.random.default_rng(seed)
    ops = []
    for _ in range(5):
        perm = [int(q) for q in rng.permutation(n)]
        for q in perm:
            ops.append(W.gate(W.random_unitary(rng, 2), (q,)))
            ops.append(W.channel(W.amplitude_damping(0.1), (q,)))
        if n >= 2:
            ops.append(W.gate(W.random_unitary(rng, 4), perm[:2]))
            ops.append(W.channel(W.depolarizing(0.02, 2), perm[-2:]))
        if n >= 3:
            ops.append(W.gate(W.random_unitary(rng, 8), perm[:3]))
    return ops


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10])
def test_runs_give_the_bits_of_single_applies(n, prec):
    say("runs n=%d %s" % (n, prec))
    if n > 9 and prec == "f64":
        pytest.skip("FP64 states of 10 qubits use passes")
    ops = ops_for(n, n)
    old = T.tanq_get_pass_limit()
    try:
        T.tanq_set_pass_limit(1)  # one by one
        for mode in (T.TANQ_FUSE_NONE, T.TANQ_FUSE_PAPER, 1, 2, 3):
            c = T.Circuit(n, ops)
            f = c.fuse(mode, prec)
            outs = []
            for limit in (1, 8):
                T.tanq_set_pass_limit(limit)
                d = T.DM(n, prec)
                d.fill_random(n)
                d.apply_fused(f)
                outs.append(d.read())
                d.free()
            T.tanq_set_pass_limit(1)
            f.free()
            c.free()
            assert np.array_equal(outs[0].view(np.uint8), outs[1].view(np.uint8)), mode
    finally:
        T.tanq_set_pass_limit(old)
