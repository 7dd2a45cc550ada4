"""What an FP64 request is admitted by: its state in real form is 4^n doubles (at 11 qubits 32 MiB), so it fits a
budget that vec(rho) (64 MiB) would not, and what it takes is that and the operands."""
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


@pytest.mark.parametrize("width", [2, 3])
def test_state_in_real_form_fits(width):
    n = 11
    say("FP64 request of 11 qubits in 64 MiB, width=%d" % width)
    ops = W.random_u3_cx(n, 2, 5, 1e-3, 1e-2)
    with T.Server(64 * MiB, max_slots=2, prec="f64", width=width, steps_per_launch=2) as srv:
        res = srv.wait(srv.submit(n, ops, probs=True))
        assert srv.stats()["peak_bytes"] <= 48 * MiB
    d = T.simulate(n, ops, 2, "f64")
    assert np.abs(res["probs"] - d.probs()[0]).max() <= 1e-12
    d.free()

