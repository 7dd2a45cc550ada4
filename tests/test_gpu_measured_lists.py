"""FP64 lists long enough for the real form that hold a measurement, a reset or a post-selection keep vec(rho): the whole
list gives the bits of its launches one by one, also in expectations that are nothing but rounding (<ZZ> of a
teleportation) and in a rare branch.  Operations that only look similar do not count as one."""
import sys

import numpy as np
import pytest

from paper_2404_13184_amd import tanq as T
from paper_2404_13184_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def outputs(n, ops, mode):
    """(state, expectations) of the list applied whole and launch by launch, and its launches."""
    c = T.Circuit(n, ops)
    f = c.fuse(mode, "f64")
    out = []
    for whole in (True, False):
        d = T.DM(n, "f64")
        pos = 0
        for r in [sum(f.launches())] if whole else f.launches():
            d.apply_fused(f, pos, pos + r)
            pos += r
        out.append((d.read(), d.expect_paulis(W.zz_paulis(n))))
        d.free()
    launches = len(f.launches())
    f.free()
    c.free()
    return out, launches


def same_bits(a, b):
    return all(np.array_equal(x.view(np.uint8), y.view(np.uint8)) for x, y in zip(a, b))


@pytest.mark.parametrize("n,width", [(11, 2), (11, 3), (12, 2)])
def test_teleportation_keeps_its_bits(n, width):
    say("teleportation n=%d width=%d" % (n, width))
    (whole, pieces), launches = outputs(n, W.teleport_layers(n, 8, n, 1e-3, 1e-2), width)
    assert launches >= 12
    assert same_bits(whole, pieces)


CLEARING = {
    "dephase": (W.dephase(), 1),
    "reset": (W.reset(), 1),
    # the dephasing of a measurement as a mixture of I and Z
    "mixture": ([np.sqrt(0.5) * W.I2, np.sqrt(0.5) * W.PZ], 1),
    "agree": (W.agree_projector(), 2),
    "three": ([np.diag([1.0] * 7 + [0.0]), np.diag([0.0] * 7 + [1.0])], 3),
}
KEEPING = {
    "damping": (W.amplitude_damping(0.3), 1),
    "flip": ([np.sqrt(0.5) * W.I2, np.sqrt(0.5) * W.PX], 1),
    "cx": ([W.cx()], 2),
    "three": ([np.eye(8)[::-1]], 3),
    # no Kraus matrix has all rows, but every pair of rows is in one of them
    "pairs": ([np.diag([1.0, 1, 0, 0]), np.diag([0.0, 0, 1, 1]), np.diag([1.0, 0, 1, 0]), np.diag([0.0, 1, 0, 1]),
               np.diag([1.0, 0, 0, 1]), np.diag([0.0, 1, 1, 0])], 2),
}


@pytest.mark.parametrize("kind,name", [("clearing", k) for k in CLEARING] + [("keeping", k) for k in KEEPING])
def test_which_operations_count(kind, name):
    n = 11
    say("list with one operation: %s %s" % (kind, name))
    mats, j = (CLEARING if kind == "clearing" else KEEPING)[name]
    ops = W.random_u3_cx(n, 10, 4, 1e-3, 1e-2)
    ops.insert(len(ops) // 2, W.channel(mats, (2, 7, 4)[:j]))
    (whole, pieces), launches = outputs(n, ops, 3 if j == 3 else 2)
    assert launches >= 12
    assert np.abs(whole[0] - pieces[0]).max() <= 1e-12 * np.abs(pieces[0]).max()
    assert same_bits(whole, pieces) == (kind == "clearing")
