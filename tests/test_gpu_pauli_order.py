"""The order in which a Pauli expectation is summed is part of its result: a value that vanishes by symmetry is the
rounding of that sum.  Parts of 256 elements (thread by thread, a tree over each wave, the waves one after the
other), added one after the other, whatever the split over workgroups: bit for bit what numpy gives in that order.
Sizes: one part, two, eight (one workgroup), nine and more (several), more elements than parts (many strings)."""
import sys

import numpy as np
import pytest

from paper_2404_13184_amd import tanq as T
from paper_2404_13184_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def in_order(v, count):
    """Sum of the float64 vector v for a call with `count` strings."""
    parts = min(max(1, v.size // 256), 512, (512 * 2 * 64) // (2 * count))
    x = np.zeros((max(1, -(-v.size // (parts * 256))), parts, 256))
    x.reshape(-1)[:v.size] = v
    acc = np.zeros((parts, 256))
    for row in x:
        acc = acc + row
    acc = acc.reshape(parts, 4, 64)
    while acc.shape[2] > 1:
        h = acc.shape[2] // 2
        acc = acc[:, :, :h] + acc[:, :, h:]
    total = 0.0
    for p in acc[:, :, 0]:
        t = 0.0
        for w in p:
            t += float(w)
        total += t
    return total


@pytest.mark.parametrize("n,prec,count", [(5, "f64", 1), (8, "f64", 7), (9, "f64", 8), (9, "f32", 8), (11, "f64", 10),
                                          (11, "f32", 70), (12, "f64", 11), (12, "f64", 300), (14, "f32", 1000)])
def test_expectations_keep_the_order_of_their_sum(n, prec, count):
    say("pauli order n=%d %s count=%d" % (n, prec, count))
    d = T.simulate(n, W.teleport_layers(n, 2, n, 1e-3, 1e-2), 2, prec)
    rng = np.random.default_rng(count)
    strings = W.zz_paulis(n) + ["".join(rng.choice(list("IXYZ"), size=n)) for _ in range(count)]
    strings = strings[:count]
    got = d.expect_paulis(strings)
    s = np.arange(1 << n, dtype=np.uint64)
    for i in list(range(min(count, n - 1))) + [count - 1]:
        st = strings[i]
        xm = sum(1 << t for t, c in enumerate(st) if c in "XY")
        zm = sum(1 << t for t, c in enumerate(st) if c in "YZ")
        e = d.gather(s + ((s ^ np.uint64(xm)) << np.uint64(n))).astype(np.complex128)
        sign = np.array([1 - 2 * (bin(int(x) & zm).count("1") & 1) for x in s])
        e = e * sign * (1j ** (st.count("Y") % 4))
        want = complex(in_order(e.real, count), in_order(e.imag, count))
        assert got[i] == want, (st, got[i], want)
    d.free()
