"""Several threads, each on a stream of its own, whose first calls on one lattice come at the same time: the tables that
a first call makes are made once and are complete for all of them, on every stream."""
import threading

import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    import paper_1404_5253_amd as wp

CALLS = ["fp64", "mixed_split", "mixed", "fp64", "mixed_split", "resolvent"]


def lattice():
    L = wp.Lattice(24, 20, two_J=1, j_max=1, swave_only=False)
    L.pseudostates()
    L.build_perm("fp64")
    return L


def call(L, what):
    if what == "resolvent":
        return L.resolvent(14.1, 0)
    sol = L.solve([3.0, 14.1], what, tol=1e-8, accept=1e-6)
    return np.array([sol.amplitude(k)["A"] for k in range(2)])


def test_first_calls_at_the_same_time():
    expected = [call(lattice(), what) for what in CALLS]
    for trial in range(5):
        L = lattice()
        torch.cuda.synchronize()
        start, got = threading.Barrier(len(CALLS)), [None] * len(CALLS)

        def work(k):
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait()
                try:
                    got[k] = call(L, CALLS[k])
                except Exception as e:   # shown by the comparison below
                    got[k] = e

        threads = [threading.Thread(target=work, args=(k,)) for k in range(len(CALLS))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for what, a, b in zip(CALLS, got, expected):
            assert np.array_equal(a, b), (trial, what, a)
