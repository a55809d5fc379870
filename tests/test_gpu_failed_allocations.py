"""Calls repeated after a device allocation failed (WP_ENOMEM): each allocation of a call in turn is refused once, and the
same call then gives the results of a lattice that never saw a failure."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp
    from paper_1404_5253_amd.serve import BatchBackend, slot_bytes

    class Refusing(wp.TorchAllocator):
        """Refuses the allocation `refuse` steps ahead (negative: none)."""

        def __init__(self):
            self.refuse = -1
            super().__init__()

        def _alloc(self, nbytes, ctx):
            self.refuse -= 1
            return None if self.refuse == -1 else super()._alloc(nbytes, ctx)


def lattice(channels):
    two_J, j_max = {"doublet": (1, 0), "pw10": (1, 1)}[channels]
    L = wp.Lattice(10, 9, two_J=two_J, j_max=j_max or 1, swave_only=j_max == 0)
    L.pseudostates()
    return L


def serve(L, mode):
    b = BatchBackend(L, slots=2, hbm_budget=2 * slot_bytes(L, mode), terms=8, tol=1e-8, accept=1e-6, mode=mode,
                     stream=wp.current_stream())
    got = {}
    b.admit_many([3.0, 14.1])
    while len(got) < 2:
        got.update({s: r["A"] for s, r in b.step()})
    b.close()
    return np.array([got[0], got[1]])


def solve(L, mode):
    sol = L.solve([3.0, 14.1], mode, tol=1e-8, accept=1e-6)
    return np.array([sol.amplitude(k)["A"] for k in range(2)])


CALLS = {
    "fp64": lambda L: solve(L, "fp64"),
    "mixed_split": lambda L: solve(L, "mixed_split"),
    "batch_fp64": lambda L: serve(L, "fp64"),
    "batch_mixed": lambda L: serve(L, "mixed"),
    "resolvent": lambda L: L.resolvent(14.1, 0),
}


def refuse_each(monkeypatch, make, call, most=80):
    """call(make()) with its k-th allocation refused, k = 0, 1, ...; returns the number of allocations."""
    expected = call(make())
    for k in range(most):
        alloc = Refusing()
        monkeypatch.setattr(wp, "TorchAllocator", lambda: alloc)
        L = make()
        alloc.refuse = k
        try:
            first = call(L)
        except wp.WpError as e:
            assert e.status == wp.WP_ENOMEM, (k, e)
            alloc.refuse = -1
            assert np.array_equal(call(L), expected), k
        else:   # fewer than k + 1 allocations
            assert alloc.refuse >= 0
            assert np.array_equal(first, expected)
            return k
    raise AssertionError(f"more than {most} allocations")


@pytest.mark.parametrize("channels", ["doublet", "pw10"])
@pytest.mark.parametrize("call", sorted(CALLS))
def test_call_after_a_refused_allocation(monkeypatch, channels, call):
    def make():
        L = lattice(channels)
        L.build_perm("fp64")
        return L
    assert refuse_each(monkeypatch, make, CALLS[call]) > 10


def build(L, precision="fp64"):
    L.build_perm(precision)
    rp, col, val = L.export_perm()
    return np.concatenate([rp, col, val.ravel()])


@pytest.mark.parametrize("channels", ["doublet", "pw10"])   # both kinds of build: candidate values, fused
def test_build_after_a_refused_allocation(monkeypatch, channels):
    assert refuse_each(monkeypatch, lambda: lattice(channels), build) > 10


@pytest.mark.parametrize("channels", ["doublet", "pw10"])
def test_no_solve_on_a_failed_rebuild(monkeypatch, channels):
    alloc = Refusing()
    monkeypatch.setattr(wp, "TorchAllocator", lambda: alloc)
    L = lattice(channels)
    L.build_perm("fp64")
    expected = solve(L, "fp64")
    alloc.refuse = 0   # the FP32 values, whose build drops the FP64 ones
    with pytest.raises(wp.WpError) as e:
        L.build_perm("fp32")
    assert e.value.status == wp.WP_ENOMEM
    for mode in ("fp64", "mixed_split"):
        with pytest.raises(wp.WpError) as e:
            solve(L, mode)
        assert e.value.status == wp.WP_ENOTREADY, mode
    L.build_perm("fp64")
    assert np.array_equal(solve(L, "fp64"), expected)
