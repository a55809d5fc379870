"""The many-channel block-CSR products at the edges of their column windows (spmm_mfma.h): windows of
4, 8, 16 and 32 columns, full, partly filled and repeated, one wavefront and several per block row.

FP64 series terms against the oracle at the tolerance of tests/parity_util.py; lattices of more than
16384 rows against the passes of 4 columns (spmm_cols above the column count), which the oracle
pins on the small lattices, at the same tolerance; the FP32 products through the mixed solve against
the FP64 amplitudes at 1e-6 (test_gpu_parity's bound for the mixed modes)."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp

from oracle import pipeline
from parity_util import SERIES_TOL, series_mismatch

SPECS = {
    "pw18": pipeline.Spec(M=6, N=7, two_J=1, j_max=2, swave_only=False, pot="mt"),    # 2 open channels
    "pw14": pipeline.Spec(M=7, N=5, two_J=3, j_max=1, swave_only=False, pot="mt"),    # 3 open channels
}


def lattice(M, N, two_J, j_max, precision="fp64"):
    L = wp.Lattice(M, N, two_J=two_J, j_max=j_max, swave_only=False)
    L.pseudostates()
    L.build_perm(precision)
    return L


@pytest.fixture(scope="module")
def systems():
    out = {}
    for name, s in SPECS.items():
        sysm = pipeline.build_system(s)
        out[name] = (sysm, sysm.P0geo.full(sysm.C), lattice(s.M, s.N, s.two_J, s.j_max))
    return out


@pytest.mark.parametrize("name,n_E", [("pw14", 1), ("pw18", 3), ("pw18", 4), ("pw14", 3), ("pw18", 8), ("pw18", 9),
                                      ("pw14", 11)])
def test_windows_match_oracle(systems, name, n_E):
    s, P0, L = systems[name]
    Es = np.linspace(2.0, 40.0, n_E)
    sol = L.solve(Es, "fp64", tol=1e-12, accept=1e-6, max_iter=300)
    mixed = L.solve(Es, "mixed_split", tol=1e-9, accept=1e-6)
    for k in {0, n_E // 2, n_E - 1}:
        ref = pipeline.solve_energy(s, Es[k], P0full=P0)
        for b, r in enumerate(ref["series"]):
            assert series_mismatch(sol.series(k, b), r) <= SERIES_TOL, (name, n_E, k, b)
        assert np.max(np.abs(mixed.amplitude(k)["A"] - sol.amplitude(k)["A"])) <= 1e-6, (name, n_E, k)


@pytest.mark.parametrize("n_E", [1, 4])
def test_one_wavefront_per_row(n_E):
    L = lattice(130, 128, 1, 1)
    Es = np.linspace(3.0, 30.0, n_E)
    kw = dict(tol=1e-6, accept=1e-4, max_iter=60)
    got, ref = L.solve(Es, "fp64", **kw), L.solve(Es, "fp64", spmm_cols=1 << 20, **kw)
    mixed = L.solve(Es, "mixed_split", tol=1e-9, accept=1e-6)
    exact = L.solve(Es, "fp64", tol=1e-10, accept=1e-6, max_iter=400)
    for k in range(n_E):
        for b in range(2):
            assert series_mismatch(got.series(k, b), ref.series(k, b), grow=False) <= SERIES_TOL, (n_E, k, b)
        assert np.max(np.abs(mixed.amplitude(k)["A"] - exact.amplitude(k)["A"])) <= 1e-6, (n_E, k)
