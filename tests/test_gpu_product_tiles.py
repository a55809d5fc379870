"""The few-channel products of 16 and more columns (tiles of 16 columns and 16 rows, 8 blocks of a row a turn),
plain and with the Arnoldi sums of the default cycle (other cycles and 4 blocks a turn: test_gpu_arnoldi_cycles):
column counts around the tiles, rows around the workgroups, one and two channels. FP64 series terms column by
column against one energy at a time at the tolerance of tests/parity_util.py; refinement amplitudes, whose FP64
residual decides when a column is done, against one energy at a time at 1e-8."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp

from parity_util import SERIES_TOL, series_mismatch


@pytest.mark.parametrize("M,N,two_J,n_E", [(5, 3, 1, 17), (4, 4, 3, 16), (13, 11, 1, 33), (33, 31, 3, 15 + 16),
                                           (16, 17, 1, 64), (66, 65, 3, 20), (66, 65, 1, 70)])
def test_columns_match_single_energies(M, N, two_J, n_E):
    L = wp.Lattice(M, N, two_J=two_J, swave_only=True)
    L.pseudostates(kind="yamaguchi") if two_J == 3 else L.pseudostates()
    L.build_perm("fp64")
    Es = np.linspace(2.0, 30.0, n_E)
    kw = dict(tol=1e-14, accept=1e-14, max_iter=12, allow_noconv=True)
    got = L.solve(Es, "fp64", **kw)
    mix = L.solve(Es, "mixed_split", tol=1e-11)
    for k in sorted({0, 1, 14, 15, 16, n_E // 2, n_E - 2, n_E - 1} & set(range(n_E))):
        one = L.solve(Es[k:k + 1], "fp64", **kw)
        d = series_mismatch(got.series(k), one.series(0), grow=False)
        assert d <= SERIES_TOL, (k, d)
        a, b = mix.amplitude(k)["A"], L.solve(Es[k:k + 1], "mixed_split", tol=1e-11).amplitude(0)["A"]
        assert np.abs(a - b).max() <= 1e-8 * np.abs(b).max(), k
