"""The few-channel product over 1 to 15 columns: every way to split them into passes, and row counts that
leave a pair of rows and a workgroup partly filled, column by column against the same energies solved one at
a time (one column a pass), at the tolerance of tests/parity_util.py."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp

from parity_util import SERIES_TOL, series_mismatch


@pytest.mark.parametrize("M,N,two_J", [(13, 11, 1), (13, 11, 3), (33, 31, 3), (30, 17, 1), (183, 183, 3)])
def test_columns_match_single_energies(M, N, two_J):
    L = wp.Lattice(M, N, two_J=two_J, swave_only=True)
    L.pseudostates(kind="yamaguchi") if two_J == 3 else L.pseudostates()
    L.build_perm("fp64")
    widths = (2, 3, 4, 5, 7, 8, 9, 12, 15) if M < 100 else (2, 3)
    Es = np.linspace(2.0, 30.0, max(widths))
    kw = dict(tol=1e-14, accept=1e-14, max_iter=12, allow_noconv=True)
    one = [L.solve(Es[k:k + 1], "fp64", **kw).series(0) for k in range(max(widths))]
    for n in widths:
        got = L.solve(Es[:n], "fp64", **kw)
        for k in range(n):
            d = series_mismatch(got.series(k), one[k], grow=False)
            assert d <= SERIES_TOL, (n, k, d)
    if M < 100:   # FP32 products of the refinement, whose FP64 residual decides when a column is done
        ref = [L.solve(Es[k:k + 1], "mixed_split", tol=1e-11).amplitude(0) for k in range(max(widths))]
        for n in (3, 6, 15):
            got = L.solve(Es[:n], "mixed_split", tol=1e-11)
            for k in range(n):
                a, b = got.amplitude(k)["A"], ref[k]["A"]
                assert np.abs(a - b).max() <= 1e-8 * np.abs(b).max(), (n, k)
