"""The FP64 matrix-core step kernels at the edges of their row and column tiles: row counts around
multiples of 16, around the sizes where a wavefront takes more row tiles (256, 512), column counts that
leave a tile partly filled. Series terms against the VALU kernel, which the oracle pins
(test_gpu_graph_and_tiles), at the tolerance of tests/parity_util.py."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp

from parity_util import SERIES_TOL, series_mismatch


@pytest.mark.parametrize("M,N,two_J,n_E", [(15, 9, 1, 1), (16, 16, 1, 3), (17, 5, 1, 11), (33, 30, 3, 40), (112, 20, 1, 5),
                                           (130, 128, 1, 9), (256, 6, 1, 3), (258, 8, 3, 1), (258, 64, 3, 31),
                                           (512, 5, 3, 2), (514, 6, 3, 3), (514, 64, 3, 31)])
def test_tiles_match_the_valu_kernel(M, N, two_J, n_E):
    L = wp.Lattice(M, N, two_J=two_J, swave_only=True)
    L.pseudostates(kind="yamaguchi") if two_J == 3 else L.pseudostates()
    L.build_perm("fp64")
    Es = np.linspace(2.0, 30.0, n_E)
    kw = dict(tol=1e-14, accept=1e-14, max_iter=16, allow_noconv=True)
    ref = L.solve(Es, "fp64", step_tile="valu", **kw)
    for tile in ("auto", "mfma8", "mfma16", "rows"):
        got = L.solve(Es, "fp64", step_tile=tile, **kw)
        for k in range(n_E):
            d = series_mismatch(got.series(k), ref.series(k), grow=False)
            assert d <= SERIES_TOL, (tile, k, d)
