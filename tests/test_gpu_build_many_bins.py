"""Builds of many momentum bins over few q bins, on both sides of the sizes from which the selection's rows no longer
fit the LDS and the build leaves the node tables (910 bins), with the smallest and the largest node table: every
stored block against the oracle, as in test_gpu_build_rows."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp

from oracle.perm import P0Lattice
from oracle import pipeline


@pytest.mark.parametrize("M,n_x,n_phi,weights", [(740, 8, 8, "unit"), (910, 8, 8, "unit"), (911, 8, 8, "unit"),
                                                 (600, 16, 8, "unit"), (910, 16, 8, "energy"), (1024, 8, 8, "unit")])
def test_many_bins_match_the_oracle(M, n_x, n_phi, weights):
    N = 2
    L = wp.Lattice(M, N, two_J=3, swave_only=True, n_x=n_x, n_phi=n_phi, weights=weights)
    L.build_perm("fp64")
    rp, col, val = L.export_perm()
    pe, qe = L.edges()
    s = pipeline.build_system(pipeline.Spec(M=2, N=2, two_J=3, pot="yamaguchi"))
    P = P0Lattice(pe, qe, s.P0geo.keys, n_x, n_phi, weights=weights)
    ref = s.C[0, 0, 0] * P.moms[:, 0]
    scale, R = np.abs(ref).max(), M * N
    got_k, ref_k = np.repeat(np.arange(R), np.diff(rp)) * R + col, P.rows * R + P.cols
    common, ig, ir = np.intersect1d(got_k, ref_k, assume_unique=True, return_indices=True)
    val = val.ravel()
    assert np.abs(val[ig] - ref[ir]).max() <= 1e-12 * scale
    for v, i in ((val, ig), (ref, ir)):
        rest = np.delete(v, i)
        assert rest.size == 0 or np.abs(rest).max() <= 1e-12 * scale
