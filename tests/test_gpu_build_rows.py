"""The build from node tables at the edges of its row tiles and lists: rows around multiples of 64, more
rows with candidates in a box than one list holds (many momentum bins over few q bins), node counts that
leave a group of four partly filled, the largest node table. Every stored block against the oracle at the
tolerance of test_gpu_parity (1e-12 of the largest element; pairs below it may differ in being stored)."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp

from oracle.perm import P0Lattice
from oracle import pipeline


@pytest.mark.parametrize("M,N,two_J,n_x,n_phi,weights", [
    (2, 2, 3, 8, 8, "unit"), (63, 5, 3, 8, 8, "unit"), (64, 9, 1, 8, 8, "energy"), (65, 17, 3, 7, 3, "unit"),
    (129, 3, 3, 5, 5, "energy"), (200, 2, 3, 3, 1, "unit"), (301, 2, 3, 16, 8, "unit"), (300, 2, 1, 8, 8, "unit"),
    (7, 65, 3, 8, 8, "unit"), (40, 40, 1, 9, 7, "unit")])
def test_stored_blocks_match_the_oracle(M, N, two_J, n_x, n_phi, weights):
    L = wp.Lattice(M, N, two_J=two_J, swave_only=True, n_x=n_x, n_phi=n_phi, weights=weights)
    L.pseudostates(kind="yamaguchi") if two_J == 3 else L.pseudostates()
    L.build_perm("fp64")
    rp, col, val = L.export_perm()
    pe, qe = L.edges()
    s = pipeline.build_system(pipeline.Spec(M=2, N=2, two_J=two_J, pot="yamaguchi" if two_J == 3 else "mt"))
    P = P0Lattice(pe, qe, s.P0geo.keys, n_x, n_phi, weights=weights)
    ref = np.einsum("abm,nm->nab", s.C, P.moms)
    scale = np.abs(ref).max()
    R = M * N
    row = np.repeat(np.arange(R), np.diff(rp))
    got_k, ref_k = row * R + col, P.rows * R + P.cols
    assert np.all(np.diff(got_k) > 0)
    common, ig, ir = np.intersect1d(got_k, ref_k, assume_unique=True, return_indices=True)
    val = val.reshape(len(col), *ref.shape[1:])
    assert np.abs(val[ig] - ref[ir]).max() <= 1e-12 * scale
    for v, i in ((val, ig), (ref, ir)):
        rest = np.delete(v, i, axis=0)
        assert rest.size == 0 or np.abs(rest).max() <= 1e-12 * scale
    assert L.perm_stats["blocks"] == len(col)
    again = L.build_perm("fp64")   # the second build runs with the first one's capacities
    assert again["blocks"] == len(col) and np.array_equal(L.export_perm()[2].reshape(val.shape), val)
