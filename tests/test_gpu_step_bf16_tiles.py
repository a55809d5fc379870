"""The BF16 step of the mixed modes at the edges of its tiles: row counts around multiples of 16 and 32
and around the sizes where a wavefront takes more row tiles (256, 512), 8 and 16 columns per workgroup,
a tile of columns partly filled. The refined amplitudes against the FP64 path, at the 1e-6 that
test_gpu_parity holds the mixed modes to."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp


@pytest.mark.parametrize("M,N,two_J,n_E", [(15, 9, 1, 1), (16, 16, 1, 3), (17, 5, 1, 11), (33, 30, 3, 40), (49, 20, 1, 5),
                                           (130, 128, 1, 9), (256, 6, 1, 3), (258, 8, 3, 1), (258, 64, 3, 31),
                                           (512, 5, 3, 2), (514, 6, 3, 3)])
def test_tiles_match_fp64(M, N, two_J, n_E):
    L = wp.Lattice(M, N, two_J=two_J, swave_only=True)
    L.pseudostates(kind="yamaguchi") if two_J == 3 else L.pseudostates()
    L.build_perm("fp64")
    Es = np.linspace(2.0, 30.0, n_E)
    ref = L.solve(Es, "fp64", tol=1e-10, accept=1e-6, max_iter=400)
    for mode in ("mixed", "mixed_split"):
        if mode == "mixed_split" and M > 512:
            continue
        sol = L.solve(Es, mode, tol=1e-9, accept=1e-6, max_iter=400)
        for k in range(n_E):
            assert np.max(np.abs(sol.amplitude(k)["A"] - ref.amplitude(k)["A"])) <= 1e-6, (mode, k)
