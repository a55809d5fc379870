"""Which FP64 step kernel a call takes by default decides last bits of the series (the tiles of 2 and 4 columns fuse
another product of G1 t than those of 8 and 16): the wide tiles from 256 workgroups of 8 columns on, the narrow ones
below, bit for bit against the same solve with the kernel asked for by name."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp


@pytest.mark.parametrize("M,N,n_E,tile", [(60, 60, 16, "rows"), (24, 50, 20, "rows"), (24, 64, 15, "rows"),   # 240, 250, 240
                                          (24, 64, 16, "mfma8"), (33, 60, 18, "mfma8")])                      # 256, 270
def test_default_tile_by_workgroups(M, N, n_E, tile):
    L = wp.Lattice(M, N, two_J=1)   # 2 channels: workgroups 2 ceil(N n_E / 8)
    L.pseudostates()
    L.build_perm("fp64")
    Es = np.linspace(2.0, 40.0, n_E)
    kw = dict(tol=1e-8, accept=1e-6, max_iter=40, allow_noconv=True)
    a, b = L.solve(Es, "fp64", **kw), L.solve(Es, "fp64", step_tile=tile, **kw)
    for k in range(n_E):
        assert np.array_equal(a.series(k, 0), b.series(k, 0)), (k, tile)
