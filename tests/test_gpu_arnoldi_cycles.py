"""The fused Arnoldi product on tiles of 16 columns (k_spmm_arn_tiles) and the Gram-Schmidt passes, over the cycle
lengths the autotuner tries and the longest one (up to 8 and up to 16 basis vectors per lane), with 8 and with 4 blocks
of a row in flight (2 channels: more than 1024 workgroups), and with more than 32768 cells, where a workgroup takes
more rows so that the partial sums fit. Split mode, amplitudes against FP64 at test_gpu_parity's 1e-6."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp


@pytest.mark.parametrize("M,N,two_J,n_E,cycles", [
    (20, 17, 1, 17, (3, 4, 8, 9, 12, 16)),   # 2 channels, few workgroups
    (20, 17, 3, 33, (8, 12, 16)),            # 1 channel
    (100, 100, 1, 64, (8, 16)),              # 1252 workgroups: 4 blocks in flight
    (186, 179, 3, 16, (8, 16)),              # 33294 cells
    (20, 17, 1, 3, (4, 8, 12, 16)),          # few columns: product, then k_sub_dots
])
def test_cycles_match_fp64(M, N, two_J, n_E, cycles):
    L = wp.Lattice(M, N, two_J=two_J)
    L.pseudostates()
    L.build_perm("fp64")
    Es = np.linspace(3.0, 40.0, n_E)
    ref = L.solve(Es, "fp64", tol=1e-9, accept=1e-6, max_iter=400)
    for m in cycles:
        sol = L.solve(Es, "mixed_split", tol=1e-9, accept=1e-6, max_iter=400, refine_every=m)
        for k in range(n_E):
            assert np.max(np.abs(sol.amplitude(k)["A"] - ref.amplitude(k)["A"])) <= 1e-6, (m, k)
