"""The order in which the many-channel FP64 products add a row's blocks (launch_spmv_gen, pk_slots).

Whether a divergent series is accepted depends on the last bits of its terms, so the kernels that may run on a
call's column count add in one order, and the results are compared bit for bit: below 16 columns, and with
more than 24 channels at any count, the matrix-core kernels against the passes of 4 columns
(spmm_cols above the column count); from 16 columns on, one wavefront of 16 against windows of 32 columns, and
the requests of a fixed stream whose acceptance the order decides."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import paper_1404_5253_amd as wp
    from paper_1404_5253_amd.serve import BatchBackend, slot_bytes

import workloads

# name: M, N, two_J, j_max; 2 open channels (two_J = 1) or 3
LATTICES = {"pw10": (23, 19, 1, 1), "pw14": (15, 18, 3, 1), "pw18": (17, 14, 1, 2), "pw26": (9, 10, 1, 3),
            "pw30": (8, 9, 3, 2)}


def lattice(M, N, two_J, j_max, **kw):
    L = wp.Lattice(M, N, two_J=two_J, j_max=j_max, swave_only=False)
    L.pseudostates(**kw)
    L.build_perm("fp64")
    return L


@pytest.fixture(scope="module")
def lattices():
    return {name: lattice(*spec) for name, spec in LATTICES.items()}


def results(L, Es, mode, **kw):
    sol = L.solve(Es, mode, tol=1e-9, accept=1e-6, max_iter=60, allow_noconv=True, **kw)
    out = [sol.amplitude(k)["A"] for k in range(len(Es))]
    if mode == "fp64":
        out += [sol.series(k, b) for k in range(len(Es)) for b in range(out[0].shape[0])]
    return out


def assert_same(a, b, what):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert np.array_equal(x, y), what


@pytest.mark.parametrize("mode", ["fp64", "mixed_split"])   # FP64 and FP32 blocks, FP64 vectors
@pytest.mark.parametrize("name,n_E", [("pw10", 1), ("pw10", 3), ("pw14", 1), ("pw14", 2), ("pw14", 5), ("pw18", 1),
                                      ("pw18", 2), ("pw18", 7), ("pw26", 1), ("pw26", 9), ("pw30", 1), ("pw30", 6)])
def test_by_slots_as_the_passes(lattices, name, n_E, mode):
    Es = np.linspace(2.0, 40.0, n_E)
    assert_same(results(lattices[name], Es, mode), results(lattices[name], Es, mode, spmm_cols=1 << 20), (name, n_E, mode))


@pytest.mark.parametrize("name", ["pw10", "pw14", "pw18"])
def test_block_after_block_at_any_width(lattices, name):
    L, Es = lattices[name], np.linspace(2.0, 40.0, 20)
    wide = results(L, Es, "fp64", step_tile="mfma8")   # one step kernel for both
    n = wide[0].shape[0]
    for k in (0, 7, 19):
        alone = results(L, Es[k:k + 1], "fp64", spmm_cols=1, step_tile="mfma8")
        assert_same([wide[k]] + wide[20 + n * k:20 + n * (k + 1)], alone, (name, k))


def test_stream_requests_stay_accepted():
    """Four of the 1735 requests that the stream of workloads.serving_requests holds for this lattice: their
    estimates end a little below the stop tolerance, and other last bits of the products end them above it."""
    L = lattice(150, 150, 1, 2, kind="mt", V_R=workloads.mt_repulsion(0))
    Es = [E for _, l, E in workloads.serving_requests(4, rate=200.0, duration=35.0) if l == 2]
    Es = [E for E in Es if any(abs(E - e) < 1e-6 for e in (1.112349956, 1.106156712, 1.090936145, 1.285894865))]
    assert len(Es) == 4
    b = BatchBackend(L, slots=32, hbm_budget=32 * slot_bytes(L, "fp64"), terms=8, tol=3e-7, accept=1e-7, max_iter=400,
                     stream=wp.current_stream(), mode="fp64")
    place = dict(zip(b.admit_many(Es), Es))
    while place:
        for slot, r in b.step():
            assert r["accepted"], place[slot]
            del place[slot]
    b.close()
