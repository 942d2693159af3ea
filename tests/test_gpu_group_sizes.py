"""qed_thin_cells at the group sizes where its kernels change (one thread to 24 particles, one
wavefront to 1024, one workgroup beyond) and at the ends of a wavefront's rows of 64, against the
oracle: the same survivors in the same order, weights bit-identical to 1024 particles (summed in
store order on both sides) and within 1e-12 beyond (at most 2^-53 sqrt(n) n of a sum of n <= 2100
terms from 0.5 to 2); and the step's prefix sums over instance counts at the edges of prep's
wavefronts and rounds."""
import numpy as np
import pytest

from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

from paper_1412_6426_amd import qed as Q  # noqa: E402
from paper_1412_6426_amd import runner as R  # noqa: E402
from paper_1412_6426_amd import workloads as W  # noqa: E402
from paper_1412_6426_amd.engine import Engine  # noqa: E402

COLS = ("x", "y", "z", "px", "py", "pz", "id", "parent", "birth")
SIZES = (1, 2, 23, 24, 25, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025, 2100)


@pytest.mark.parametrize("cap", [1, 20, 24, 64, 1000, 1024])
@pytest.mark.parametrize("species", [0, 2])
def test_groups_at_the_kernel_edges(orc, species, cap):
    n, dx, origin = (len(SIZES), 2, 2), (1.0, 1.0, 1.0), (0.0, 0.0, 0.0)
    rng = np.random.default_rng(cap)
    cell = np.repeat(np.arange(len(SIZES)), SIZES)
    rng.shuffle(cell)
    m = len(cell)
    cols = W._seed_columns(cell + rng.uniform(0.01, 0.99, m), rng.uniform(0.01, 0.99, m),
                           rng.uniform(0.01, 0.99, m), rng.normal(size=m), rng.normal(size=m),
                           rng.normal(size=m), first_id=1)
    cols["w"] = rng.uniform(0.5, 2.0, m)
    caps = (m + 3,) * 3
    e = Engine([caps], [5])
    for s in range(3):
        e.load(0, s, cols if s == species else W.empty_columns())
    e.set_step(9)
    f = Engine.make_field(Q.QED_FIELD_YEE, grid=[torch.zeros(1, device="cuda")] * 6, n=n, dx=dx,
                          origin=origin)
    e.thin_cells(species, f, cap)
    torch.cuda.synchronize()
    rec = e.thin_cells_records()[0]
    st = orc.Store(m + 3, with_events=species != 2)
    st.load({k: v for k, v in cols.items() if species != 2 or k != "n_events"})
    orec = orc.thin_cells(st, species == 2, n, dx, origin, cap, 5, 9)
    want, got = st.view(), e.read(0, species)
    for c in COLS:
        assert np.array_equal(got[c], want[c]), c
    small = np.array([SIZES[int(x)] <= 1024 for x in want["x"]], bool)
    assert np.array_equal(got["w"][small], want["w"][small])
    np.testing.assert_allclose(got["w"], want["w"], rtol=1e-12, atol=0)
    for k in ("live_before", "kept", "groups", "groups_thinned"):
        assert rec[k] == orec[k], k


@pytest.mark.parametrize("instances", [1, 2, 63, 64, 65, 128, 255, 256, 257, 513])
def test_prefix_sums_over_instances(instances):
    """Uneven instances together give each instance what it gives alone."""
    w = W.rotating_e(n=1, a0=1700.0, capacity=200, lepton_capacity=40)
    sizes = [1 + (7 * i) % 5 for i in range(instances)]
    seeds = [100 + i for i in range(instances)]

    def run(which):
        e = Engine([(40, 40, 200)] * len(which), [seeds[i] for i in which])
        e.build_tables()
        for j, i in enumerate(which):
            for s, c in enumerate(W.rotating_e_initial(sizes[i], seed=i)):
                e.load(j, s, c)
        R.run(e, R.field_of(w), R.params_of(w), 3)
        return e

    e = run(range(instances))
    for i in sorted({0, instances // 2, instances - 2, instances - 1} - {-1}):
        one = run([i])
        for s in range(3):
            a, b = e.read(i, s), one.read(0, s)
            oa, ob = np.argsort(a["id"]), np.argsort(b["id"])
            for c in COLS:
                assert np.array_equal(a[c][oa], b[c][ob]), (i, s, c)
