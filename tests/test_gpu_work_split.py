"""How few particles are spread over the wavefronts: seed counts at the edges of the chunk rule
(one lepton a wavefront, one more than the spread, one batch of 64 lanes for each, one more)
against the oracle, and a same-step shower whose children outnumber the generation kernel's
wavefronts in some generations and not in others."""
import pytest

from tests.conftest import gpu_available
from tests.parity_util import compare_all, oracle_field, oracle_params, oracle_stores

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

from oracle import oracle as orc  # noqa: E402
from paper_1412_6426_amd import runner as R  # noqa: E402
from paper_1412_6426_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 65535, 65536, 65537])
def test_seed_counts_at_the_chunk_edges(n):
    w = W.rotating_e(n=n, a0=1700.0, capacity=4 * n + 64, lepton_capacity=2 * n + 16)
    init = W.rotating_e_initial(n, seed=n)
    e = R.engine_single(w, init)
    stats = R.run(e, R.field_of(w), R.params_of(w), 4)
    os_ = oracle_stores(orc, init, w.capacity)
    ostats = orc.run(os_, oracle_field(orc, w), oracle_params(orc, w), 4)
    compare_all(e, os_, label=f"{n} seeds")
    for s, o in zip(stats, ostats):
        for key in ("advanced", "emitted", "pairs", "substeps", "nsub_hist", "photon_hist"):
            assert s[key] == o[key], key


@pytest.mark.parametrize("n,generations", [(1, 3), (9, 24)])
def test_children_dealt_over_all_wavefronts(n, generations):
    w = W.shower(n=n, dt=12_000.0, steps=2, capacity=(400 * n + 200, 400 * n + 200,
                                                      9000 * n + 4000))
    init = W.shower_initial(w)
    e = R.engine_single(w, init, same_step=True)
    stats = R.run(e, R.field_of(w), R.params_of(w, same_step_generations=generations), w.n_steps)
    os_ = oracle_stores(orc, init, w.capacity)
    ostats = orc.run(os_, oracle_field(orc, w),
                     oracle_params(orc, w, same_step_generations=generations), w.n_steps)
    for s, o in zip(stats, ostats):
        for key in ("emitted", "pairs", "children_advanced", "deferred", "substeps"):
            assert s[key] == o[key], key
    for s in range(3):
        g, o = e.read(0, s), os_[s].view()
        assert sorted(g["id"].tolist()) == sorted(o["id"].tolist())
