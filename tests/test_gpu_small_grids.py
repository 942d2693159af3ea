"""Few leptons on fewer wavefronts than the device has SIMDs (grid_blocks), at the edges of the
chunk rule for that many (one lepton a wavefront, one batch of 64 for each, one more) against the
oracle."""
import pytest

from tests.conftest import gpu_available
from tests.parity_util import compare_all, oracle_field, oracle_params, oracle_stores

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

from oracle import oracle as orc  # noqa: E402
from paper_1412_6426_amd import runner as R  # noqa: E402
from paper_1412_6426_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("grid,block", [(1, 64), (1, 256), (3, 128), (16, 256)])
@pytest.mark.parametrize("per_wave", [1, 63, 64, 65, 129])
def test_counts_at_the_chunk_edges_of_a_small_grid(grid, block, per_wave):
    n = grid * (block // 64) * per_wave + (1 if per_wave == 1 else 0)
    w = W.rotating_e(n=n, a0=1700.0, capacity=6 * n + 64, lepton_capacity=2 * n + 16)
    init = W.rotating_e_initial(n, seed=n)
    e = R.engine_single(w, init)
    stats = R.run(e, R.field_of(w), R.params_of(w, grid_blocks=grid, block=block), 4)
    os_ = oracle_stores(orc, init, w.capacity)
    ostats = orc.run(os_, oracle_field(orc, w), oracle_params(orc, w), 4)
    compare_all(e, os_, label=f"{n} leptons, {grid} workgroups of {block}")
    for s, o in zip(stats, ostats):
        for key in ("advanced", "emitted", "pairs", "substeps", "nsub_hist", "photon_hist"):
            assert s[key] == o[key], key
