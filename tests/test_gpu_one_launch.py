"""Leptons and photons of a step in one launch against a launch each (a caller that times the two
kernels apart gets those): the same particles to the last bit in both orders of the workgroups
(photons under and over eight times the leptons), with workgroups of either kind under, at and
over one per compute unit, and in both precisions."""

import numpy as np
import pytest

from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

from paper_1412_6426_amd import runner as R  # noqa: E402
from paper_1412_6426_amd import workloads as W  # noqa: E402
from paper_1412_6426_amd.autotune import HipTimer  # noqa: E402

COLUMNS = ("x", "y", "z", "px", "py", "pz", "w", "id", "parent", "birth")


def photons(n):
    """n photons from far under to over the pair threshold of the field."""
    rng = np.random.default_rng(n)
    k = 10.0 ** rng.uniform(1.0, 4.0, n)[:, None] * np.eye(3)[rng.integers(0, 3, n)]
    one = np.ones(n)
    return dict(x=one * 0.1, y=one * 0.2, z=one * 0.3, px=k[:, 0].copy(), py=k[:, 1].copy(),
                pz=k[:, 2].copy(), w=one, id=(1 << 40) + np.arange(n, dtype=np.uint64),
                parent=np.full(n, 0xFFFFFFFFFFFFFFFF, dtype=np.uint64),
                birth=np.zeros(n, dtype=np.uint64))


def one_run(n_lep, n_pho, grid, precision, timer):
    w = W.rotating_e(n=n_lep, a0=1700.0, capacity=2 * n_pho + 8 * n_lep + 64,
                     lepton_capacity=2 * n_lep + n_pho + 64)
    init = list(W.rotating_e_initial(n_lep, seed=3))
    init[2] = photons(n_pho)
    e = R.engine_single(w, init)
    params = R.params_of(w, precision=precision, grid_blocks=grid)
    if timer is not None:
        params.events[0] = timer.a
        params.events[3] = timer.b
    stats = R.run(e, R.field_of(w), params, 3)
    out = []
    for s in range(3):
        g = e.read(0, s)
        order = np.argsort(g["id"], kind="stable")
        out.append({c: np.asarray(g[c])[order] for c in COLUMNS})
    return stats, out


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_lep,n_pho,grid", [
    (1, 1, 0), (700, 5_599, 0), (700, 5_600, 0), (300, 70_000, 0), (60_000, 100_000, 0),
    (2_000, 300_000, 1), (2_000, 300_000, 255), (2_000, 300_000, 256), (2_000, 300_000, 700)])
def test_one_launch_and_a_launch_each_agree(n_lep, n_pho, grid, precision):
    s1, a = one_run(n_lep, n_pho, grid, precision, None)
    s2, b = one_run(n_lep, n_pho, grid, precision, HipTimer())
    for x, y in zip(s1, s2):
        for key in ("advanced", "emitted", "pairs", "substeps", "nsub_hist", "photon_hist"):
            assert x[key] == y[key], key
    for p, q in zip(a, b):
        for c in COLUMNS:
            assert np.array_equal(p[c], q[c]), c
