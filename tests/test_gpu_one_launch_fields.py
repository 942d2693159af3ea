"""Leptons and photons of a step in one launch against a launch each (which a caller gets who times
the two kernels apart), over the field modes, several uneven instances (one empty, one frozen) and
workgroups of 64 and 256 threads: the same particles to the last bit.  Photon counts sit around
the batches of 64 and the chunks of 64 and 128 that a wavefront takes two at a time."""
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
from paper_1412_6426_amd.autotune import HipTimer  # noqa: E402
from paper_1412_6426_amd.engine import Engine  # noqa: E402

COLUMNS = ("x", "y", "z", "px", "py", "pz", "w", "id", "parent", "birth")
SIZES = [(700, 5_599), (0, 0), (1, 64 * 3 + 1), (40, 127), (3_000, 129), (5, 100_001), (0, 1),
         (64, 65)]
FROZEN = 3


def columns(rng, n, lo, hi, first_id):
    d = rng.normal(size=(n, 3))
    d *= (10.0 ** rng.uniform(lo, hi, n) / np.linalg.norm(d, axis=1))[:, None]
    x = rng.uniform(0.0, 7.0, (n, 3))
    return W._seed_columns(*(np.ascontiguousarray(v) for v in (*x.T, *d.T)), first_id=first_id)


def one_run(field, precision, block, tile, grid, split):
    rng = np.random.default_rng(7)
    caps = [(2 * l + p // 4 + 64, l + p // 4 + 64, 2 * p + 9 * l + 64) for l, p in SIZES]
    e = Engine(caps, [20 + i for i in range(len(SIZES))])
    e.build_tables()
    for i, (l, p) in enumerate(SIZES):
        e.load(i, 0, columns(rng, l - l // 2, 2.0, 3.0, 1))
        e.load(i, 1, columns(rng, l // 2, 2.0, 3.0, 1 << 30))
        e.load(i, 2, columns(rng, p, 1.0, 4.0, 1 << 40))
    e.set_frozen(FROZEN)
    if field == "yee":
        w = W.standing_wave_grid(n=1, a0=1700.0, cells=20)
        y = R.YeeGrid(w)
        y.fill(0.3, e.stream)
        f = R.field_of(w, y.g)
    elif field == "cp":
        f = Engine.make_field(Q.QED_FIELD_CP_STANDING, amp=1500.0)
    else:
        f = Engine.make_field(Q.QED_FIELD_UNIFORM, e0=(300.0, 0.0, 100.0), b0=(0.0, 1200.0, 0.0))
    p = Engine.make_params(dt=2 * np.pi / 200, eps_r=W.eps_r_for_wavelength(0.8e-6),
                           precision=precision, block=block, tile=tile, grid_blocks=grid)
    timer = HipTimer() if split else None
    if split:
        p.events[0] = timer.a
        p.events[3] = timer.b
    stats = R.run(e, f, p, 3)
    torch.cuda.synchronize()
    out = []
    for i in range(len(SIZES)):
        for s in range(3):
            g = e.read(i, s)
            # removed photons share an id, and the order of children follows the work split
            order = np.argsort(g["id"], kind="stable")
            order = order[g["id"][order] != Q.QED_NO_PARENT]
            out.append({c: np.asarray(g[c])[order] for c in COLUMNS})
    return stats, out


@pytest.mark.parametrize("block,tile,grid", [(0, 0, 0), (64, 0, 0), (128, 64, 3), (256, 200, 0)])
@pytest.mark.parametrize("precision", [Q.QED_FP64, Q.QED_MIXED])
@pytest.mark.parametrize("field", ["uniform", "cp", "yee"])
def test_one_launch_and_a_launch_each_agree(field, precision, block, tile, grid):
    print(f"one launch: {field} precision {precision} block {block} tile {tile}", flush=True)
    s1, a = one_run(field, precision, block, tile, grid, False)
    s2, b = one_run(field, precision, block, tile, grid, True)
    assert sum(s["pairs"] for s in s1) > 0 and sum(s["emitted"] for s in s1) > 0
    for x, y in zip(s1, s2):
        for key in ("advanced", "emitted", "pairs", "substeps", "nsub_hist", "photon_hist"):
            assert x[key] == y[key], key
    for p, q in zip(a, b):
        for c in COLUMNS:
            assert np.array_equal(p[c], q[c]), c
