"""qed_thin_cells' weight_after of a single group, whichever kernel decides it (one thread to 24
particles, one wavefront to 1024): the sum, in store order, of weight times factor with one
rounding each, which exact rationals give to the last bit."""
from fractions import Fraction

import numpy as np
import pytest

from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

from paper_1412_6426_amd import qed as Q  # noqa: E402
from paper_1412_6426_amd import workloads as W  # noqa: E402
from paper_1412_6426_amd.engine import Engine  # noqa: E402


@pytest.mark.parametrize("m", [2, 23, 24, 25, 63, 64, 65, 130, 700, 1024])
def test_weight_after_is_the_sum_in_store_order(m):
    for seed in range(4):
        rng = np.random.default_rng(100 * m + seed)
        half = np.full(m, 0.5)
        cols = W._seed_columns(half, half, half, half, half, half, first_id=1 + 5000 * seed)
        cols["w"] = rng.uniform(0.5, 2.0, m)
        e = Engine([(1, 1, m)], [seed])
        e.load(0, 2, cols)
        e.set_step(3)
        f = Engine.make_field(Q.QED_FIELD_YEE, grid=[torch.zeros(1, device="cuda")] * 6,
                              n=(2, 2, 2), dx=(1.0, 1.0, 1.0))
        e.thin_cells(2, f, m // 2)
        torch.cuda.synchronize()
        rec = e.thin_cells_records()[0]
        kept = np.isin(cols["id"], e.read(0, 2)["id"])
        total = some = 0.0
        for w, k in zip(cols["w"], kept):
            total += w
            some += w if k else 0.0
        factor, after = total / some, 0.0
        for w in cols["w"][kept]:
            after = float(Fraction(float(w)) * Fraction(factor) + Fraction(after))
        assert rec["groups_thinned"] == 1 and rec["kept"] == int(kept.sum())
        assert rec["weight_before"] == total
        assert rec["weight_after"] == after
