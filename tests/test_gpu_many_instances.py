"""qed_thin_cells with more instances than a grid's y and z extents hold: every instance's count
and record, and the compacted columns.  One block per instance holds its particles, so the record
follows from the counts alone; weights are 1, and a thinned group keeps its total weight to
rounding (sums of at most 3 terms)."""
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


@pytest.mark.parametrize("instances", [65535, 65536, 70001])
def test_thin_cells_of_many_instances(orc, instances):
    sizes = np.arange(instances) % 4
    print(f"thin cells: {instances} instances", flush=True)
    e = Engine([(1, 1, 3)] * instances, (np.arange(instances) + 5).tolist())
    slots = 3 * instances
    d = e.cols[2]
    d["x"].fill_(0.5), d["y"].fill_(0.5), d["z"].fill_(0.5), d["w"].fill_(1.0)
    d["id"].copy_(torch.arange(1, slots + 1))
    raw = (Q.qed_instance * instances).from_buffer_copy(e.inst.cpu().numpy().tobytes())
    for i in range(instances):
        raw[i].count[2] = int(sizes[i])
    e.inst.copy_(torch.from_numpy(np.frombuffer(bytes(raw), np.uint8).copy()))
    e.set_step(7)
    f = Engine.make_field(Q.QED_FIELD_YEE, grid=[torch.zeros(1, device="cuda")] * 6, n=(2, 2, 2),
                          dx=(1.0, 1.0, 1.0))
    e.thin_cells(2, f, 2)
    torch.cuda.synchronize()
    recs = np.frombuffer(e._tc_rec.cpu().numpy().tobytes(), dtype=[
        ("live_before", "i8"), ("kept", "i8"), ("groups", "i8"), ("groups_thinned", "i8"),
        ("weight_before", "f8"), ("weight_after", "f8")])
    kept = e.counts()[:, 2]
    assert np.array_equal(recs["live_before"], sizes)
    assert np.array_equal(recs["groups"], (sizes > 0).astype(int))
    assert np.array_equal(recs["groups_thinned"], (sizes > 2).astype(int))
    assert np.array_equal(recs["weight_before"], sizes.astype(float))
    assert np.array_equal(recs["kept"], kept)
    np.testing.assert_allclose(recs["weight_after"], sizes, rtol=1e-15, atol=0)
    assert np.array_equal(kept[sizes < 3], sizes[sizes < 3])
    for i in (0, 3, 7, instances // 2, 65534, instances - 2, instances - 1):
        st = orc.Store(3, with_events=False)
        m = int(sizes[i])
        one, x = np.ones(m), np.full(m, 0.5)
        cols = W._seed_columns(x, x, x, 0 * one, 0 * one, 0 * one, first_id=3 * i + 1)
        cols["w"] = one
        st.load({k: v for k, v in cols.items() if k != "n_events"})
        orc.thin_cells(st, True, (2, 2, 2), (1.0, 1.0, 1.0), (0.0, 0.0, 0.0), 2, i + 5, 7)
        want, got = st.view(), e.read(i, 2)
        assert np.array_equal(got["id"], want["id"]) and np.array_equal(got["w"], want["w"])
