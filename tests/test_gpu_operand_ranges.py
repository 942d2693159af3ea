"""Steps whose operands leave 2^-900..2^900, where the sub-step's roots and quotients take the
library's forms: finite momenta of 10^136 (p^2 beyond 2^900) in a weak field with a step so long
that leptons emit and photons convert, and a field of 10^-140 (its square below 2^-900), against
the oracle."""
import numpy as np
import pytest

from tests.conftest import gpu_available
from tests.parity_util import compare_all, compare_stats, oracle_field, oracle_params, oracle_stores

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

from oracle import oracle as orc  # noqa: E402
from paper_1412_6426_amd import runner as R  # noqa: E402
from paper_1412_6426_amd import workloads as W  # noqa: E402


def columns(rng, n, scale, first_id):
    d = rng.normal(size=(n, 3))
    d *= (scale * rng.uniform(1.0, 3.0, n) / np.linalg.norm(d, axis=1))[:, None]
    x = rng.uniform(0.0, 7.0, (n, 3))
    return W._seed_columns(*(np.ascontiguousarray(v) for v in (*x.T, *d.T)), first_id=first_id)


@pytest.mark.parametrize("field", ["rotating", "uniform"])
@pytest.mark.parametrize("p_scale,amp,dt,forced,busy", [
    (1e136, 1e-130, 1e134, 1, True),   # p^2 beyond 2^900, chi of order one
    (1e136, 1e-130, 1e134, 3, True),
    (1e140, 1e3, 1e-3, 1, False),      # chi^2 beyond 2^900 as well
    (1e2, 1e-140, 0.03, 0, False),     # chi^2 below 2^-900
    (1e-140, 1e-140, 0.03, 0, False),  # p^2 and k^2 as well
])
def test_operands_beyond_the_fast_range(field, p_scale, amp, dt, forced, busy):
    print(f"operands: {field} p {p_scale} amp {amp}", flush=True)
    eps_r = W.eps_r_for_wavelength(0.8e-6)
    f = (W.FieldSpec(kind=W.FIELD_ROTATING_E, amp=amp, omega=1e-3) if field == "rotating" else
         W.FieldSpec(kind=W.FIELD_UNIFORM, e0=(amp, 0.2 * amp, 0.0), b0=(0.0, 0.3 * amp, amp)))
    w = W.Workload(name="operands", eps_r=eps_r, dt=dt, n_steps=3, field=f,
                   capacity=(4_000, 4_000, 8_000), seed=3, n_seed=200)
    rng = np.random.default_rng(11)
    init = [columns(rng, 200, p_scale, 1), columns(rng, 100, p_scale, 1 << 30),
            columns(rng, 300, p_scale, 1 << 40)]
    e = R.engine_single(w, init)
    stats = R.run(e, R.field_of(w), R.params_of(w, forced_substeps=forced), w.n_steps)
    os_ = oracle_stores(orc, init, w.capacity)
    ostats = orc.run(os_, oracle_field(orc, w), oracle_params(orc, w, forced_substeps=forced),
                     w.n_steps)
    if busy:
        assert sum(s["emitted"] for s in stats) > 100 and sum(s["pairs"] for s in stats) > 10
    assert sum(s["nonfinite"] for s in stats) == 0
    compare_all(e, os_, label=f"{field} {p_scale}")
    compare_stats(stats, ostats, label=f"{field} {p_scale}")
