"""Finite differences: the initial state comes with the record that the next
step works from, unless the fused kernel is chosen.  Steps in every order of
the two forms, and a second initial state in the same solve, against the
oracle, with the bars of the other parity tests."""
import pytest

from paper_1608_06345_amd import lbm
from paper_1608_06345_amd.inputs import shear_wave_fields
from parity_util import TOL_FP32, TOL_FP64, assert_close, oracle_run

pytestmark = pytest.mark.gpu

REC, FUSED = lbm.LBM_VARIANT_TWO_PASS, lbm.LBM_VARIANT_LANE


@pytest.mark.parametrize("dim,shape,dt", [
    (2, (1, 1, 1), 0.0696), (2, (51, 5, 1), 0.0696), (2, (257, 3, 1), 0.0696),
    (3, (31, 3, 5), 0.0835), (3, (48, 43, 41), 0.0835),
])
@pytest.mark.parametrize("precision,tol", [(lbm.LBM_FP64, TOL_FP64), (lbm.LBM_FP32_DEV, TOL_FP32)])
@pytest.mark.parametrize("order", [(REC, REC), (REC, FUSED), (FUSED, REC)])
def test_record_of_initial_state(dim, shape, dt, precision, tol, order):
    with lbm.Solver(dim, 1.4, 0.12, 0.13, *shape, precision=precision, dt=dt) as s:
        for seed in (3, 4):
            f = shear_wave_fields(dim, *shape, seed=seed)
            o = oracle_run(dim, 1.4, 0.12, 0.13, shape, f, 3, dt=dt)
            s.set_variant(order[0])
            s.init_fields(*f)
            s.step(1)
            s.set_variant(order[1])
            s.step(1)
            s.set_variant(order[0])
            s.step(1)
            rho, u, _ = s.moments()
            assert_close((rho, u, s.temperature()), o, tol, f"{shape} {precision} {order} {seed}")
