"""Setting the fields: S_0 and its collision come from one kernel (a wave
serves 64 cells, 32 in the split layout, and the last one repeats the last
cell).  S_0 is read at step 0, the collided populations at step 1, against the
oracle with the bars of the other parity tests."""
import pytest

from paper_1608_06345_amd import lbm
from paper_1608_06345_amd.inputs import shear_wave_fields
from parity_util import TOL_FP32, TOL_FP64, assert_close, gpu_run, oracle_run

pytestmark = pytest.mark.gpu

TOL_FP16_SHORT = 1e-3  # runs of tens of steps (as in the half-storage tests)


@pytest.mark.parametrize("dim,shape", [
    (2, (1, 1, 1)),      # one cell
    (2, (21, 3, 1)),     # 63 cells
    (2, (13, 5, 1)),     # 65
    (2, (257, 5, 1)),    # five 256-cell groups and a rest
    (3, (31, 1, 1)),
    (3, (11, 3, 1)),     # 33 cells
    (3, (13, 5, 7)),
    (3, (41, 37, 45)),   # past the one-wave workgroups
])
@pytest.mark.parametrize("precision,tol", [(lbm.LBM_FP64, TOL_FP64), (lbm.LBM_FP32_DEV, TOL_FP32),
                                           (lbm.LBM_FP16_SCALED, TOL_FP16_SHORT)])
def test_initial_state_and_first_step(dim, shape, precision, tol):
    f = shear_wave_fields(dim, *shape, seed=5)
    for steps in (0, 1):
        o = oracle_run(dim, 1.4, 0.7, 0.8, shape, f, steps)
        for variant in (lbm.LBM_VARIANT_LANE, lbm.LBM_VARIANT_SPLIT):
            g = gpu_run(dim, 1.4, 0.7, 0.8, shape, f, steps, precision=precision,
                        variant=variant)
            assert_close(g, o, tol, f"{shape} steps {steps} precision {precision} {variant}")
