"""The lattice step on grids whose rows do not fill whole waves: a wave
serves 64 (split layout: 32) consecutive cells, so it crosses row and slab
ends wherever nx is not a multiple of that, and the last wave repeats the last
cell.  Against the oracle, with the bars of the other parity tests."""
import pytest

from paper_1608_06345_amd import lbm
from paper_1608_06345_amd.inputs import shear_wave_fields
from parity_util import TOL_FP32, TOL_FP64, assert_close, gpu_run, open_of, oracle_run

pytestmark = pytest.mark.gpu

OPEN, PER = lbm.LBM_BC_ZERO_GRADIENT, lbm.LBM_BC_PERIODIC
TOL_FP16_SHORT = 1e-3  # runs of tens of steps (as in the half-storage tests)


@pytest.mark.parametrize("dim,shape,bc", [
    (2, (63, 9, 1), 0),                              # just under a wave
    (2, (65, 9, 1), 0),                              # just over one
    (2, (3, 87, 1), lbm.LBM_BC(PER, OPEN)),          # 21 rows in a wave
    (2, (257, 66, 1), lbm.LBM_BC(OPEN, PER)),        # runs of two tiles per XCD, ragged
    (3, (31, 5, 7), 0),
    (3, (33, 5, 7), lbm.LBM_BC(OPEN, PER, PER)),
    (3, (5, 3, 4), lbm.LBM_BC(PER, PER, OPEN)),      # whole slabs inside a wave
    (3, (129, 17, 9), lbm.LBM_BC(PER, OPEN, PER)),
])
@pytest.mark.parametrize("precision,tol", [(lbm.LBM_FP64, TOL_FP64), (lbm.LBM_FP32_DEV, TOL_FP32),
                                           (lbm.LBM_FP16_SCALED, TOL_FP16_SHORT)])
def test_rows_across_waves(dim, shape, bc, precision, tol):
    f = shear_wave_fields(dim, *shape, seed=11)
    o = oracle_run(dim, 1.4, 0.7, 0.8, shape, f, 12, open_end=open_of(bc))
    for variant in (lbm.LBM_VARIANT_LANE, lbm.LBM_VARIANT_SPLIT):
        g = gpu_run(dim, 1.4, 0.7, 0.8, shape, f, 12, bc=bc, precision=precision,
                    variant=variant)
        assert_close(g, o, tol, f"{shape} precision {precision} variant {variant}")
