"""Half storage: each initial value is rounded to half once, so that both
register layouts store the same bits.  The readout of step 0, sums of the stored
halves in one order, is then equal bit for bit."""
import numpy as np
import pytest

from paper_1608_06345_amd import lbm
from paper_1608_06345_amd.inputs import smooth_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,shape", [(2, (1, 1, 1)), (2, (257, 5, 1)), (3, (13, 5, 7)),
                                       (3, (41, 37, 45))])
def test_layouts_store_the_same_halves(dim, shape):
    f = smooth_fields(dim, *shape, seed=6, a_rho=0.05, a_u=0.05, a_T=0.05)
    got = []
    for variant in (lbm.LBM_VARIANT_LANE, lbm.LBM_VARIANT_SPLIT):
        with lbm.Solver(dim, 1.4, 0.7, 0.8, *shape, precision=lbm.LBM_FP16_SCALED) as s:
            s.set_variant(variant)
            s.init_fields(*f)
            got.append(s.moments())
    for a, b in zip(*got):
        assert np.array_equal(a, b)
