"""FP64 finite-difference steps in the kernels that the grid chooses (tests/
test_fd_route_host.py has the rule): the tiles in each of their instantiations
(64 x 4 x 4, 64 x 8 x 4 and 64 x 16 cells, streamed stores where nx is a
multiple of 16), with grids thinner than a tile's column or row and rows of 1 to
3 cells, and the staged chunks of grids with one plane.  Against the oracle, with
the bar of the other parity tests."""
import pytest

from paper_1608_06345_amd import lbm
from paper_1608_06345_amd.inputs import shear_wave_fields
from parity_util import TOL_FP64, assert_close, gpu_run, open_of, oracle_run

pytestmark = pytest.mark.gpu

OPEN, PER = lbm.LBM_BC_ZERO_GRADIENT, lbm.LBM_BC_PERIODIC
R = 1.196979770393074359


def _dt(dim):
    return (0.25 if dim == 2 else 0.3) / (3 * R)


def _compare(dim, shape, bc, steps, energy=False):
    from oracle.model import OracleLBM
    tg = 0.13 if energy else 0.12
    f = shear_wave_fields(dim, *shape, seed=11)
    o = OracleLBM(dim, 1.4, 0.1, tg, *shape, open_end=open_of(bc), dt=_dt(dim),
                  energy_fix=energy)
    o.init_fields(*f)
    o.step(steps)
    rho, u, E = o.moments()
    with lbm.Solver(dim, 1.4, 0.1, tg, *shape, bc=bc, dt=_dt(dim),
                    collision=lbm.LBM_COLLISION_ENERGY_CONSERVING if energy
                    else lbm.LBM_COLLISION_PAPER) as s:
        s.set_variant(lbm.LBM_VARIANT_TWO_PASS)
        s.init_fields(*f)
        s.step(steps)
        g = s.moments()
        T = s.temperature()
    assert_close((g[0], g[1], T), (rho, u, o.temperature(u, E)), TOL_FP64,
                 f"FD FP64 {shape} bc={bc} {steps} steps")


@pytest.mark.parametrize("shape,bc", [
    # one plane (78000 cells and more), and just short of the tiles
    ((256, 330, 1), lbm.LBM_BC(PER, OPEN, PER)),
    ((512, 161, 1), lbm.LBM_BC(OPEN, PER, OPEN)),
    ((512, 33, 4), lbm.LBM_BC(PER, PER, OPEN)),
])
@pytest.mark.parametrize("energy", [False, True])
def test_staged_chunks(shape, bc, energy):
    _compare(3, shape, bc, 5, energy)
