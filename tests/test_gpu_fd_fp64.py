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
    e = assert_close((g[0], g[1], T), (rho, u, o.temperature(u, E)), TOL_FP64,
                     f"FD FP64 {shape} bc={bc} {steps} steps")
    print(f"\nPARITY FD FP64 {shape} bc={bc} {steps} steps energy={energy} rho/u/T={e}")


@pytest.mark.parametrize("shape,bc", [
    # one plane (78000 cells and more), and just short of the tiles
    ((256, 330, 1), lbm.LBM_BC(PER, OPEN, PER)),
    ((512, 161, 1), lbm.LBM_BC(OPEN, PER, OPEN)),
    ((512, 33, 4), lbm.LBM_BC(PER, PER, OPEN)),
])
@pytest.mark.parametrize("energy", [False, True])
def test_staged_chunks(shape, bc, energy):
    _compare(3, shape, bc, 5, energy)


@pytest.mark.parametrize("shape,bc", [
    ((64, 35, 37), lbm.LBM_BC(PER, OPEN, PER)),    # 64 x 4 x 4, streamed
    ((64, 70, 58), lbm.LBM_BC(PER, PER, OPEN)),    # 64 x 8 x 4, streamed
    ((80, 66, 61), lbm.LBM_BC(OPEN, PER, PER)),    # the same, ragged along every axis
    ((176, 150, 3), lbm.LBM_BC(PER, PER, OPEN)),   # columns of three and two planes
    ((200, 200, 2), 0),
    ((400, 2, 100), lbm.LBM_BC(PER, OPEN, PER)),   # one to three rows
    ((333, 3, 80), 0),
    ((1000, 1, 79), 0),
    ((2, 300, 140), lbm.LBM_BC(PER, PER, OPEN)),   # two and three cells
    ((3, 300, 90), 0),
    ((43, 48, 39), 0),                             # odd rows, cells a multiple of 16
])
def test_tiles_3d(shape, bc):
    _compare(3, shape, bc, 5)


@pytest.mark.parametrize("shape,bc", [
    ((1008, 130, 1), 0),                           # streamed, ragged along y
    ((1024, 160, 1), lbm.LBM_BC(OPEN, OPEN)),      # streamed, whole tiles
    ((703, 275, 1), lbm.LBM_BC(PER, OPEN)),
    ((1999, 80, 1), lbm.LBM_BC(OPEN, PER)),
    ((703, 272, 1), 0),                            # odd rows, cells a multiple of 16
    ((64000, 3, 1), lbm.LBM_BC(OPEN, OPEN)),
    ((64000, 3, 1), 0),
    ((32768, 2, 1), lbm.LBM_BC(PER, OPEN)),
    ((90000, 1, 1), 0),
    ((2, 5000, 1), lbm.LBM_BC(PER, OPEN)),
    ((3, 64001, 1), 0),
])
def test_tiles_2d(shape, bc):
    _compare(2, shape, bc, 5)


@pytest.mark.parametrize("dim,shape", [(2, (703, 275, 1)), (2, (1008, 130, 1)), (3, (64, 70, 58))])
def test_tiles_energy_conserving(dim, shape):
    _compare(dim, shape, 0, 5, energy=True)


@pytest.mark.parametrize("dim,shape,steps", [(2, (48, 2401, 1), 300), (3, (64, 33, 38), 100)])
def test_tiles_many_steps(dim, shape, steps):
    _compare(dim, shape, 0, steps)
