"""The forward step's corner cell takes the values and the flag of the fluid cell across the
corner.  Where the corner lies beside a tile's edge that cell is two layers outside the tile:
flags, hybrid masks and the operator against the oracle there (a corner in column 15 or row 17,
and away from the edges).  Tolerance: the repository's bound of one operator evaluation."""
import numpy as np
import pytest

import hweno_inputs as hi
from oracle.scheme2d import Scheme2D
from parity import TOL, array_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ng", [2, 3])
@pytest.mark.parametrize("nx,ny,corner", [(35, 33, (15, 15)), (35, 33, (15, 14)), (40, 36, (17, 17)), (50, 38, (31, 17)), (40, 36, (20, 15))])
def test_operator_around_the_corner(nx, ny, corner, ng):
    import paper_2002_08816_amd as hw
    h = 0.1
    dom = (0.0, nx * h, 0.0, ny * h)
    at = (corner[0] * h, corner[1] * h)
    s = hw.Solver(2, nx, ny, domain=dom, eq="euler", ng_edge=ng, tc_mode="kxrcf", bc="step", step=at)
    o = Scheme2D("euler", nx, ny, *dom, bc="step", ng_edge=ng, tc_mode="kxrcf", step_corner=at)
    s.flag_export(True)
    for seed in (5, 6, 7):
        U = hi.euler_wall_state(nx, ny, seed)
        U[1:] *= 0.2
        L, W = s.apply_operator(U)
        T, H = s.flags(0)
        Lo, info = o.operator(U)
        fluid = np.ones((ny, nx), dtype=bool)
        fluid[:corner[1], corner[0]:] = False
        assert np.array_equal(T[fluid], info["T"][fluid]) and np.array_equal(H[fluid], info["H"][fluid])
        assert array_err(L, Lo) < TOL
    s.close()
