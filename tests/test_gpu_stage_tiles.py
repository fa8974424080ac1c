"""The 2D stage kernel's two staging paths against the oracle: a tile whose 20 x 20 staged
positions are all mesh cells is loaded without boundary mapping, every other tile with it.
The meshes are at the edges of that rule: 33 cells (no such tile), 34 (one, ending at the last
cell), 35 and 50 (the next tile column or row begins).  Tolerance: the repository's bound of one
operator evaluation."""
import numpy as np
import pytest

import hweno_inputs as hi
from oracle.physics import Equation
from oracle.scheme2d import Scheme2D
from parity import TOL, array_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hw():
    import paper_2002_08816_amd as pkg
    return pkg


@pytest.mark.parametrize("nx,ny", [(33, 34), (34, 34), (35, 50), (50, 35)])
@pytest.mark.parametrize("eq,bc", [("euler", ("transmissive", "reflective")), ("euler", ("periodic", "periodic")),
                                   ("burgers", ("periodic", "transmissive")), ("advection", ("periodic", "periodic"))])
@pytest.mark.parametrize("ng", [2, 3])
def test_operator_at_the_edges_of_the_unmapped_tiles(hw, nx, ny, eq, bc, ng):
    h = 1.0 / ny
    U = hi.euler_wall_state(nx, ny, 3)
    U[1:] *= 0.02   # linear cells between the jumps too
    if eq != "euler":
        U = np.ascontiguousarray(U[:, :1])
    kw = dict(bc=bc, ng_edge=ng, tc_mode="kxrcf")
    s = hw.Solver(2, nx, ny, domain=(0.0, nx * h, 0.0, 1.0), eq=eq, adv=(0.7, -0.45), **kw)
    s.flag_export(True)
    L, W = s.apply_operator(U)
    T, H = s.flags(0)
    o = Scheme2D(Equation(eq, 2, adv=(0.7, -0.45)), nx, ny, 0.0, nx * h, 0.0, 1.0, **kw)
    Lo, info = o.operator(U)
    assert info["T"].any() and not info["H"].all()
    assert np.array_equal(T, info["T"]) and np.array_equal(H, info["H"])
    assert array_err(L, Lo) < TOL
    assert array_err(W, info["limited"]) < TOL
    s.close()
