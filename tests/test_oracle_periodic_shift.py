"""The oracle's operator on a mesh that is periodic in one direction and has walls in the other
commutes with a shift along the periodic direction: the wrapped rows beyond the mesh are mesh rows in
every respect, ghosts beside the walls included.  Tolerance: round-off of one operator evaluation."""
import numpy as np
import pytest

import hweno_inputs as hi
from oracle.physics import Equation
from oracle.scheme2d import Scheme2D


@pytest.mark.parametrize("nx,ny", [(9, 40), (17, 40), (40, 9)])
@pytest.mark.parametrize("eq,bc", [("euler", ("transmissive", "periodic")), ("euler", ("reflective", "periodic")),
                                   ("euler", ("periodic", "transmissive")), ("euler", ("periodic", "reflective")),
                                   ("burgers", ("transmissive", "periodic")), ("burgers", ("periodic", "transmissive"))])
def test_operator_commutes_with_a_periodic_shift(eq, bc, nx, ny):
    U = hi.euler_wall_state(nx, ny, 4)
    U[1:] *= 0.02
    if eq != "euler":
        U = np.ascontiguousarray(U[:, :1])
    h = 1.0 / ny
    o = Scheme2D(Equation(eq, 2), nx, ny, 0.0, nx * h, 0.0, 1.0, bc=bc, ng_edge=3, tc_mode="kxrcf")
    axis = -2 if bc[1] == "periodic" else -1
    L, info = o.operator(U)
    assert info["T"].any()
    for k in (1, 5):
        Lk, infok = o.operator(np.roll(U, k, axis=axis))
        assert np.array_equal(np.roll(infok["T"], -k, axis=axis), info["T"])
        assert np.abs(np.roll(Lk, -k, axis=axis) - L).max() < 1e-14 * np.abs(L).max()
