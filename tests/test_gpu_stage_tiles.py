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
from parity import TOL, array_err, p1_field_err

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


@pytest.mark.parametrize("tc", ["kxrcf", "all"])
@pytest.mark.parametrize("ng", [2, 3])
@pytest.mark.parametrize("eq,n,copies", [("euler", 120, 3), ("burgers", 135, 5), ("advection", 140, 5)])
def test_one_launch_stage_equals_the_list_passes(hw, eq, n, copies, ng, tc):
    """A periodic mesh small enough for the one-launch stage, and its data repeated on a mesh
    that runs the flags, limiter, HWENO and stage launches: the same operator in every copy,
    with the same flags, after one operator and after two steps (rounding differs only where
    the compiler contracts differently: the operator's bound)."""
    U = hi.euler_wall_state(n, n, 4)
    U[1:] *= 0.02
    if eq != "euler":
        U = np.ascontiguousarray(U[:, :1])
    out = []
    for k in (1, copies):
        s = hw.Solver(2, k * n, k * n, domain=(0.0, float(k), 0.0, float(k)), eq=eq, adv=(0.7, -0.45),
                      bc="periodic", ng_edge=ng, tc_mode=tc)
        s.flag_export(True)
        V = np.ascontiguousarray(np.tile(U, (1, 1, k, k)))
        L, W = s.apply_operator(V)
        F = s.flags(0)
        st0 = s.stats()[1:]
        s.set_state(V)
        s.steps(2, dt=2e-4)
        out.append((L, W, F, s.get_state()[0], s.stats()[1:], st0))
        s.close()
    (L, W, F, S, c, c0), (Lk, Wk, Fk, Sk, ck, ck0) = out
    for j, i in ((0, 0), (copies - 1, copies // 2)):
        sl = np.s_[..., j * n:(j + 1) * n, i * n:(i + 1) * n]
        assert np.array_equal(F[0], Fk[0][sl]) and np.array_equal(F[1], Fk[1][sl])
        assert array_err(Lk[sl], L) < TOL and array_err(Wk[sl], W) < TOL
        assert array_err(Sk[sl], S) < TOL
    assert [m * copies ** 2 for m in c[0] + c[1]] == list(ck[0] + ck[1])
    assert c0[0][0] * copies ** 2 == ck0[0][0] > 0 and c0[1][0] * copies ** 2 == ck0[1][0]


@pytest.mark.parametrize("eq,bc,nx,ny", [("euler", ("reflective", "transmissive"), 329, 321),
                                         ("euler", ("transmissive", "periodic"), 321, 337),
                                         ("burgers", ("transmissive", "transmissive"), 650, 641)])
def test_list_passes_on_a_mesh_with_walls(hw, eq, bc, nx, ny):
    """The launches of the larger meshes with mirrored sides and ragged tiles, against the
    oracle."""
    h = 1.0 / ny
    U = hi.euler_wall_state(nx, ny, 6)
    U[1:] *= 0.02
    if eq != "euler":
        U = np.ascontiguousarray(U[:, :1])
    kw = dict(bc=bc, ng_edge=3, tc_mode="kxrcf")
    s = hw.Solver(2, nx, ny, domain=(0.0, nx * h, 0.0, 1.0), eq=eq, **kw)
    s.flag_export(True)
    L, W = s.apply_operator(U)
    T, H = s.flags(0)
    o = Scheme2D(Equation(eq, 2), nx, ny, 0.0, nx * h, 0.0, 1.0, **kw)
    Lo, info = o.operator(U)
    assert np.array_equal(T, info["T"]) and np.array_equal(H, info["H"])
    assert array_err(L, Lo) < TOL
    assert array_err(W, info["limited"]) < TOL
    s.close()


@pytest.mark.parametrize("eq,bc,ng,tc,nx,ny", [
    ("euler", ("periodic", "reflective"), 2, "kxrcf", 35, 2145), ("euler", ("reflective", "transmissive"), 2, "all", 17, 3217),
    ("euler", ("transmissive", "reflective"), 3, "all", 17, 3217), ("euler", ("reflective", "periodic"), 3, "kxrcf", 35, 2145),
    ("advection", ("transmissive", "periodic"), 2, "kxrcf", 17, 12817),
    ("burgers", ("periodic", "transmissive"), 2, "all", 17, 12817)])
def test_list_passes_with_walls_and_a_step(hw, eq, bc, ng, tc, nx, ny):
    """Strips of more tiles than the one-launch stage takes, so that the flags, limiter, HWENO and
    stage launches run: the operator, and one Runge-Kutta step (the limited values of u^n in its
    second and third stage), against the oracle."""
    h = 1.0 / 64
    U = hi.euler_wall_state(nx, ny, 5)
    U[1:] *= 0.02
    if eq != "euler":
        U = np.ascontiguousarray(U[:, :1])
    kw = dict(bc=bc, ng_edge=ng, tc_mode=tc)
    s = hw.Solver(2, nx, ny, domain=(0.0, nx * h, 0.0, ny * h), eq=eq, adv=(0.7, -0.45), **kw)
    s.flag_export(True)
    L, W = s.apply_operator(U)
    T, H = s.flags(0)
    o = Scheme2D(Equation(eq, 2, adv=(0.7, -0.45)), nx, ny, 0.0, nx * h, 0.0, ny * h, **kw)
    Lo, info = o.operator(U)
    assert np.array_equal(T, info["T"]) and np.array_equal(H, info["H"]) and T.any()
    assert array_err(L, Lo) < TOL
    assert array_err(W, info["limited"]) < TOL
    s.set_state(U)
    s.steps(1, dt=1e-3)
    V, infos = o.rk3_step(U, 1e-3)
    for st in range(3):
        assert np.array_equal(s.flags(st)[0], infos[st]["T"])
    assert p1_field_err(s.get_state()[0], V) < TOL
    s.close()
