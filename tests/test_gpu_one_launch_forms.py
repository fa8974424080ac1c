"""The one-launch stage with two threads per cell (up to 256 tiles) and with one (more tiles):
the same data on a mesh of the first kind and repeated on one of the second, and both against
the oracle at the edge between them, with walls and ragged tiles.  Tolerance: the repository's
bound of one operator evaluation."""
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


def state(eq, nx, ny):
    U = hi.euler_wall_state(nx, ny, 4)
    U[1:] *= 0.02
    return U if eq == "euler" else np.ascontiguousarray(U[:, :1])


@pytest.mark.parametrize("tc", ["kxrcf", "all"])
@pytest.mark.parametrize("ng", [2, 3])
@pytest.mark.parametrize("eq", ["euler", "burgers", "advection"])
def test_two_threads_per_cell_equal_one(hw, eq, ng, tc):
    n, k = 100, 3
    U = state(eq, n, n)
    out = []
    for m in (1, k):
        s = hw.Solver(2, m * n, m * n, domain=(0.0, float(m), 0.0, float(m)), eq=eq, adv=(0.7, -0.45),
                      bc="periodic", ng_edge=ng, tc_mode=tc)
        s.flag_export(True)
        V = np.ascontiguousarray(np.tile(U, (1, 1, m, m)))
        L, W = s.apply_operator(V)
        F = s.flags(0)
        s.set_state(V)
        s.steps(2, dt=2e-4)
        out.append((L, W, F, s.get_state()[0], s.stats()))
        s.close()
    (L, W, F, S, st), (Lk, Wk, Fk, Sk, stk) = out
    for j, i in ((0, 0), (k - 1, 1)):
        sl = np.s_[..., j * n:(j + 1) * n, i * n:(i + 1) * n]
        assert np.array_equal(F[0], Fk[0][sl]) and np.array_equal(F[1], Fk[1][sl])
        assert array_err(Lk[sl], L) < TOL and array_err(Wk[sl], W) < TOL and array_err(Sk[sl], S) < TOL
    assert [m * k * k for m in st[1] + st[2]] == list(stk[1] + stk[2])
    assert np.allclose(st[0], stk[0], rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("nx,ny", [(250, 241), (255, 258), (9, 40)])
@pytest.mark.parametrize("eq,bc,ng", [("euler", ("reflective", "transmissive"), 2), ("euler", ("periodic", "transmissive"), 3),
                                      ("burgers", ("periodic", "transmissive"), 3)])
def test_both_forms_against_the_oracle(hw, eq, bc, ng, nx, ny):
    h = 1.0 / ny
    U = state(eq, nx, ny)
    kw = dict(bc=bc, ng_edge=ng, tc_mode="kxrcf")
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


@pytest.mark.parametrize("eq,n", [("euler", 40), ("burgers", 300)])
def test_one_launch_steps_by_every_call(hw, eq, n):
    """The stages set the time step, the time, the step count, the speeds and the list lengths by
    themselves: one state advanced by steps(), step(), profile() and run() is the same, bit for
    bit, and the oracle's."""
    U = state(eq, n, n)
    kw = dict(bc="periodic", ng_edge=2, tc_mode="kxrcf")
    s = hw.Solver(2, n, n, eq=eq, **kw)
    s.set_state(U)
    s.steps(11)
    ref, t = s.get_state()
    stats = s.stats()
    assert s.time() == (t, 11)
    s.set_state(U)
    s.steps(3)
    s.step()
    s.profile(2)
    s.apply_operator(U)          # leaves the state and its speeds alone
    s.steps(4)
    s.step()
    got, t2 = s.get_state()
    assert np.array_equal(got, ref) and t2 == t and s.time() == (t, 11)
    for a, b in zip(s.stats(), stats):
        assert np.array_equal(np.asarray(a), np.asarray(b))
    s.set_state(U)
    steps, T = s.run(t)
    assert T == t and abs(steps - 11) <= 1 and np.abs(s.get_state()[0] - ref).max() < 1e-12 * np.abs(ref).max()
    s.steps(2)                   # past the final time of the run before
    assert s.time()[1] == steps + 2 and s.time()[0] > t
    s.set_state(U)
    s.steps(2, dt=1e-4)
    o = Scheme2D(Equation(eq, 2), n, n, 0.0, 1.0, 0.0, 1.0, **kw)
    V = U
    for _ in range(2):
        V, _ = o.rk3_step(V, 1e-4)
    assert array_err(s.get_state()[0], V) < TOL and abs(s.time()[0] - 2e-4) < 1e-18
    s.close()


@pytest.mark.parametrize("nx,ny", [(9, 40), (12, 40), (16, 40), (17, 40), (40, 9), (321, 330)])
@pytest.mark.parametrize("eq,ng", [("euler", 2), ("euler", 3), ("burgers", 3)])
def test_walls_in_x_with_y_periodic(hw, eq, ng, nx, ny):
    """The cells where the periodic rows meet the transmissive columns (one-launch stage; list
    passes on the last mesh for Euler)."""
    h = 1.0 / ny
    U = state(eq, nx, ny)
    kw = dict(bc=("transmissive", "periodic"), ng_edge=ng, tc_mode="kxrcf")
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


@pytest.mark.parametrize("ng", [2, 3])
@pytest.mark.parametrize("n,copies", [(13, 8), (16, 7), (41, 3), (96, 2)])
def test_small_meshes_of_troubled_cells_equal_their_copies(hw, n, copies, ng):
    """Euler with every cell troubled: meshes that take four launches, and their data repeated on
    one that takes one launch."""
    U = state("euler", n, n)
    out = []
    for m in (1, copies):
        s = hw.Solver(2, m * n, m * n, domain=(0.0, float(m), 0.0, float(m)), eq="euler", bc="periodic", ng_edge=ng,
                      tc_mode="all")
        s.flag_export(True)
        V = np.ascontiguousarray(np.tile(U, (1, 1, m, m)))
        L, W = s.apply_operator(V)
        F = s.flags(0)
        s.set_state(V)
        s.steps(2, dt=2e-4)
        out.append((L, W, F, s.get_state()[0], s.stats()))
        s.close()
    (L, W, F, S, st), (Lk, Wk, Fk, Sk, stk) = out
    sl = np.s_[..., (copies - 1) * n:, n:2 * n]
    assert np.array_equal(F[0], Fk[0][sl]) and np.array_equal(F[1], Fk[1][sl])
    assert array_err(Lk[sl], L) < TOL and array_err(Wk[sl], W) < TOL and array_err(Sk[sl], S) < TOL
    assert [m * copies * copies for m in st[1] + st[2]] == list(stk[1] + stk[2])
    assert np.allclose(st[0], stk[0], rtol=1e-12, atol=0.0)
