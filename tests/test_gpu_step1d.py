"""Whole 1D steps in one workgroup per instance (every instance of at most 1024 cells) against
the oracle, at the edges of its thread counts (128, 256, 512, 1024) and of the rule, for every
law, boundary and troubled-cell mode; and its instances inside a batch against a batch that an
instance of 1025 cells sends through the tile kernels.  Tolerances: the repository's bounds
after time stepping; between the two GPU forms, whose arithmetic per cell is the same, the
bound of one operator evaluation per field."""
import numpy as np
import pytest

import hweno_inputs as hi
from oracle.physics import Equation
from oracle.scheme1d import Scheme1D
from parity import TOL, check_run, p1_field_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hw():
    import paper_2002_08816_amd as pkg
    return pkg


def scalar_state(n, seed):
    x = (np.arange(n) + 0.5) / n
    U = np.zeros((2, 1, n))
    U[0, 0] = 1.0 + 0.5 * np.sin(2 * np.pi * x) + 0.3 * (x > 0.37) - 0.2 * (x > 0.71)
    U[1, 0] = 0.002 * np.random.default_rng(seed).normal(size=n)
    return U


@pytest.mark.parametrize("n", [7, 64, 128, 129, 256, 257, 512, 513, 1024, 1025])
@pytest.mark.parametrize("eq,bc,tc", [("euler", "transmissive", "kxrcf"), ("euler", "reflective", "kxrcf"),
                                      ("euler", "periodic", "all"), ("burgers", "periodic", "kxrcf"),
                                      ("burgers", "transmissive", "all"), ("advection", "periodic", "none")])
def test_steps_against_the_oracle(hw, n, eq, bc, tc):
    U = hi.euler_riemann_1d(4, n)[0] if eq == "euler" else scalar_state(n, 5)
    if eq == "euler" and n < 64:   # too few cells for the generator's jumps: a smooth state
        U = hi.example_3_2(n, x1=2.0)
    s = hw.Solver(1, n, eq=eq, adv=(0.8,), bc=bc, tc_mode=tc)
    s.set_state(U)
    s.flag_export(True)
    s.steps(3)
    got, t = s.get_state()
    o = Scheme1D(Equation(eq, 1, adv=(0.8,)), n, 0.0, 1.0, bc=bc, tc_mode=tc)
    Uo, to, k, _ = o.run(U, nsteps=3, cfl=0.6)
    assert k == 3 and abs(t - to) <= 1e-13 * to
    check_run(got, Uo, f"{eq} {bc} {tc} n={n}")
    alpha = s.stats()[0][0]
    assert abs(alpha - o.alpha(got)) <= 1e-12 * alpha
    # flags of the last step's first stage: those of the state after two steps
    s2 = hw.Solver(1, n, eq=eq, adv=(0.8,), bc=bc, tc_mode=tc)
    s2.set_state(U)
    s2.steps(2)
    s2.flag_export(True)
    s2.apply_operator(s2.get_state()[0])
    for a, b in zip(s.flags(0), s2.flags(0)):
        assert np.array_equal(a, b)
    s.close()
    s2.close()


def test_a_run_stops_at_its_final_time_and_on_a_bad_state(hw):
    n = 300
    U = hi.euler_riemann_1d(2, n)[0]
    s = hw.Solver(1, n, eq="euler", bc="transmissive", tc_mode="kxrcf")
    s.set_state(U)
    steps, t = s.run(0.03)
    one = s.get_state()[0]
    assert t == 0.03 and s.time() == (0.03, steps) and steps > 16
    s.set_state(U)
    k, t2 = s.run(0.03, max_steps=21)
    assert k == 21 and 0.0 < t2 < 0.03
    k2, t3 = s.run(0.03)
    assert k + k2 == steps and t3 == 0.03 and np.array_equal(s.get_state()[0], one)
    bad = U.copy()
    bad[0, 2, 150] = -1.0   # negative pressure
    s.set_state(bad)
    with pytest.raises(Exception) as e:
        s.run(0.03)
    assert "non-" in str(e.value)
    s.close()


def test_batch_of_short_instances_equals_the_tile_kernels(hw):
    sizes = [100, 1000, 37, 512, 700]
    Us = [hi.euler_riemann_1d(b + 3, n)[0] for b, n in enumerate(sizes)]
    out = []
    for extra in ([], [1025]):
        bs = hw.BatchSolver(sizes + extra, eq="euler", bc="transmissive", tc_mode="kxrcf")
        bs.set_states(Us + [hi.euler_riemann_1d(40, n)[0] for n in extra])
        bs.steps(6, persistent=False)
        out.append((bs.get_states(), bs.times()[0]))
        bs.close()
    for b in range(len(sizes)):
        assert p1_field_err(out[0][0][b], out[1][0][b]) < TOL
        assert abs(out[0][1][b] - out[1][1][b]) <= 1e-14


@pytest.mark.parametrize("eq,bc,tc", [("euler", "transmissive", "kxrcf"), ("euler", "reflective", "kxrcf"),
                                      ("euler", "periodic", "all"), ("euler", "periodic", "none"),
                                      ("burgers", "transmissive", "kxrcf"), ("advection", "periodic", "all")])
def test_whole_steps_equal_the_stage_launches_to_the_bit(hw, eq, bc, tc):
    """An instance's values do not depend on the launch form, nor, with it, on the other instances
    of its batch: with an instance of 1025 cells beside them the same instances run through the
    tile kernels."""
    sizes = [100, 1000, 64, 512, 700, 300, 1024, 257, 7]
    if eq != "euler":
        Us = [scalar_state(n, n) for n in sizes + [1025]]
    elif bc == "transmissive":
        Us = [hi.euler_riemann_1d(b + 3, n)[0] if n >= 64 else hi.example_3_2(n, x1=2.0) for b, n in enumerate(sizes + [1025])]
    elif bc == "reflective":
        Us = []
        for n in sizes + [1025]:   # (a slow density wave with a jump of the pressure)
            U = hi.example_3_2(n, x1=2.0)
            U[:, 1] *= 0.1
            U[0, 2] += 1.0 * (np.arange(n) > 0.4 * n)
            Us.append(U)
    else:
        Us = [hi.example_3_2(n, x1=2.0) for n in sizes + [1025]]
    out = []
    for m in (len(sizes), len(sizes) + 1):
        bs = hw.BatchSolver((sizes + [1025])[:m], eq=eq, bc=bc, tc_mode=tc, adv=(0.8,))
        bs.set_states(Us[:m])
        bs.flag_export(True)
        bs.steps(9)
        out.append((bs.get_states(), bs.times()[0], [bs.flags(st) for st in range(3)]))
        bs.close()
    for b, n in enumerate(sizes):
        assert np.all(np.isfinite(out[0][0][b]))
        assert np.array_equal(out[0][0][b], out[1][0][b]) and out[0][1][b] == out[1][1][b], n
        for st in range(3):
            assert np.array_equal(out[0][2][st][0][b], out[1][2][st][0][b])
            assert np.array_equal(out[0][2][st][1][b], out[1][2][st][1][b])


@pytest.mark.parametrize("n", [300, 512, 1000, 1024, 1100])
def test_a_state_of_nan_stands_still(hw, n):
    """Cells whose speeds are no numbers make the Lax-Friedrichs speed infinite and the CFL step
    zero, in the whole-step form (up to 1024 cells) as in the tile kernels: the time of a run that
    has gone bad stays finite."""
    s = hw.Solver(1, n, eq="euler", bc="transmissive", tc_mode="kxrcf")
    s.set_state(np.full((2, 3, n), np.nan))
    s.steps(1, dt=1e-3)
    assert s.stats()[0][0] == np.inf
    s.steps(3)
    assert s.time() == (1e-3, 1)
    s.close()


def test_launch_forms_are_obeyed(hw):
    """A call that names a launch form gets it, on batches of short instances too; the tuner
    times whole steps beside the tile forms, and its choice can be set again.  All forms give the
    same values."""
    from paper_2002_08816_amd import capi
    form = lambda bs, asked=-1: capi._lib.hw_step_form(bs.h, asked)
    stages, persistent, whole = 0, 1, 2
    short, skewed = [300, 700, 64], [64] * 1000 + [1000]
    out = []
    for k, (sizes, own) in enumerate(((short, whole), (skewed, stages), (short + [1100], stages))):
        bs = hw.BatchSolver(sizes, eq="euler", bc="transmissive", tc_mode="kxrcf")
        Us = [hi.euler_riemann_1d(b % 7 + 3, n)[0] for b, n in enumerate(sizes)]
        assert form(bs) == own and form(bs, 0) == stages and form(bs, 1) == persistent
        states = []
        for asked in (None, False, True):
            bs.set_states(Us)
            bs.steps(9, persistent=asked)
            states.append(np.concatenate(bs.get_states(), axis=-1))
        bs.set_form(128, 0)
        assert form(bs) == own
        bs.set_form(128, 0, 1)
        assert form(bs) == stages
        bs.set_form(128, 1, 4)
        assert form(bs) == stages
        bs.set_states(Us)
        bs.steps(9)
        states.append(np.concatenate(bs.get_states(), axis=-1))
        tile, pers, grid = bs.tune()
        tuned = form(bs)
        bs.set_states(Us)
        bs.steps(9)
        states.append(np.concatenate(bs.get_states(), axis=-1))
        if pers or grid > 0:
            bs.set_form(tile, pers, grid)
            assert form(bs) == tuned == stages
        assert pers == 0 or grid > 1
        for s in states[1:]:
            assert np.array_equal(s, states[0], equal_nan=True)
        bs.set_meshes([np.linspace(0.0, 1.0, n + 1) for n in sizes])
        assert form(bs) == stages
        bs.set_meshes(None)
        assert form(bs) == own
        bs.close()


def test_blast_batch_in_every_form_with_a_longer_instance(hw):
    """Reflective walls in the tile kernels, one workgroup per tile and persistent, against the
    oracle: an instance of 1100 cells keeps the batch from whole steps."""
    from paper_2002_08816_amd import capi
    sizes = [1100, 400]
    Us = [hi.example_3_8(n) for n in sizes]
    os_ = [Scheme1D("euler", n, 0.0, 1.0, bc="reflective", tc_mode="kxrcf") for n in sizes]
    for k in range(51):
        if k == 50:
            refs = [o.rk3_step(U, o.cfl_dt(U, 0.6))[0] for o, U in zip(os_, Us)]
            for asked in (False, True):
                bs = hw.BatchSolver(sizes, eq="euler", bc="reflective", tc_mode="kxrcf")
                assert capi._lib.hw_step_form(bs.h, -1) == 0
                bs.set_states(Us)
                bs.steps(1, persistent=asked)
                for got, ref in zip(bs.get_states(), refs):
                    assert p1_field_err(got, ref) < TOL
                bs.close()
        Us = [o.rk3_step(U, o.cfl_dt(U, 0.6))[0] for o, U in zip(os_, Us)]


def test_eight_step_graph_of_stage_launches(hw):
    """Eleven steps of the stage launches (a replay of the eight-step graph and three of one step)
    and eleven single replays, one workgroup per tile and persistent."""
    from paper_2002_08816_amd import capi
    sizes = [64, 300, 1100, 2000]
    Us = [hi.euler_riemann_1d(b + 3, n)[0] for b, n in enumerate(sizes)]
    res = []
    for asked in (False, True):
        for parts in ([11], [1] * 11):
            bs = hw.BatchSolver(sizes, eq="euler", bc="transmissive", tc_mode="kxrcf")
            assert capi._lib.hw_step_form(bs.h, -1) == 0
            bs.set_states(Us)
            for n in parts:
                bs.steps(n, persistent=asked)
            res.append(np.concatenate(bs.get_states(), axis=-1))
            bs.close()
    assert np.all(np.isfinite(res[0]))
    for r in res[1:]:
        assert np.array_equal(r, res[0])
