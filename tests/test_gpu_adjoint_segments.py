"""The recorded run's last segment is kept by the forward run itself and the others are replayed
from their checkpoints with the same kernels, so the gradient is the same number for every
checkpoint interval (k = 1: all but the last step replayed; k >= nsteps: none), when asked for
again after other segments have taken the workspace, and after the weights are set
(which makes every segment a replayed one).  The recorded run leaves the handle as plain
steps of the same size do.  All comparisons are for equality."""
import numpy as np
import pytest

import hweno_inputs as hi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eq,tc,bc,nx,ny", [
    ("euler", "kxrcf", "periodic", 40, 32), ("euler", "kxrcf", "periodic", 420, 330), ("euler", "none", "periodic", 32, 24),
    ("euler", "kxrcf", "step", 60, 20), ("euler", "kxrcf", "dmr", 28, 10),
    ("burgers", "kxrcf", "periodic", 33, 20), ("advection", "all", "transmissive", 24, 31)])
def test_gradient_does_not_depend_on_the_segments(eq, tc, bc, nx, ny):
    import paper_2002_08816_amd as hw
    kw = dict(domain=(0.0, nx * 0.05, 0.0, ny * 0.05))
    if bc == "step":
        kw["step"] = (0.6, 0.2)
    rng = np.random.default_rng(3)
    nc = 4 if eq == "euler" else 1
    U = np.zeros((3, nc, ny, nx))
    shock = 1.0 + 0.6 * (np.arange(nx) > nx // 2)[None, :] + 0.1 * np.sin(np.arange(ny))[:, None]
    if eq == "euler":
        U[0, 0], U[0, 1], U[0, 2], U[0, 3] = shock, 0.3 * shock, -0.2 * shock, 2.5 * shock
    else:
        U[0, 0] = shock
    U[1:] = 0.01 * rng.normal(size=U[1:].shape)
    if bc == "dmr":
        kw["domain"] = (0.0, nx / (2 * ny), 0.0, 0.5)
        U = hi.euler_dmr_state(nx, ny, 0.5 / ny, 5)
    lam = rng.normal(size=U.shape)
    n, dt = 5, 2.885e-4 if bc == "dmr" else 0.004
    s = hw.Solver(2, nx, ny, eq=eq, ng_edge=3 if bc == "dmr" else 2, tc_mode=tc, bc=bc, **kw)
    s.set_state(U)
    s.steps(n, dt)
    ref, t = s.get_state()
    stats = s.stats()
    g = None
    for k in (7, 5, 3, 2, 1):
        s.set_state(U)
        s.forward_ckpt(n, dt, k)
        got, tk = s.get_state()
        assert np.array_equal(got, ref) and tk == t
        for a, b in zip(s.stats(), stats):
            assert np.array_equal(np.asarray(a), np.asarray(b)), k
        gk = s.adjoint(lam)
        assert np.all(np.isfinite(gk))
        if g is None:
            g = gk
        assert np.array_equal(gk, g), k
        assert np.array_equal(s.adjoint(lam), g), k
        if eq == "euler":   # the default weights again
            s.set_linear_weights([0.98, 0.01, 0.01])
            assert np.array_equal(s.adjoint(lam), g), k
    # and a run goes on from there as after plain steps
    s.steps(2, dt)
    a = s.get_state()[0]
    s.set_state(U)
    s.steps(n, dt)
    s.steps(2, dt)
    assert np.array_equal(a, s.get_state()[0])
    s.close()


@pytest.mark.parametrize("eq,nx,ny", [("burgers", 33, 20), ("burgers", 650, 641), ("advection", 33, 20),
                                      ("euler", 40, 32), ("euler", 330, 322)])
def test_a_gradient_leaves_the_list_lengths_alone(eq, nx, ny):
    """The list lengths are those of the last step before and after a gradient, whose replayed
    stages have lists of their own (one-launch stages and list passes)."""
    import paper_2002_08816_amd as hw
    nc = 4 if eq == "euler" else 1
    U = hi.euler_wall_state(nx, ny, 4)[:, :nc].copy()
    U[1:] *= 0.02
    s = hw.Solver(2, nx, ny, eq=eq, ng_edge=2, tc_mode="kxrcf", bc="periodic", domain=(0.0, nx / ny, 0.0, 1.0))
    s.set_state(U)
    s.forward_ckpt(5, 2e-4, 2)
    before = s.stats()
    assert sum(before[1]) > 0
    s.adjoint(np.ones_like(U))
    for a, b in zip(s.stats(), before):
        assert np.array_equal(np.asarray(a), np.asarray(b))
    s.close()
