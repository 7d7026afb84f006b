"""Calls captured into HIP graphs after stau_factor: the operator's factors
exist then, whatever form the call's solve takes, so that stau_step,
stau_step_rk and stau_lbvp launch kernels only.  Each operator is factored
after two others have taken the cache's places; the graph is replayed several
times, with new inputs, the program's own eager work and synchronisations
between the replays, each replay against the eager calls of a second object,
bit for bit.  Tridiagonal solve (no non-constant coefficient) and banded LU
(a one-term one), 2-D and 3-D."""
import math

import numpy as np
import pytest

import seeded_inputs as si

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("no GPU", allow_module_level=True)

from paper_1905_10388_amd import RBSolver  # noqa: E402

DT = 1e-3


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _solver(dim, gamma):
    kw = dict(dim=3, Ny=8, Ly=3.0) if dim == 3 else {}
    return RBSolver(32, 16, 4.0, 1e5, 1.0, gamma=gamma, **kw)


def _field(shape, seed):
    X = 0.1 * si.complex_noise(shape, seed) * np.exp(-np.arange(shape[-1]) / 3.0)
    X[..., shape[-3] - 1, :, :] = 0
    if len(shape) == 4:
        X[shape[0] // 2] = 0
        X[:, 0] = 0
    mean = X[0] if len(shape) == 3 else X[0, 0]
    mean[:] = mean.real
    return torch.from_numpy(X).cuda()


def _capture(call):
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        call()
    return graph


@pytest.mark.parametrize("gamma", [(), (0.3,)], ids=["tridiagonal", "banded"])
@pytest.mark.parametrize("dim", [2, 3])
def test_boundary_value_solve(dim, gamma):
    g, e = _solver(dim, gamma), _solver(dim, gamma)
    F = _field(g.ev_shape, 110)
    out = g.lbvp(F).clone()
    for _ in range(2):  # two other operators
        g.step(DT)
    g.factor(0.0, 1.0)
    graph = _capture(lambda: g.lbvp(F, out=out))
    for n in range(4):
        F.copy_(_field(g.ev_shape, 111 + n))
        ref = _np(e.lbvp(F))
        graph.replay()
        assert np.array_equal(_np(out), ref), n


@pytest.mark.parametrize("gamma", [(), (0.3,)], ids=["tridiagonal", "banded"])
@pytest.mark.parametrize("dim", [2, 3])
def test_steps(dim, gamma):
    g, e = _solver(dim, gamma), _solver(dim, gamma)
    X0 = _field(g.state_shape, 120)
    for s in (g, e):
        s.set_state(X0)
        s.step(DT)  # SBDF1, then SBDF2
    g.lbvp(_field(g.ev_shape, 121))  # (a second operator)
    g.factor(3.0 / (2.0 * DT), 1.0)

    def two():  # (the history slots change places with each step)
        g.step(DT)
        g.step(DT)
    graph = _capture(two)
    for n in range(3):
        for _ in range(2):
            e.step(DT)
        ref = _np(e.X)
        graph.replay()
        assert np.array_equal(_np(g.X), ref), n


@pytest.mark.parametrize("gamma", [(), (0.3,)], ids=["tridiagonal", "banded"])
def test_runge_kutta_step(gamma):
    g, e = _solver(2, gamma), _solver(2, gamma)
    X0 = _field(g.state_shape, 130)
    for s in (g, e):
        s.set_state(X0)
        s.step_rk(0.5 * DT, "RK222")  # (allocates the stages' workspace)
    g.lbvp(_field(g.ev_shape, 131))
    g.factor(1.0 / (DT * (1.0 - 1.0 / math.sqrt(2.0))), 1.0)
    graph = _capture(lambda: g.step_rk(DT, "RK222"))
    for n in range(3):
        e.step_rk(DT, "RK222")
        ref = _np(e.X)
        graph.replay()
        assert np.array_equal(_np(g.X), ref), n
