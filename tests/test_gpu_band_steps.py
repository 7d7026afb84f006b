"""Steps, boundary value solves and stages that take the banded LU.  Without a
non-constant coefficient these reduce to tridiagonal systems; a one-term
Gamma(z) w keeps the band as narrow (kl, ku unchanged) and takes the banded
forms, so that each of them is reached from a step here:

* sparse factor records (factor_layout "auto") against the whole band
  ("band") over three steps (the SBDF1 and SBDF2 factor slots), a boundary
  value solve (a third operator) and a Runge-Kutta step: the same bits, since
  a missing entry is a zero of the band.  Without Gamma the same for the
  component solve of three operators through the two slots.
* every banded solve form (records, streamed whole band, two-block, pair, small
  staged) in the check build: three steps and a boundary value solve, every
  index check holds, the values are the default library's (1e-13 relative:
  the two builds are compiled separately).
* the mixed step's refined solve differs from the banded FP64 sweeps in the
  last bits (equal bits would be those sweeps, taken silently) and agrees with
  them to the refinement's accuracy, 1e-9.
* steps and boundary value solves through the banded slots leave each other's
  results alone."""
import os

import numpy as np
import pytest

import seeded_inputs as si
from oracle import RBOracle, RBParams

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("no GPU", allow_module_level=True)

from paper_1905_10388_amd import RBSolver, _lib  # noqa: E402

GAMMA = (0.3,)
DT = 5e-5


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _field(shape, seed, scale):
    X = scale * si.complex_noise(shape, seed) * np.exp(-np.arange(shape[-1]) / 4.0)
    X[..., shape[-3] - 1, :, :] = 0
    if len(shape) == 4:
        X[shape[0] // 2] = 0
    mean = X[0] if len(shape) == 3 else X[0, 0]
    mean[:] = mean.real
    return torch.from_numpy(X).cuda()


def _solver3(Nx, Ny, Nz, layout, gamma):
    return RBSolver(Nx, Nz, 4.0, 1e7, 1.0, dim=3, Ny=Ny, Ly=4.0, factor_layout=layout, gamma=gamma)


@pytest.mark.parametrize("shape", [(128, 128, 8), (64, 256, 32), (256, 256, 16), (256, 256, 128)],
                         ids=lambda s: "x".join(map(str, s)))
def test_steps_on_records_give_the_band_values(shape):
    Nx, Ny, Nz = shape
    out, ws = {}, {}
    for layout in ("band", "auto"):
        g = _solver3(Nx, Ny, Nz, layout, GAMMA)
        g.set_state(_field(g.state_shape, 150, 1.0))
        r = []
        for _ in range(3):
            g.step(DT)
            r.append(_np(g.X))
        r.append(_np(g.lbvp(_field(g.ev_shape, 151, 1.0))))
        g.step_rk(DT, "RK222")
        r.append(_np(g.X))
        out[layout], ws[layout] = r, g.query()["workspace_bytes"]
        g.close()
        del g
        torch.cuda.empty_cache()
    # two slots' records were built: nine units of eight columns per eight modes
    assert ws["auto"] - ws["band"] >= 2 * (Nx // 2 + 1) * Ny * (9 * Nz // 8) * (32 + 64)
    for n, (a, b) in enumerate(zip(out["auto"], out["band"])):
        assert np.isfinite(a).all() and np.array_equal(a, b), (shape, n)


@pytest.mark.parametrize("shape", [(128, 128, 8), (64, 256, 32)], ids=lambda s: "x".join(map(str, s)))
def test_component_solves_of_three_operators_on_records(shape):
    out = []
    for layout in ("band", "auto"):
        g = _solver3(*shape, layout, ())
        B = _field(g.ev_shape, 152, 1.0)
        r = []
        for a0 in (1.0 / DT, 1.5 / DT, 1.0 / DT, 2.0 / DT, 1.5 / DT):
            g.factor(a0)
            r.append(_np(g.solve(B)))
        out.append(r)
        g.close()
    for n, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b), n
    assert np.array_equal(out[0][0], out[0][2]) and np.array_equal(out[0][1], out[0][4])


# (name, constructor arguments, dt) of the banded solve forms
FORMS = [
    ("3d-128x128x16-records", dict(Nx=128, Nz=16, Lx=4.0, Ra=1e7, Pr=1.0, dim=3, Ny=128, Ly=4.0), 5e-5),
    ("3d-128x128x16-band", dict(Nx=128, Nz=16, Lx=4.0, Ra=1e7, Pr=1.0, dim=3, Ny=128, Ly=4.0,
                                factor_layout="band"), 5e-5),
    ("2d-1024x256-two-block", dict(Nx=1024, Nz=256, Lx=4.0, Ra=1e8, Pr=1.0), 1e-5),
    ("2d-4096x64-pair", dict(Nx=4096, Nz=64, Lx=16.0, Ra=1e7, Pr=7.0), 2e-5),
    ("2d-64x32", dict(Nx=64, Nz=32, Lx=4.0, Ra=1e4, Pr=1.0), 1e-3),
]


@pytest.mark.parametrize("form", FORMS, ids=[f[0] for f in FORMS])
def test_check_build_on_banded_steps(form):
    if not os.path.exists(_lib.LIB_CHECK_PATH):  # pragma: no cover
        pytest.skip("libstau_check.so not built (__graft_entry__.build() builds it)")
    name, kw, dt = form
    out = []
    for library in ("check", "default"):
        g = RBSolver(**kw, gamma=GAMMA, library=library)
        g.set_state(_field(g.state_shape, 153, 1e-2))
        for _ in range(3):
            g.step(dt)
        g.check()
        X = _np(g.X)
        Xb = g.lbvp(_field(g.ev_shape, 154, 1.0))
        g.check(Xb)
        out.append((X, _np(Xb)))
        g.close()
    for a, b in zip(*out):
        assert np.linalg.norm(a - b) <= 1e-13 * np.linalg.norm(b), name


@pytest.mark.parametrize("shape", [(16, 8, 16), (2048, 1, 16), (64, 1, 32)],
                         ids=["3d-16x8x16", "2d-2048x16", "2d-64x32-two-block"])
def test_refined_solve_is_taken_beside_the_banded_fp64_sweeps(shape):
    Nx, Ny, Nz = shape
    kw = dict(dim=3, Ny=Ny, Ly=4.0) if Ny > 1 else {}
    o = RBOracle(Nx, Nz, 4.0, RBParams(1e5, 1.0, gamma=GAMMA), **kw)
    X0 = torch.from_numpy(o.initial_state(si.workload_noise((Nx, Ny, Nz) if kw else (Nx, Nz), 0), amp=1e-2)).cuda()
    out = []
    for solve in ("fp64", "refined"):
        g = RBSolver(Nx, Nz, 4.0, 1e5, 1.0, precision="mixed", mixed_solve=solve, gamma=GAMMA, **kw)
        g.set_state(X0)
        g.step(1e-4)
        out.append(_np(g.X))
    a, r = out
    d = np.abs(a - r).max() / np.abs(a).max()
    assert 0.0 < d < 1e-9, d


def test_boundary_value_solves_and_steps_through_the_banded_slots():
    g, alone = (RBSolver(64, 32, 4.0, 1e4, 1.0, gamma=GAMMA) for _ in range(2))
    F = _field(g.ev_shape, 155, 1.0)
    X0 = _field(g.state_shape, 156, 0.1)
    first = _np(g.lbvp(F))
    for s in (g, alone):
        s.set_state(X0)
    for _ in range(4):  # three operators through two slots
        for s in (g, alone):
            s.step(1e-3)
        assert np.array_equal(_np(g.lbvp(F)), first)
    assert np.array_equal(_np(g.X), _np(alone.X))
