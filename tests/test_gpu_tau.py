"""The pencil solve by reduction to tridiagonal systems (every step, stage and
boundary value solve without a non-constant coefficient), at the sizes where
its chunks, tiles and tables have their edges: chains of two elements up to
256 (Nz = 4 to 512; chunks of 8), pencils per block from one to eight with a
partial last block, both dimensions, unequal wavenumber spacings (tables
shared by few pencils), the mean pencil, k / 2 above and below the highest
degree (both forms of the pressure), and a0 = 0.

* Two SBDF steps (both operators) from a rough state and a boundary value
  solve against the oracle per field, 1e-10 relative: the FP64 bar of every
  trajectory test.
* The boundary value solve against the banded LU of the same operator (the
  component calls stau_factor / stau_solve), 1e-10 relative over the state.
* An operator that the reduction does not take (a non-constant coefficient)
  and one that it does, alternated on one pencils object with the component
  solve: none disturbs the others' factors.
"""
import numpy as np
import pytest

import seeded_inputs as si
from gpu_helpers import field_errors, rel_err
from oracle import RBOracle, RBParams

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("no GPU", allow_module_level=True)

from paper_1905_10388_amd import RBSolver  # noqa: E402

BAR = 1e-10

# dim, Nx, Ny, Nz, Lx, Ly, dt
SHAPES = [(2, 8, 1, 4, 4.0, 1.0, 1e-3), (2, 16, 1, 8, 1.0, 1.0, 1e-3), (2, 64, 1, 16, 16.0, 1.0, 1e-3),
          (2, 64, 1, 32, 0.25, 1.0, 1e-4), (2, 8, 1, 512, 4.0, 1.0, 1e-3),
          (3, 4, 8, 4, 4.0, 2.0, 1e-3), (3, 8, 8, 16, 4.0, 4.0, 1e-3), (3, 32, 4, 8, 8.0, 0.5, 1e-3),
          (3, 4, 4, 128, 4.0, 3.0, 1e-3)]


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _state(o, seed):
    dec = np.exp(-np.arange(o.Nz) / max(2.0, o.Nz / 8.0))
    X = si.complex_noise(o.state_shape, seed) * dec * 0.1
    X[..., o.Px - 1, :, :] = 0
    if o.dim == 3:
        X[o.Ny // 2] = 0
        X[:, 0] = 0          # (the kx = 0 plane stands for a real field only with ky symmetry)
    mean = X[0] if o.dim == 2 else X[0, 0]
    mean[:] = mean.real
    return X


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(str(v) for v in s[:4]))
def test_steps_and_bvp_against_oracle_and_banded_lu(shape):
    dim, Nx, Ny, Nz, Lx, Ly, dt = shape
    o = RBOracle(Nx, Nz, Lx, RBParams(1e5, 0.7), dim=dim, Ny=Ny, Ly=Ly)
    g = RBSolver(Nx, Nz, Lx, 1e5, 0.7, dim=dim, Ny=Ny, Ly=Ly)
    X = _state(o, 11)
    g.set_state(torch.from_numpy(X).cuda())
    for _ in range(2):
        X = o.step(X, dt)
        g.step(dt)
    errs = field_errors(o, _np(g.X), X)
    assert max(errs.values()) < BAR, errs

    F = _state(o, 12)[..., :o.ne, :].copy()
    Xb = _np(g.lbvp(torch.from_numpy(F).cuda()))
    errs = field_errors(o, Xb, o.lbvp(F))
    assert max(errs.values()) < BAR, errs
    g.factor(0.0, 1.0)
    PF = np.zeros_like(F)
    PF[...] = F @ o.C.toarray().T
    PF[..., Nz - 1] = 0
    assert rel_err(Xb, _np(g.solve(torch.from_numpy(PF).cuda()))) < BAR


def test_band_and_tridiagonal_factors_side_by_side():
    dt = 1e-3
    plain = RBSolver(32, 16, 4.0, 1e5, 1.0)
    ncc = RBSolver(32, 16, 4.0, 1e5, 1.0, gamma=(0.3, 0.1))
    X = torch.from_numpy(_state(RBOracle(32, 16, 4.0, RBParams(1e5, 1.0)), 13)).cuda()
    B = torch.from_numpy(si.complex_noise(plain.ev_shape, 14)).cuda()

    def run(g, mixed_in):
        g.set_state(X)
        out = []
        if mixed_in:
            g.factor(2.0 / dt)
        for i in range(4):
            if mixed_in:
                out.append(_np(g.solve(B)))
                g.lbvp(B)
            g.step(dt * (1.0 + 0.1 * (i % 3)))  # three operators through two slots
        return _np(g.X), out

    for g in (plain, ncc):
        alone, _ = run(g, False)
        with_calls, solves = run(g, True)
        assert np.array_equal(alone, with_calls)
        assert all(np.array_equal(s, solves[0]) for s in solves)
