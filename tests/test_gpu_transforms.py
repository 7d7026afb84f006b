"""The transforms at compile-time padded lengths (24 to 768 points in y, 24 to
6144 in x, 24 to 768 in 3-D, 24 to 768 in z), at their tile edges: fewer columns than a tile,
exactly one tile, several; few rows and many with a partial last block; and
lengths next to them that the general kernels take (12 points; 1536 in 3-D).

* The explicit term (both y directions with the y derivatives formed on the
  way) and a padded grid transform there and back, FP64, against the oracle,
  1e-13 relative: the bar of the other transform tests.
* Two SBDF steps against the oracle per field, 1e-10 relative (the right-hand
  sides of the z forward transform).
* One mixed step whose explicit term outweighs the rest of the right-hand side
  (amplitude 1e3, dt = 1) against the oracle per field within the mixed step's
  stated bound, 1e-5.
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

# dim, Nx, Ny, Nz
Y_SHAPES = [(3, 8, 8, 4), (3, 4, 16, 8), (3, 32, 16, 4), (3, 64, 8, 4), (3, 64, 32, 4), (3, 8, 64, 8),
            (3, 4, 128, 4), (3, 32, 128, 4), (3, 4, 256, 4), (3, 16, 256, 4), (3, 4, 512, 4), (3, 16, 512, 4)]
X_SHAPES = [(2, Nx, 1, 8) for Nx in (8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096)] + [
    (3, 16, 4, 4), (3, 16, 64, 64), (3, 32, 4, 8), (3, 32, 64, 64), (3, 64, 8, 4), (3, 128, 4, 4), (3, 256, 4, 4),
    (3, 512, 4, 4), (3, 1024, 4, 4)]
# half and whole tiles of every z length (whole ones from 4096 pencils and fields)
Z_SHAPES = [(2, 8, 1, Nz) for Nz in (16, 32, 64, 128, 256, 512)] + [(3, 64, 32, 16), (3, 64, 32, 32)]
Z_LARGE = [(3, 64, 32, 64), (2, 4096, 1, 128), (2, 4096, 1, 256), (2, 2048, 1, 512)]


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _pair(shape, **kw):
    dim, Nx, Ny, Nz = shape
    o = RBOracle(Nx, Nz, 4.0, RBParams(1e4, 1.0), dim=dim, Ny=Ny, Ly=3.0)
    return o, RBSolver(Nx, Nz, 4.0, 1e4, 1.0, dim=dim, Ny=Ny, Ly=3.0, **kw)


def _state(o, seed):
    X = si.complex_noise(o.state_shape, seed) * np.exp(-np.arange(o.Nz) / (o.Nz / 6.0))
    X[..., o.Px - 1, :, :] = 0
    if o.dim == 3:
        X[o.Ny // 2] = 0
        X[:, 0] = 0          # (the kx = 0 plane stands for a real field only with ky symmetry)
    mean = X[0] if o.dim == 2 else X[0, 0]
    mean[:] = mean.real
    return X


@pytest.mark.parametrize("shape", Y_SHAPES + X_SHAPES + Z_SHAPES + Z_LARGE, ids=lambda s: "-".join(str(v) for v in s))
def test_explicit_term_and_grid_round_trip(shape):
    o, g = _pair(shape)
    X = _state(o, 41)
    assert rel_err(_np(g.nonlinear(torch.from_numpy(X).cuda())), o.nonlinear(X)) < 1e-13
    G = g.coeff_to_grid(("b",), 1.5, X=torch.from_numpy(X).cuda())
    ref = o.to_grid(X[..., o.vi["b"], :])
    assert rel_err(_np(G)[0], ref if o.dim == 2 else ref.transpose(1, 0, 2)) < 1e-13
    # (a grid aligned to its doubles only)
    G = torch.empty(G.numel() + 1, dtype=G.dtype, device=G.device)[1:].view(G.shape).copy_(G)
    Xg = g.grid_to_coeff(("w",), G, 1.5, X=torch.zeros_like(torch.from_numpy(X)).cuda())
    assert rel_err(_np(Xg)[..., o.vi["w"], :], o.from_grid(ref)) < 1e-13


@pytest.mark.parametrize("shape", Z_SHAPES, ids=lambda s: "-".join(str(v) for v in s))
def test_steps(shape):
    o, g = _pair(shape)
    X = 0.1 * _state(o, 43)
    g.set_state(torch.from_numpy(X).cuda())
    for _ in range(2):
        X = o.step(X, 1e-4)
        g.step(1e-4)
    errs = field_errors(o, _np(g.X), X)
    assert max(errs.values()) < 1e-10, errs


@pytest.mark.parametrize("shape", Y_SHAPES + X_SHAPES + Z_SHAPES, ids=lambda s: "-".join(str(v) for v in s))
def test_mixed_explicit_term(shape):
    o, g = _pair(shape, precision="mixed", dct="fft")
    X = 1e3 * _state(o, 42)
    g.set_state(torch.from_numpy(X).cuda())
    g.step(1.0)
    errs = field_errors(o, _np(g.X), o.step(X, 1.0))
    assert max(errs.values()) < 1e-5, errs
