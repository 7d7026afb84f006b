"""The first factorisation of a pencils object on a stream of its own.  The
banded factors' storage is allocated and zeroed by the call that first needs
it; the factorisation follows at once on the caller's stream, which is not
ordered after the null stream that zeroes.  On a fresh object each call that
allocates (the component solve, the adjoint step, the eigenvalue solve) gives
the bits on a side stream that it gives on the default stream, in the
two-block (2-D) and the single-block (3-D) layout."""
import numpy as np
import pytest

import seeded_inputs as si

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("no GPU", allow_module_level=True)

from paper_1905_10388_amd import RBSolver, StauError  # noqa: E402

# Nx, Ny, Nz
SHAPES = [(512, 1, 128), (64, 1, 8), (64, 32, 32)]


def _solver(shape):
    Nx, Ny, Nz = shape
    kw = dict(dim=3, Ny=Ny, Ly=4.0) if Ny > 1 else {}
    return RBSolver(Nx, Nz, 4.0, 1e5, 1.0, **kw)


def _solve(g):
    B = torch.from_numpy(si.complex_noise(g.ev_shape, 101)).cuda()
    torch.cuda.synchronize()

    def call():
        g.factor(1e3)
        return g.solve(B)
    return call


def _adjoint(g):
    X = torch.from_numpy(si.complex_noise(g.state_shape, 102)).cuda()
    Xb = torch.from_numpy(si.complex_noise(g.state_shape, 103)).cuda()
    hb = g.new_adjoint_state()[1]
    torch.cuda.synchronize()

    def call():
        g.adjoint_step(X, 1, 1e-3, 1e-3, Xb, hb)
        return Xb
    return call


def _evp(g):
    return lambda: g.evp(0.5, nev=1)[0]


CALLS = {"solve": _solve, "adjoint": _adjoint, "evp": _evp}


@pytest.mark.parametrize("shape, name", [(s, n) for s in SHAPES for n in CALLS
                                         if n == "solve" or s[1:] == (1, 8)],
                         ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_first_factorisation_on_a_side_stream(shape, name):
    out = []
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        g = _solver(shape)
        call = CALLS[name](g)
        with torch.cuda.stream(stream):
            r = call()
        torch.cuda.synchronize()
        out.append(r.cpu().numpy())
        g.close()
    assert np.isfinite(out[0]).all() and np.abs(out[0]).max() > 0
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("gamma", [(), (0.3,)], ids=["tridiagonal", "banded"])
def test_singular_pencil_is_forgotten_by_the_next_factorisation(gamma):
    """stau_last_singular_pencil names the pencil of a failed factorisation
    until one succeeds, in a step as in the component call, whatever form of
    factors the step's operator has."""
    g = RBSolver(16, 8, 4.0, 1e4, 1.0, gamma=gamma)
    for ok in (lambda: g.step(1e-3), lambda: g.factor(1e3)):
        with pytest.raises(StauError, match="SINGULAR"):
            g.factor(0.0, 0.0)
        assert g.last_singular_pencil() >= 0
        ok()
        assert g.last_singular_pencil() == -1
