"""The tridiagonal pencil solve at every block form of its launch: NP pencils
per block (halved from 256 / Nz, at most eight, while there are fewer blocks
than compute units), L lanes per chain and E degrees per lane.  On 256 units
the shapes below take

  NP = 8: (L, E) = (2, 1), (2, 2), (2, 4), (2, 8);
  NP = 4: (4, 2), (4, 8);    NP = 2: (4, 1), (8, 2), (8, 4), (8, 8);
  NP = 1: (16, 2), (16, 8) and 3-D (16, 16);

in 2-D and 3-D, with a partial last block wherever NP > 1 does not divide the
number of pencil slots (every 2-D shape).

* A boundary value solve (a0 = 0) of every pencil against the banded LU of the
  same operator (stau_factor, stau_solve), 1e-10 relative over the state; the
  inactive slots zero.
* That solve and an SBDF1 step against the oracle on pencils at every place of
  the first block and of the last ones, per pencil, 1e-10 relative: the FP64
  bar of the other solve tests.
* The check build (index checks of the kernels compiled in) on the same calls:
  every check holds, the values are the default library's within 1e-13."""
import os

import numpy as np
import pytest

import seeded_inputs as si
from gpu_helpers import rel_err
from oracle import RBOracle, RBParams

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("no GPU", allow_module_level=True)

from paper_1905_10388_amd import RBSolver, _lib  # noqa: E402

BAR = 1e-10
DT = 1e-3

# dim, Nx, Ny, Nz -> NP, L, E on 256 units
SHAPES = {(2, 4096, 1, 4): (8, 2, 1), (2, 4096, 1, 8): (8, 2, 2), (3, 64, 64, 16): (8, 2, 4), (3, 64, 64, 32): (8, 2, 8),
          (2, 2048, 1, 16): (4, 4, 2), (2, 4096, 1, 64): (4, 4, 8), (3, 64, 32, 16): (4, 4, 2),
          (2, 1024, 1, 8): (2, 4, 1), (2, 1024, 1, 32): (2, 8, 2), (2, 1024, 1, 64): (2, 8, 4), (3, 64, 16, 128): (2, 8, 8),
          (2, 64, 1, 64): (1, 16, 2), (3, 8, 4, 256): (1, 16, 8), (3, 8, 4, 512): (1, 16, 16)}


def block_form(P, N, units):
    """The launch's rule: (NP, L, E)."""
    NP = min(8, max(1, 256 // N))
    while NP > 1 and -(-P // NP) < units:
        NP //= 2
    L = min(16 // NP, N // 2)
    return NP, L, N // 2 // L


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _field(shape, seed):
    Nz = shape[-1]
    X = 0.1 * si.complex_noise(shape, seed) * np.exp(-np.arange(Nz) / max(2.0, Nz / 8.0))
    X[..., shape[-3] - 1, :, :] = 0
    if len(shape) == 4:
        X[shape[0] // 2] = 0
        X[:, 0] = 0  # (the kx = 0 plane stands for a real field only with ky symmetry)
    mean = X[0] if len(shape) == 3 else X[0, 0]
    mean[:] = mean.real
    return X


def _box(dim, Nx):
    return dict(Lx=max(4.0, Nx / 32.0), Ly=3.0)


def _solver(shape, library="default"):
    dim, Nx, Ny, Nz = shape
    b = _box(dim, Nx)
    return RBSolver(Nx, Nz, b["Lx"], 1e5, 0.7, dim=dim, Ny=Ny, Ly=b["Ly"], library=library)


def _run(g, X0, F):
    g.set_state(torch.from_numpy(X0).cuda())
    g.step(DT)
    Xb = g.lbvp(torch.from_numpy(F).cuda())
    return _np(g.X), _np(Xb)


def test_shapes_take_the_stated_block_forms():
    for (dim, Nx, Ny, Nz), form in SHAPES.items():
        P = (Nx // 2 + 1) * (Ny if dim == 3 else 1)
        assert block_form(P, Nz, 256) == form, (dim, Nx, Ny, Nz)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(str(v) for v in s))
def test_block_forms(shape):
    dim, Nx, Ny, Nz = shape
    b = _box(dim, Nx)
    o = RBOracle(Nx, Nz, b["Lx"], RBParams(1e5, 0.7), dim=dim, Ny=Ny, Ly=b["Ly"])
    g = _solver(shape)
    X0, F = _field(o.state_shape, 140), _field(o.state_shape, 141)[..., :o.ne, :].copy()
    Xs, Xb = _run(g, X0, F)

    # every pencil: banded LU
    g.factor(0.0, 1.0)
    PF = F @ o.C.toarray().T
    PF[..., Nz - 1] = 0
    assert rel_err(Xb, _np(g.solve(torch.from_numpy(PF).cuda()))) < BAR
    for X in (Xs, Xb):
        assert np.all(X[..., o.Px - 1, :, :] == 0) and (dim == 2 or np.all(X[Ny // 2] == 0))

    # the oracle on the pencils of the first block, of its neighbour and of the last two
    everything = list(o.pencils())
    P = len(everything)
    NP = block_form(P, Nz, torch.cuda.get_device_properties(0).multi_processor_count)[0]
    slots = set(range(2 * NP + 1)) | set(range(P - 2 * NP - 2, P)) | {P // 2, P // 3}
    sample = [p for i, p in enumerate(everything) if i in slots and p[4]]
    o.pencils = lambda: iter(sample)
    for X, ref in ((Xb, o.lbvp(F)), (Xs, o.step(X0, DT))):
        for key, *_ in sample:
            assert rel_err(X[key], ref[key]) < BAR, (key, rel_err(X[key], ref[key]))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(str(v) for v in s))
def test_block_forms_in_the_check_build(shape):
    if not os.path.exists(_lib.LIB_CHECK_PATH):  # pragma: no cover
        pytest.skip("libstau_check.so not built (__graft_entry__.build() builds it)")
    out = []
    for library in ("check", "default"):
        g = _solver(shape, library)
        X0, F = _field(g.state_shape, 142), _field(g.state_shape, 143)[..., :g.info["ne"], :].copy()
        r = _run(g, X0, F)
        g.check()
        out.append(r)
        g.close()
    for a, b in zip(*out):
        assert np.linalg.norm(a - b) <= 1e-13 * np.linalg.norm(b)
