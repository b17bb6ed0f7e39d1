"""The operator and the Eq. (17) preconditioner at the edges of their launch
rules for small batches, against the oracle: chunks of 4, 8 and 16 planes with
ragged last ones (the chunk shrinks while there are fewer blocks than compute
units), and the electrode term of every stencil order on the register sizes
20, 36 and 40 and on rectangular planes with an odd and an even number of LDS
transform passes (the planes change buffers after an odd number)."""
import numpy as np
import pytest

import oracle as O
from workloads import Grid, random_field

pytestmark = pytest.mark.gpu

PLANES = [(20, 20), (36, 36), (40, 40), (6, 4), (10, 9), (16, 18), (22, 14)]


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _solver(g, V):
    from paper_1009_5300_amd import iobm
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(V)
    return s


@pytest.mark.parametrize("nf", [1, 2, 3])
@pytest.mark.parametrize("nx,ny", PLANES)
def test_electrode_term(torch, nx, ny, nf):
    """Rounding of the stencil and the transforms: 1e-12 and 2e-5 of the largest value, as for the other planes."""
    from paper_1009_5300_amd import iobm
    g = Grid(nx, ny, 2 * nf + 3, 0.4, nf, hz_=0.45)
    V = 0.2 * random_field(g.shape, 11, complex_=False)
    s, P = _solver(g, V), O.Problem(g, V)
    x = random_field((2,) + g.shape, 21)
    ref = P.apply(0.9, x.reshape(2, -1)).reshape(x.shape)
    xt = torch.as_tensor(x, device="cuda")
    y = s.apply(0.9, xt, iobm.C128).cpu().numpy()
    assert np.abs(y - ref).max() <= 1e-12 * np.abs(ref).max()
    y32 = s.apply(0.9, xt.to(torch.complex64), iobm.C64_REFINED).cpu().numpy()
    assert np.abs(y32 - ref).max() <= 2e-5 * np.abs(ref).max()


@pytest.mark.parametrize("nz,nrhs", [(3, 1), (5, 40), (33, 1), (33, 60), (64, 33), (129, 1), (256, 1)])
def test_stencil_chunks(torch, nz, nrhs):
    from paper_1009_5300_amd import iobm
    g = Grid(8, 6, nz, 0.4, 1)
    V = 0.2 * random_field(g.shape, 12, complex_=False)
    s, P = _solver(g, V), O.Problem(g, V)
    x = random_field((nrhs,) + g.shape, 22)
    ref = P.apply(0.9, x.reshape(nrhs, -1)).reshape(x.shape)
    y = s.apply(0.9, torch.as_tensor(x, device="cuda"), iobm.C128).cpu().numpy()
    assert np.abs(y - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nz,nrhs", [(3, 1), (33, 1), (33, 16), (33, 70), (80, 9), (80, 300)])
def test_eq17_chunks(torch, nz, nrhs):
    """z, and a solve that uses the kernel's own r^T z: its true residual is at most the tolerance."""
    from paper_1009_5300_amd import iobm
    g = Grid(8, 6, nz, 0.4, 1)
    V = 0.2 * random_field(g.shape, 13, complex_=False)
    s = _solver(g, V)
    r = random_field((nrhs,) + g.shape, 3)
    ref = O.precond.truncated_laplacian(g, r, 2.0)
    z = s.precondition(iobm.PC_TRUNCATED_LAPLACIAN, torch.as_tensor(r, device="cuda"), alpha=2.0).cpu().numpy()
    assert np.abs(z - ref).max() <= 1e-13 * np.abs(ref).max()
    if nrhs > 16:
        return
    P = O.Problem(g, V)
    out = s.solve([0.9], opts=iobm.default_opts(precision=iobm.C128, precond=iobm.PC_TRUNCATED_LAPLACIAN), want_psi=True)
    assert out["status"] == 0
    psi = out["psi"].cpu().numpy().reshape(len(out["T"]), -1)
    for k, m in enumerate(out["modes"][0]):
        b = P.rhs(0.9, int(m), "L").ravel()
        assert np.linalg.norm(P.apply(0.9, psi[k]).ravel() - b) <= 1e-9 * np.linalg.norm(b)
