"""The mode-space iteration of the lateral-Fourier preconditioner at the edges
of its kernels: plane counts around the chunk of 8 planes and around the
changes of the mode-block width (64 and 128 planes), every register plane
size and the LDS one, rectangular and odd planes, the nonlocal term, and
systems that need many times the steps that the ring of residuals holds.  psi is checked in the oracle's own system: its residual is
at most 10 tol ||b|| (the solver stops at tol = 1e-10 on its own FP64 residual
of the same system; the two evaluations differ by FP64 rounding, some 1e-13 of
||b||)."""
import numpy as np
import pytest

import oracle as O
from workloads import Grid
from workloads.synth import _kb_projectors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _potential(g, depth, rng):
    """Gaussian wells of the given depth along the axis over a weak random field."""
    k, j, i = np.meshgrid(np.arange(g.nz), np.arange(g.ny), np.arange(g.nx), indexing="ij")
    V = 0.02 * rng.uniform(-1, 1, g.shape)
    for f in (0.3, 0.7):
        r2 = (((i - g.nx / 2) * g.hx) ** 2 + ((j - g.ny / 2) * g.hy) ** 2 + ((k - f * g.nz) * g.hz) ** 2)
        V -= depth * np.exp(-r2 / (2 * 1.5 ** 2))
    return V


CASES = [(8, 8, nz, nf, 0.2, 0) for nf, nz in ((1, 2), (2, 4), (3, 7), (2, 8), (2, 9), (2, 64), (1, 65), (2, 128),
                                               (2, 129), (1, 256))]
CASES += [(n, n, 10, 2, 0.2, 0) for n in (12, 16, 24, 32)]
CASES += [(9, 6, 33, 3, 0.2, 0), (21, 10, 17, 2, 0.2, 0)]
CASES += [(8, 8, 40, 2, 0.6, 4), (10, 9, 30, 1, 0.6, 3), (8, 8, 72, 1, 1.6, 0)]  # nonlocal; many steps


@pytest.mark.parametrize("precision", [0, 1], ids=["c128", "c64"])
@pytest.mark.parametrize("nx,ny,nz,nf,depth,rank", CASES)
def test_psi_solves_the_oracles_system(torch, nx, ny, nz, nf, depth, rank, precision):
    from paper_1009_5300_amd import iobm
    g = Grid(nx, ny, nz, 0.45, nf, hz_=0.5)
    rng = np.random.default_rng(nx + 7 * ny + 31 * nz + nf)
    V = _potential(g, depth, rng)
    nl = None
    if rank:
        centres = [np.array([g.nx * g.hx / 2, g.ny * g.hy / 2, f * g.nz * g.hz]) for f in (0.3, 0.7)]
        nl = _kb_projectors(g, centres, 0.6, rank, rng)
    P = O.Problem(g, V, nl)
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(V)
    if nl is not None:
        s.set_nonlocal(nl)
    E = [0.35, 1.3]
    for side in (0, 1):
        out = s.solve(E, opts=iobm.default_opts(precision=precision, side=side), want_psi=True)
        assert out["status"] == 0, out.get("error")
        psi = out["psi"].cpu().numpy().reshape(len(out["T"]), -1)
        k = 0
        for e, Ee in enumerate(E):
            for m in out["modes"][e]:
                b = P.rhs(Ee, int(m), "LR"[side]).ravel()
                r = np.linalg.norm(P.apply(Ee, psi[k]).ravel() - b) / np.linalg.norm(b)
                assert r <= 1e-9, (Ee, int(m), side, r)
                k += 1
        assert np.abs(out["T"] + out["R"] - 1).max() <= 1e-7


@pytest.mark.parametrize("seed", [1, 5, 20])
def test_iterations_of_a_chain_stay_bounded(torch, seed):
    """Each of these chains (24 x 24 x 96 with projectors, 230 to 240 states) has a state that lost the conjugacy of
    its directions to rounding when beta came from the residual products alone, and took 947, 2713 and 1204 steps;
    the recurrence that applies the operator takes at most 255 on such chains.  Bound: twice that."""
    from perf import cases
    case = next(c for c in cases.listed() if c["name"] == "solve_chain")
    state = cases.prepare(case, seed)
    out = state["solver"].solve(state["E"], opts=state["opts"])
    assert out["status"] == 0
    assert max(st[0] for st in np.array(out["stats"])) <= 510


@pytest.mark.parametrize("n,m,nz,nf,h,depth,seeds", [(12, 12, 64, 1, 0.5, 3.0, (4, 11)), (10, 9, 48, 2, 0.5, 2.0, (5, 22)),
                                                     (12, 12, 48, 3, 0.35, 5.0, (3, 6, 7, 13))])
def test_states_that_stagnate_in_mode_space(torch, n, m, nz, nf, h, depth, seeds):
    """Deep wells whose complex64 states need up to a thousand steps a replacement: the mode-space recurrence alone
    leaves states of each grid above 1e-10 at 6,000 steps, where the one that applies the operator takes at most 5,750
    on such potentials.  Each converges within 8,000, and psi to the complex128 solve's: both stop at 1e-10 of the
    right-hand side, and these wells' resolvents are some 1e3 in these units: 1e-6 of the largest |psi|."""
    from paper_1009_5300_amd import iobm
    s = iobm.Solver(n, m, nz, (h, h, h), nf)
    for seed in seeds:
        rng = np.random.default_rng(seed)
        k, j, i = np.meshgrid(np.arange(nz), np.arange(m), np.arange(n), indexing="ij")
        V = 0.02 * rng.uniform(-1, 1, (nz, m, n))
        for f in (0.3, 0.7):
            V -= depth * np.exp(-(((i - n / 2) * h) ** 2 + ((j - m / 2) * h) ** 2 + ((k - f * nz) * h) ** 2) / 4.5)
        s.set_potential(V)
        E = list(rng.uniform(0.1, 1.0, 6))
        for graph in (0, 1):
            out = s.solve(E, opts=iobm.default_opts(precision=iobm.C64_REFINED, max_iter=8000, graph=graph), want_psi=True)
            assert out["status"] == 0, (seed, graph, max(st[0] for st in out["stats"]))
        ref = s.solve(E, opts=iobm.default_opts(precision=iobm.C128), want_psi=True)
        assert ref["status"] == 0
        assert float((out["psi"] - ref["psi"]).abs().max()) <= 1e-6 * float(ref["psi"].abs().max())


@pytest.mark.parametrize("precision", [0, 1], ids=["c128", "c64"])
@pytest.mark.parametrize("n,nz,nf,depth,rank", [(48, 9, 2, 0.2, 0), (48, 9, 1, 0.6, 2), (24, 15, 2, 0.6, 4), (32, 7, 3, 0.2, 2)])
def test_wide_planes(torch, n, nz, nf, depth, rank, precision):
    """The largest register planes, with and without the nonlocal term (in complex128 two lanes share a line from 24
    points on, and the mirror lines of the transform are exchanged between them).  An odd number of states and of
    planes: the last block of 48 x 48 planes in complex128 and of 24 x 24 ones holds a plane past the last.  psi in
    the oracle's own system, as above."""
    from paper_1009_5300_amd import iobm
    g = Grid(n, n, nz, 0.45, nf, hz_=0.5)
    rng = np.random.default_rng(n + nz + nf)
    V = _potential(g, depth, rng)
    nl = None
    if rank:
        centres = [np.array([g.nx * g.hx / 2, g.ny * g.hy / 2, f * g.nz * g.hz]) for f in (0.3, 0.7)]
        nl = _kb_projectors(g, centres, 0.6, rank, rng)
    P = O.Problem(g, V, nl)
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(V)
    if nl is not None:
        s.set_nonlocal(nl)
    out = s.solve([0.35], opts=iobm.default_opts(precision=precision), want_psi=True)
    assert out["status"] == 0, out.get("error")
    assert len(out["T"]) % 2 == 1
    psi = out["psi"].cpu().numpy().reshape(len(out["T"]), -1)
    for k, m in enumerate(out["modes"][0]):
        b = P.rhs(0.35, int(m), "L").ravel()
        assert np.linalg.norm(P.apply(0.35, psi[k]).ravel() - b) <= 1e-9 * np.linalg.norm(b), int(m)
    assert np.abs(out["T"] + out["R"] - 1).max() <= 1e-7
