#!/usr/bin/env python3
"""Throughput benchmark of the IOBM scattering solve on one MI355X.

Workload: the large cross-section wire (48 x 48 x 128 grid, h = 0.4 bohr,
4th-order FD, jellium electrodes, seeded smooth random V of amplitude
0.02 Ha), 16 energies with 45-57 open lateral channels each, 768
scattering states per pass.  One step = one iobm_solve over the whole batch:
mode setup, right-hand sides, batched complex64 COCG with the lateral-
Fourier preconditioner and FP64 iterative refinement to ||r|| <= 1e-10 ||b||,
readout of every transmission amplitude.  V and every work buffer are
resident on the GPU before the timed region.

Prints one JSON line: solves/s of the whole job, the roofline of the
dominant kernel and of the stencil operator (HIP events on the solver's
stream over the timed region), the plain FP64 single-right-hand-side COCG
on a sample of channels (the comparison point, also the |Delta T| check),
the paper's Eq. (17) preconditioner on one energy, and the CPU oracle timed
on a bounded sample of the workload.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0  # MI355X HBM3E
# HBM traffic of the dominant kernel, measured with rocprofv3 counters
# (FETCH_SIZE and WRITE_SIZE, calibrated on a plain copy kernel), kept with
# the git blob ids of the sources it was measured on: the kernels, and the
# solver driver, whose iteration schedule sets the sizes of the launches
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic.txt")
KERNEL_SOURCES = ["paper_1009_5300_amd/csrc/ops.hip", "paper_1009_5300_amd/csrc/modal.hip",
                  "paper_1009_5300_amd/csrc/modal.h", "paper_1009_5300_amd/csrc/fftreg.h",
                  "paper_1009_5300_amd/csrc/common.h", "paper_1009_5300_amd/csrc/internal.h",
                  "paper_1009_5300_amd/csrc/api.hip"]


def _blob_id(path):
    import hashlib
    data = open(os.path.join(ROOT, path), "rb").read()
    return hashlib.sha1(b"blob %d\0" % len(data) + data).hexdigest()


def _measured_traffic(kernel, launches_per_solve=None):
    """HBM bytes per launch of `kernel` from the committed counter summary,
    or None if there is none or the kernel sources changed since.  A record
    taken per solve is divided by `launches_per_solve`: the residual-driven
    check schedule may split one solve's iterations into a different number
    of launches from run to run, while the bytes per solve stay put."""
    if not os.path.exists(TRAFFIC_FILE):
        return None
    rec = {}
    for line in open(TRAFFIC_FILE):
        line = line.strip()
        if line and not line.startswith("#") and "=" in line:
            k, v = line.split("=", 1)
            rec[k.strip()] = v.strip()
    if rec.get("kernel_class") != kernel:
        return None
    for src in KERNEL_SOURCES:
        if rec.get("blob " + src) != _blob_id(src):
            return None
    try:
        if "hbm_bytes_per_solve" in rec:
            if not launches_per_solve:
                return None
            return float(rec["hbm_bytes_per_solve"]) / launches_per_solve
        return float(rec["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def copy_calibration(gib=1.0, reps=4):
    """A plain device copy of known size (the counter calibration run):
    reads and writes `gib` GiB per launch."""
    import torch
    n = int(gib * (1 << 30)) // 4
    a = torch.ones(n, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    torch.cuda.synchronize()
    for _ in range(reps):
        b.copy_(a)
    torch.cuda.synchronize()
    print(json.dumps({"copy_calibration": {"bytes_read_per_launch": 4 * n, "bytes_written_per_launch": 4 * n,
                                           "launches": reps}}), flush=True)


def _kernel_stats(s, cls):
    n, ms, alg = s.profile_end(cls)
    if n == 0:
        return None
    return {"launches": n, "total_ms": ms, "avg_ms": ms / n, "alg_bytes_per_launch": alg / n,
            "achieved_GBps": alg / (ms * 1e-3) / 1e9}


def _cpu_info():
    model = None
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    try:
        ncpu = len(os.sched_getaffinity(0))
    except AttributeError:
        ncpu = os.cpu_count()
    return model, ncpu


def cpu_baseline():
    """The oracle on a bounded sample of the workload: the same recipe
    (48 x 48 cross-section, h = 0.4, 4th-order FD, V statistics, first
    energy, all 45 open channels) on a z-shortened 48 x 48 x 6 grid (the two
    electrode plane groups and two interior planes; about 10-30 s of CPU
    work), solved with the oracle's dense path (its sparse LU does not finish on a 48 x 48
    cross-section: the dense 4608 x 4608 self-energy blocks defeat the
    ordering).  Times the assembly (self-energies by explicit sums), the
    solve of every channel and the current readout.  The full 128-plane grid
    is out of the oracle's reach, so this rate overstates the oracle on the
    real workload.  Returns solves/s."""
    import numpy as np
    from threadpoolctl import threadpool_info

    import oracle as O
    from workloads import Grid, make

    g = Grid(48, 48, 6, 0.4, 2)
    w = make(4, g)
    E = float(w.energies[0])
    t0 = time.perf_counter()
    P = O.Problem(g, w.V)
    modes = O.open_channels(g, E)
    psi = P.solve(E, modes, dense=True, check=False)
    T = [P.currents(E, m, p)[0] for m, p in zip(modes, psi)]
    dt = time.perf_counter() - t0
    threads = max([d.get("num_threads", 1) for d in threadpool_info()] + [1])
    model, ncpu = _cpu_info()
    assert np.all(np.isfinite(T))
    return {"value": len(modes) / dt, "unit": "solves/s", "cores": threads, "kind": "oracle",
            "host_cpus": ncpu, "cpu_model": model,
            "sample": f"48x48x6 grid (the workload recipe on a z-shortened copy of its cross-section), "
                      f"E={E} Ha, {len(modes)} channels, dense LU (LAPACK, {threads} BLAS threads) + "
                      f"solves + current readout in {dt:.1f} s"}


MFMA_F32_PEAK_TFLOPS = 157.3  # MI355X dense FP32 matrix


def chain_workload(args):
    """Workload 3 (24 x 24 x 96, h = 0.35, 6th-order FD, six wells with a
    rank-4 separable nonlocal term each, 32 energies, 236 states): solves/s
    and the MFMA projection kernel's achieved FLOP/s.  A secondary
    measurement: this batch (104 MB per complex64 vector) lives in the
    256 MB last-level cache, so it is not HBM-bound."""
    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import make

    torch.cuda.set_device(0)
    w = make(3)
    g = w.grid
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(w.V)
    s.set_nonlocal(w.nonlocal_)
    opts = iobm.default_opts()
    out = s.solve(w.energies, opts=opts)
    for _ in range(args.warmup):
        out = s.solve(w.energies, opts=opts)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        out = s.solve(w.energies, opts=opts)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    assert out["status"] == 0, out.get("error")
    nrhs = len(out["T"])
    s.profile_begin([iobm.K_NONLOCAL, iobm.K_NONLOCAL_C128, iobm.K_STENCIL])
    for _ in range(args.steps):
        out = s.solve(w.energies, opts=opts)
    kb = {}
    for name, cls, peak in (("nonlocal_c64", iobm.K_NONLOCAL, MFMA_F32_PEAK_TFLOPS),
                            ("nonlocal_c128", iobm.K_NONLOCAL_C128, 78.6)):
        n, ms, flops = s.profile_end(cls)
        if n:
            tf = flops / (ms * 1e-3) / 1e12
            kb[name] = {"launches": n, "avg_ms": round(ms / n, 4), "flops_per_launch": flops / n,
                        "achieved_TFLOPs": round(tf, 3), "peak_TFLOPs": peak, "frac": round(tf / peak, 5)}
    n, ms, b = s.profile_end(iobm.K_STENCIL)
    s.profile_begin([])
    nsup = len(np.unique(np.concatenate([np.asarray(x).ravel() for x in w.nonlocal_.support])))
    stats = np.array(out["stats"], dtype=float)
    print(json.dumps({
        "metric": "scattering solves/sec, atomic chain with nonlocal term", "value": round(args.steps * nrhs / (t1 - t0), 2),
        "unit": "solves/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(1e3 * (t1 - t0) / args.steps, 3), "higher_is_better": True, "dtype": "c64+f64",
        "data": "synthetic",
        "config": {"workload": "chain 24x24x96 h=0.35 6th-order FD, 6 wells with rank-4 nonlocal terms, "
                               "32 energies, 236 scattering states", "nonlocal_support_points": int(nsup),
                   "projectors": int(sum(np.asarray(d).shape[0] for d in w.nonlocal_.D))},
        "nonlocal_mfma": kb,
        "stencil_avg_ms": round(ms / n, 4) if n else None,
        "solve_stats": {"iters_mean": float(stats[:, 0].mean()), "refinements_mean": float(stats[:, 1].mean()),
                        "max_rel_residual": float(stats[:, 3].max()),
                        "max_flux_error": float(np.abs(stats[:, 4]).max())},
    }), flush=True)


def adjoint_workload(args):
    """Workload 5 (32 x 32 x 96, h = 0.4, 4th-order FD, four wells, 4
    energies, 28 scattering states): dT/dV by the adjoint method, i.e. the
    forward solves, the readout, the adjoint solves and the gradient
    contraction, per second."""
    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import make

    torch.cuda.set_device(0)
    w = make(5)
    g = w.grid
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(w.V)
    T, grad = s.grad_transmission(w.energies)
    for _ in range(args.warmup):
        T, grad = s.grad_transmission(w.energies)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        T, grad = s.grad_transmission(w.energies)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    nstates = sum(len(s.channels(E)[0]) for E in w.energies)
    print(json.dumps({
        "metric": "transmission gradients dT/dV per second (forward + adjoint solves)",
        "value": round(args.steps / (t1 - t0), 3), "unit": "gradients/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(1e3 * (t1 - t0) / args.steps, 3), "higher_is_better": True,
        "dtype": "c64+f64", "data": "synthetic",
        "config": {"workload": "adjoint 32x32x96 h=0.4 4th-order FD, 4 wells, 4 energies",
                   "forward_states": int(nstates), "adjoint_states": int(nstates)},
        "T_total": float(T), "max_abs_grad": float(grad.abs().max()),
    }), flush=True)


def na_sweep(atoms=(3, 4, 5, 6, 7, 8)):
    """The paper's preconditioner experiment (Sec. III, Table 2) on the
    synthetic Na-like wires: average COCG iterations per incident wave at the
    jellium Fermi level without a preconditioner, with Eq. (17) at
    alpha = 3.0, 2.4, 1.8, and with the lateral-Fourier preconditioner;
    complex128 iterations, convergence checked after every iteration, FP64
    residual 1e-10.  One COCG solve per cos / sin standing wave, so a +-G
    channel pair counts its two solves once each."""
    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import na_wire

    torch.cuda.set_device(0)
    cases = [("none", iobm.PC_NONE, 1.8), ("alpha=3.0", iobm.PC_TRUNCATED_LAPLACIAN, 3.0),
             ("alpha=2.4", iobm.PC_TRUNCATED_LAPLACIAN, 2.4), ("alpha=1.8", iobm.PC_TRUNCATED_LAPLACIAN, 1.8),
             ("lateral_fft", iobm.PC_LATERAL_FFT, 1.8)]
    rows = []
    for n in atoms:
        w = na_wire(n)
        g = w.grid
        s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
        s.set_potential(w.V)
        row = {"n_atom": n, "nz": g.nz}
        Tref = None
        for name, pc, alpha in cases:
            o = iobm.default_opts(precision=iobm.C128, precond=pc, alpha=alpha, check_every=1, max_iter=400000)
            t0 = time.perf_counter()
            out = s.solve(w.energies, opts=o)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            ids = [int(m) for m in out["modes"][0]]
            row[name] = {"iters_per_wave": round(_iters_per_wave(out, g), 1), "status": int(out["status"]),
                         "s": round(dt, 3)}
            if Tref is None:
                Tref = out["T"]
                row["channels"] = len(ids)
                row["T_total"] = float(out["T"].sum())
            else:
                row[name]["max_dT"] = float(np.abs(out["T"] - Tref).max())
        rows.append(row)
    mean = {name: float(np.mean([r[name]["iters_per_wave"] for r in rows])) for name, _, _ in cases}
    print(json.dumps({"experiment": "preconditioner sweep on synthetic Na-like wires (Table 2 analogue)",
                      "energy_Ha": float(na_wire(atoms[0]).energies[0]), "rows": rows,
                      "mean_iters_per_wave": {k: round(v, 1) for k, v in mean.items()},
                      "speedup_vs_none": {k: round(mean["none"] / v, 2) for k, v in mean.items()}}), flush=True)


def _iters_per_wave(out, g):
    """Mean COCG iterations per standing-wave solve.  The channels of a +-G
    pair are solved as one cos and one sin standing wave, and each of the two
    channels reports both solves summed; a self-paired channel is one solve.
    So the solves number the channels, and weighting the pair's reports by
    1/2 counts every solve once."""
    ids = [int(m) for e in range(len(out["modes"])) for m in out["modes"][e]]
    wgt = [1.0 if ((g.ny - m // g.nx) % g.ny) * g.nx + (g.nx - m % g.nx) % g.nx == m else 0.5 for m in ids]
    return sum(st[0] * c for st, c in zip(out["stats"], wgt)) / len(ids)


def precision_sweep():
    """Iterations of the preconditioned COCG per standing-wave solve, and its
    wall time, for each preconditioner (none, the paper's Eq. (17) at
    alpha = 1.8, Jacobi, lateral-Fourier) in complex128 and in complex64 with
    FP64 residual replacement (search direction restarted at a replacement,
    or kept), on the wide wire's first energy (48 x 48 x 128, 45
    channels) and on the shortest synthetic Na-like wire (36 x 36 x 80, 9
    channels).  Transmissions of every variant against the first."""
    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import make, na_wire

    torch.cuda.set_device(0)
    cases = [("wide_48x48x128_E0.71", make(4), [0.71]), ("na3_36x36x80_EF", na_wire(3), None)]
    pcs = [("none", iobm.PC_NONE), ("eq17_alpha1.8", iobm.PC_TRUNCATED_LAPLACIAN), ("jacobi", iobm.PC_JACOBI),
           ("lateral_fft", iobm.PC_LATERAL_FFT)]
    precs = [("c128", iobm.C128, 0), ("c64_restart", iobm.C64_REFINED, 0), ("c64_keep", iobm.C64_REFINED, 1)]
    res = {}
    for name, w, Es in cases:
        g = w.grid
        Es = list(w.energies) if Es is None else Es
        s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
        s.set_potential(w.V)
        s.solve(Es, opts=iobm.default_opts(precond=iobm.PC_LATERAL_FFT))  # tune, allocate
        s.solve(Es, opts=iobm.default_opts(precision=iobm.C128, precond=iobm.PC_LATERAL_FFT))
        Tref = None
        rows = {}
        for pname, pc in pcs:
            for qname, prec, rep in precs:
                o = iobm.default_opts(precision=prec, precond=pc, keep_direction=rep, max_iter=400000, check_every=4)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                out = s.solve(Es, opts=o)
                torch.cuda.synchronize()
                dt = time.perf_counter() - t0
                if Tref is None:
                    Tref = out["T"]
                rows[f"{pname}/{qname}"] = {"iters_per_wave": round(_iters_per_wave(out, g), 1),
                                            "s": round(dt, 3), "status": int(out["status"]),
                                            "max_dT": float(np.abs(out["T"] - Tref).max())}
                print(json.dumps({"case": name, "variant": f"{pname}/{qname}", **rows[f"{pname}/{qname}"]}),
                      flush=True)
        res[name] = rows
    print(json.dumps({"experiment": "preconditioner x precision sweep", "rows": res}), flush=True)


def block_sweep(only=None):
    """Block COCG per energy against per-state COCG, both in complex128, on
    the wide wire (48 x 48 x 128): the lateral-Fourier preconditioner over
    all 16 energies (768 states), the paper's Eq. (17) (alpha = 1.8) and no
    preconditioner on the first energy (45 states).  Iterations per
    standing-wave solve, solves/s, and |Delta T| against the per-state run;
    one line per variant as it finishes."""
    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import make

    torch.cuda.set_device(0)
    w = make(4)
    g = w.grid
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(w.V)
    s.solve(w.energies, opts=iobm.default_opts(precision=iobm.C128))  # tune, allocate
    rows = {}
    for pname, pc, Es in (("lateral_fft", iobm.PC_LATERAL_FFT, list(w.energies)),
                          ("eq17_alpha1.8", iobm.PC_TRUNCATED_LAPLACIAN, [w.energies[0]]),
                          ("none", iobm.PC_NONE, [w.energies[0]])):
        if only and pname != only:
            continue
        Tref = None
        for mode, blk in (("per_state", 0), ("block", 1)):
            print(json.dumps({"starting": f"{pname}/{mode}"}), flush=True)
            o = iobm.default_opts(precision=iobm.C128, precond=pc, block=blk, max_iter=100000,
                                  check_every=4 if pc != iobm.PC_LATERAL_FFT else 2)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            out = s.solve(Es, opts=o)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            Tref = out["T"] if Tref is None else Tref
            rows[f"{pname}/{mode}"] = {"states": len(out["T"]), "iters_per_wave": round(_iters_per_wave(out, g), 1),
                                       "solves_per_s": round(len(out["T"]) / dt, 2), "s": round(dt, 3),
                                       "status": int(out["status"]),
                                       "max_dT_vs_per_state": float(np.abs(out["T"] - Tref).max())}
            print(json.dumps({"variant": f"{pname}/{mode}", **rows[f"{pname}/{mode}"]}), flush=True)
    print(json.dumps({"experiment": "block COCG vs per-state COCG (complex128), wide wire 48x48x128",
                      "rows": rows}), flush=True)


def smatrix_workload(args):
    """The headline wire (48 x 48 x 128, 16 energies) solved from both
    electrodes for the full flux-normalised scattering matrix of every
    energy (1,536 scattering states), default options: states per second,
    the unitarity error, and the eigenchannel transmissions (eigenvalues of
    t^dagger t, from the transmission block) of the first energy."""
    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import make

    torch.cuda.set_device(0)
    w = make(4)
    g = w.grid
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(w.V)
    opts = iobm.default_opts()
    for _ in range(max(1, args.warmup)):
        S, stats, status = s.smatrix(w.energies, opts=opts)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        S, stats, status = s.smatrix(w.energies, opts=opts)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    assert status == 0
    nst = sum(x.shape[0] for x in S)
    unit = max(float(np.abs(x.conj().T @ x - np.eye(x.shape[0])).max()) for x in S)
    n0 = S[0].shape[0] // 2
    t = S[0][n0:, :n0]  # transmission block, left incidence
    eig = np.sort(np.linalg.eigvalsh(t.conj().T @ t))[::-1]
    print(json.dumps({
        "metric": "scattering-matrix states/sec (both electrodes, every open channel)",
        "value": round(args.steps * nst / (t1 - t0), 2), "unit": "states/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(1e3 * (t1 - t0) / args.steps, 3), "higher_is_better": True,
        "dtype": "c64+f64", "data": "synthetic",
        "config": {"workload": "wide 48x48x128 h=0.4 4th-order FD, 16 energies, S-matrix of both leads",
                   "states": int(nst)},
        "max_unitarity_error": unit, "total_transmission_E0": float(eig.sum()),
        "eigenchannels_E0_top5": [float(x) for x in eig[:5]],
    }), flush=True)


def bloch_workload(args):
    """The wide wire (48 x 48 x 128, 4th-order FD) at a general lateral Bloch
    vector kappa = (0.37 pi / L_x, 0.61 pi / L_y), the first 4 energies of
    the headline workload: the scattering matrices at kappa and -kappa
    (every open channel from both leads, each state paired with its partner
    at -kappa), biconjugate gradients with the lateral-Fourier
    preconditioner, in complex64 with FP64 replacement (the value) and in
    complex128.  Scattering states per second (both members of a pair count)
    and the achieved HBM bandwidth of the phased stencil."""
    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import make

    torch.cuda.set_device(0)
    w = make(4)
    g = w.grid
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(w.V)
    kap = (0.37 * np.pi / (g.nx * g.hx), 0.61 * np.pi / (g.ny * g.hy))
    Es = list(w.energies[:4])
    nst = 2 * 2 * sum(len(s.channels_bloch(E, kap)[0]) for E in Es)
    res = {}
    for name, prec in (("c64", iobm.C64_REFINED), ("c128", iobm.C128)):
        opts = iobm.default_opts(precision=prec)
        for _ in range(max(1, args.warmup)):
            Sp, Sm, stats, status = s.smatrix_bloch(Es, kap, opts=opts)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            Sp, Sm, stats, status = s.smatrix_bloch(Es, kap, opts=opts)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        assert status == 0
        s.profile_begin([iobm.K_BLOCH_STENCIL, iobm.K_BLOCH_VECTOR, iobm.K_PRECOND_FFT, iobm.K_BOUNDARY,
                         iobm.K_STENCIL_C128])
        s.smatrix_bloch(Es, kap, opts=opts)
        kern = {}
        for kname, cls in (("stencil_bloch", iobm.K_BLOCH_STENCIL), ("vector_bloch", iobm.K_BLOCH_VECTOR),
                           ("precond_fft", iobm.K_PRECOND_FFT), ("boundary", iobm.K_BOUNDARY),
                           ("restart_residual", iobm.K_STENCIL_C128)):
            n, ms, b = s.profile_end(cls)
            if n:
                kern[kname] = {"launches": n, "avg_ms": round(ms / n, 4), "total_ms": round(ms, 3),
                               "alg_bytes_per_launch": b / n, "achieved_GBps": round(b / (ms * 1e-3) / 1e9, 1)}
        s.profile_begin([])
        unit = 0.0
        for Sa in Sp:
            n = Sa.shape[0] // 2
            unit = max(unit, float(np.abs(Sa.conj().T @ Sa - np.eye(2 * n)).max()))
        st = np.array(stats, dtype=float)
        res[name] = {"value": round(args.steps * nst / (t1 - t0), 2), "ms_per_step": round(1e3 * (t1 - t0) / args.steps, 3),
                     "kernels": kern, "pair_iters_mean": float(st[:, 0].mean()),
                     "restarts_mean": float(st[:, 1].mean()), "max_rel_residual": float(st[:, 3].max()),
                     "max_unitarity_error": unit, "S_plus": Sp}
    dS = max(float(np.abs(a - b).max()) for a, b in zip(res["c64"].pop("S_plus"), res["c128"].pop("S_plus")))
    main_ = res["c64"]
    sb = main_["kernels"].get("stencil_bloch")
    print(json.dumps({
        "metric": "scattering states/sec at a lateral Bloch vector (S(kappa) and S(-kappa))",
        "value": main_["value"], "unit": "states/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": main_["ms_per_step"], "higher_is_better": True,
        "dtype": "c64+f64", "data": "synthetic",
        "config": {"workload": "wide 48x48x128 h=0.4 4th-order FD at kappa = (0.37 pi/Lx, 0.61 pi/Ly), 4 energies, "
                               "both leads", "states": int(nst), "precision": "complex64 biconjugate gradients, FP64 "
                               "reductions and replacement to 1e-10", "preconditioner": "lateral-Fourier at G + kappa"},
        "roofline": None if not sb else {"bound": "hbm", "achieved": sb["achieved_GBps"], "peak": 8000.0,
                                         "unit": "GB/s", "frac": round(sb["achieved_GBps"] / 8000.0, 4),
                                         "traffic": None, "kernel": "stencil_bloch"},
        "c64": main_, "c128": res["c128"], "max_dS_c64_vs_c128": dS,
    }), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true", help="skip plain-CG and Eq. (17) samples")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain copy kernel of known size (for the HBM counter calibration)")
    ap.add_argument("--workload", default="4", choices=["3", "4", "5", "na", "precision", "block", "bloch",
                                                         "smatrix"],
                    help="4: the headline wide-wire batch (default); 3: the atomic chain with the nonlocal "
                         "term on MFMA (secondary measurement); 5: the adjoint gradient dT/dV; na: iteration "
                         "counts of the paper's preconditioner experiment on synthetic Na-like wires")
    ap.add_argument("--preconditioner", default=None, choices=["lateral_fft", "eq17_alpha1.8", "none"],
                    help="--workload block: run this preconditioner only")
    args = ap.parse_args()
    if args.copy_calibration:
        copy_calibration()
        return
    if args.gpus == 1 and args.workload == "3":
        chain_workload(args)
        return
    if args.gpus == 1 and args.workload == "5":
        adjoint_workload(args)
        return
    if args.gpus == 1 and args.workload == "na":
        na_sweep()
        return
    if args.gpus == 1 and args.workload == "precision":
        precision_sweep()
        return
    if args.gpus == 1 and args.workload == "block":
        block_sweep(args.preconditioner)
        return
    if args.gpus == 1 and args.workload == "bloch":
        bloch_workload(args)
        return
    if args.gpus == 1 and args.workload == "smatrix":
        smatrix_workload(args)
        return
    if args.gpus != 1:
        print("bench.py measures one GPU (use --gpus 1): the scattering states of different energies are "
              "independent, and runs across several GPUs are not supported.",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_1009_5300_amd import iobm
    from workloads import make

    torch.cuda.set_device(0)
    w = make(4)
    g = w.grid
    s = iobm.Solver(g.nx, g.ny, g.nz, g.spacings, g.nf)
    s.set_potential(w.V)
    opts = iobm.default_opts()
    # one-time setup (not a step): allocation of the batch workspaces, inside
    # the first solve
    torch.cuda.synchronize()
    t_setup = time.perf_counter()
    out = s.solve(w.energies, opts=opts)
    torch.cuda.synchronize()
    t_setup = time.perf_counter() - t_setup
    for _ in range(args.warmup):
        out = s.solve(w.energies, opts=opts)
    torch.cuda.synchronize()

    # timed region 1: throughput, no instrumentation
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        out = s.solve(w.energies, opts=opts)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    nrhs = len(out["T"])
    assert out["status"] == 0, out.get("error")
    value = args.steps * nrhs / (t1 - t0)
    stats = np.array(out["stats"], dtype=float)
    # timed region 2: the same steps with HIP events recorded on the solver's
    # stream around every launch of the profiled kernel classes; the library
    # reports each launch's algorithmic bytes
    classes = {"fft_planes": iobm.K_FFT_PLANES, "plane_pass": iobm.K_FFT_PLANES_UPD, "zfilter": iobm.K_ZFILTER,
               "stencil_c128": iobm.K_STENCIL_C128, "boundary": iobm.K_BOUNDARY,
               "accumulate": iobm.K_ACCUMULATE, "dot": iobm.K_DOT}
    s.profile_begin(list(classes.values()))
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    for _ in range(args.steps):
        out = s.solve(w.energies, opts=opts)
    torch.cuda.synchronize()
    t3 = time.perf_counter()
    kern = {k: _kernel_stats(s, c) for k, c in classes.items()}
    s.profile_begin([])
    # the dominant single kernel by summed time
    dom_name = max((k for k in kern if kern[k]), key=lambda k: kern[k]["total_ms"])
    dom = kern[dom_name]
    roofline = {"bound": "hbm", "achieved": round(dom["achieved_GBps"], 1), "peak": HBM_PEAK_GBPS,
                "unit": "GB/s", "frac": round(dom["achieved_GBps"] / HBM_PEAK_GBPS, 4),
                "traffic": _measured_traffic(dom_name, dom["launches"] / args.steps), "kernel": dom_name,
                "avg_launch_ms": round(dom["avg_ms"], 4),
                "alg_bytes_per_launch": dom["alg_bytes_per_launch"]}
    # the operator's stencil: the iteration with the lateral-Fourier
    # preconditioner does not apply it, so it is timed in plain operator
    # applications (complex64) to a batch of one energy's states
    x = torch.view_as_complex(torch.randn((192,) + w.grid.shape + (2,), dtype=torch.float32, device="cuda"))
    s.apply(float(w.energies[0]), x, iobm.C64_REFINED)
    s.profile_begin([iobm.K_STENCIL])
    for _ in range(5):
        s.apply(float(w.energies[0]), x, iobm.C64_REFINED)
    st = _kernel_stats(s, iobm.K_STENCIL)
    s.profile_begin([])
    del x
    stencil = {"achieved": round(st["achieved_GBps"], 1), "unit": "GB/s",
               "frac": round(st["achieved_GBps"] / HBM_PEAK_GBPS, 4), "avg_launch_ms": round(st["avg_ms"], 4),
               "alg_bytes_per_launch": st["alg_bytes_per_launch"],
               "note": "operator application to 192 complex64 vectors: reads x, writes the stencil's result"}
    tot_ms = sum(v["total_ms"] for v in kern.values() if v)
    tot_b = sum(v["alg_bytes_per_launch"] * v["launches"] for v in kern.values() if v)
    whole = {"achieved": round(tot_b / (tot_ms * 1e-3) / 1e9, 1), "unit": "GB/s",
             "frac": round(tot_b / (tot_ms * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
             "kernel_ms_per_step": round(tot_ms / args.steps, 2)}

    result = {
        "metric": "scattering solves/sec + stencil HBM GB/s at |dT|<=1e-6 vs plain FP64 CG",
        "value": round(value, 2), "unit": "solves/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(1e3 * (t1 - t0) / args.steps, 3),
        "ms_per_step_instrumented": round(1e3 * (t3 - t2) / args.steps, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "c64+f64",
        "data": "synthetic",
        "config": {"workload": "wide 48x48x128 h=0.4 4th-order FD, 16 energies, 768 scattering states",
                   "precision": "complex64 COCG, FP64 reductions and refinement to 1e-10",
                   "preconditioner": "lateral-Fourier (flat-wire inverse)"},
        "roofline": roofline,
        "stencil": stencil,
        "all_kernels": whole,
        "setup_s": round(t_setup, 3),
        "kernels": {k: ({kk: (round(vv, 4) if isinstance(vv, float) else vv) for kk, vv in v.items()} if v else None)
                    for k, v in kern.items()},
        "solve_stats": {"per": "channel (cos + sin standing-wave solves of a +-G pair summed)",
                        "iters_mean": float(stats[:, 0].mean()), "iters_max": int(stats[:, 0].max()),
                        "refinements_mean": float(stats[:, 1].mean()),
                        "max_rel_residual": float(stats[:, 3].max()),
                        "max_flux_error": float(np.abs(stats[:, 4]).max())},
    }

    if not args.no_extras:
        # plain FP64 single-right-hand-side COCG (no preconditioner) on a sample
        # of channels: the comparison point of the metric and the |dT| check
        plain = iobm.default_opts(precision=iobm.C128, precond=iobm.PC_NONE, check_every=32)
        Tb = {}
        k = 0
        for e, E in enumerate(w.energies):
            for m in out["modes"][e]:
                Tb[(e, int(m))] = out["T"][k]
                k += 1
        sample = [(0, int(out["modes"][0][0])), (len(w.energies) - 1, int(out["modes"][-1][0]))]
        dts, iters, dT, statuses = [], [], [], []
        for e, m in sample:
            torch.cuda.synchronize()
            a = time.perf_counter()
            o1 = s.solve([w.energies[e]], channels=[[m]], opts=plain)
            torch.cuda.synchronize()
            dts.append(time.perf_counter() - a)
            iters.append(o1["stats"][0][0])
            statuses.append(int(o1["status"]))
            dT.append(abs(o1["T"][0] - Tb[(e, m)]))
        result["plain_fp64_cg"] = {"value": round(len(sample) / sum(dts), 4), "unit": "solves/s",
                                   "status": statuses,
                                   "sample": f"{len(sample)} channels (lowest channel at the first and "
                                             f"last energy), one complex128 COCG solve each, no preconditioner",
                                   "iters": iters, "speedup_of_value": round(value / (len(sample) / sum(dts)), 1)}
        result["max_dT_vs_plain_fp64_cg"] = float(max(dT))
        # the paper's Eq. (17) preconditioner against no preconditioner, both
        # in complex128 (weak preconditioners converge faster in complex128 than
        # in complex64 with replacement), batched over the first energy; the
        # paper's Table 2 reports 1.27 / 1.67 / 2.24x fewer iterations at
        # alpha = 3.0 / 2.4 / 1.8
        pcg = {}
        for name, pc in (("none", iobm.PC_NONE), ("eq17_alpha1.8", iobm.PC_TRUNCATED_LAPLACIAN)):
            o = iobm.default_opts(precision=iobm.C128, precond=pc, alpha=1.8, check_every=32, max_iter=400000)
            torch.cuda.synchronize()
            a = time.perf_counter()
            o2 = s.solve([w.energies[0]], opts=o)
            torch.cuda.synchronize()
            b = time.perf_counter() - a
            pcg[name] = {"solves_per_s": round(len(o2["T"]) / b, 3), "iters_per_wave": round(_iters_per_wave(o2, g), 1),
                         "status": int(o2["status"]),
                         "max_dT_vs_value": float(np.abs(o2["T"] - out["T"][:len(o2["T"])]).max())}
        pcg["iteration_ratio_none_over_eq17"] = round(pcg["none"]["iters_per_wave"] /
                                                      pcg["eq17_alpha1.8"]["iters_per_wave"], 2)
        pcg["sample"] = f"first energy, {len(o2['T'])} channels, complex128, batched"
        result["paper_pcg"] = pcg

    if not args.no_cpu_baseline:
        result["cpu_baseline"] = cpu_baseline()

    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
