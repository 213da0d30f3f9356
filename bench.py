#!/usr/bin/env python3
"""Benchmark of the SEM elastic time step on one MI355X.

Workload: layered elastic cube on 64^3 hexahedra (262,144 elements, NGLL 5,
16,974,593 unique GLL points), interior vertices jittered by +-10% of h,
three flat layers (vp 6000/4000/2500 m/s, vp/vs 1.73, rho 2500) with a +-5%
Gaussian random field (correlation length 4 elements), vertical Ricker point
force (10 Hz) at the centre vertex, 8 receivers on the top face, dt from
Courant number 0.4.  FP32 storage and arithmetic, graph-coloured assembly.

A step is one explicit Newmark step: correct/predict update, the element
force operator f = -K u over every element (the hot path), source injection
and receiver recording.  ``value`` is element-local GLL-point force
evaluations per second over the timed steps (E n^3 per step).

Prints ONE JSON line.  Also reports the force kernel's roofline (HIP events
on the library stream), the force apply alone with coloured and with atomic
assembly, and the FP64 CPU oracle timed on a bounded sample.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E


def progress(msg: str):
    """One line per finished phase on stderr (stdout carries only the JSON line)."""
    print(f"[bench] {msg}", file=sys.stderr, flush=True)
NE, NGLL = 64, 5


def bytes_per_element_model(n: int, nglob: int, nspec: int, geometry: str = "stored") -> float:
    """The byte model: algorithmic HBM bytes per element per force apply, for the
    formulation with a per-point inverse Jacobian: node numbers 4 n^3, Gamma and
    det J 10 s n^3 (10 s per element on affine elements), lambda and mu 2 s n^3,
    u read once and f written once per unique node 3 s G/E each (s = 4, FP32).
    Kept for every path, including those that read less (the trilinear
    geometry, the affine numbering), so fractions compare like for like."""
    n3 = n ** 3
    geo = 10 * 4 * (n3 if geometry != "regular" else 1)
    return 4 * n3 + geo + 2 * 4 * n3 + 2 * 12.0 * nglob / nspec


def bytes_per_element(n: int, nglob: int, nspec: int, geometry: str = "stored", affine: bool = False) -> float:
    """The bytes this library's force pass actually needs per element (FP32,
    its layout): node numbers 4 n^3 (16 for an affine numbering); geometry:
    Gamma 9*4 n^3 (stored; det J is folded into the material), the 3x8
    trilinear coefficients 96 (rebuilt per point) or one Gamma 36 (regular);
    lambda W det J and mu W det J 2*4 n^3; u read once and f written once per
    unique node (3*4*G/E each)."""
    n3 = n ** 3
    geo = {"stored": 36 * n3, "trilinear": 96, "regular": 36}[geometry]
    nodes = 16 if affine else 4 * n3
    return nodes + geo + 8 * n3 + 2 * 12.0 * nglob / nspec


def bytes_per_element_pass(n: int, nglob: int, nspec: int, geometry: str, affine: bool) -> float:
    """The bytes that the element launch of a time step needs per element where
    its nodal sum belongs to the Newmark pass: what bytes_per_element counts,
    with the element-local forces (3*4 n^3) written in the place of f."""
    return bytes_per_element(n, nglob, nspec, geometry, affine) + 12.0 * n ** 3 - 12.0 * nglob / nspec


def traffic_from_profiles(src_hash: str, key: str = "trilinear"):
    """HBM bytes per launch measured with rocprofv3 PMC counters (`key`: the
    geometry path, whose element launch is meant, or that path with the suffix
    `_skeleton` or `_sum`), if they were taken on the current kernel sources."""
    p = os.path.join(ROOT, "profiles", "force_traffic.json")
    if not os.path.exists(p):
        return None
    try:
        d = json.load(open(p))
    except Exception:
        return None
    if d.get("kernel_source_sha256") != src_hash:
        return None
    return d.get(key, {}).get("bytes_per_launch")


def kernel_source_hash() -> str:
    src = b"".join(open(os.path.join(ROOT, "paper_2606_12850_amd", "csrc", f), "rb").read()
                   for f in ("force_line.hpp", "force_line.hip", "elem_common.hpp", "nodal.hpp"))
    return hashlib.sha256(src).hexdigest()


def write_traffic(run_dir: str):
    """profiles/force_traffic.json from the FETCH_SIZE and WRITE_SIZE runs of
    `bench.py --profile-force` (trilinear): KiB per dispatch of the NGLL 5 line
    kernel, its memory skeleton and the nodal sum, each scaled by what the same
    counter reads for the 1 GiB device copy that follows them."""
    import collections
    import csv
    copy_bytes = 1 << 30
    out = {"kernel_source_sha256": kernel_source_hash(), "unit": "bytes per launch",
           "workload": "layered jittered cube 64^3, NGLL 5 (one launch of 262144 elements, one nodal sum)"}
    for geo, gid in (("trilinear", 2),):
        d = {}
        for ctr in ("FETCH_SIZE", "WRITE_SIZE"):
            agg = collections.defaultdict(list)
            path = os.path.join(run_dir, f"pmc_{geo}_{ctr}", "run_counter_collection.csv")
            for r in csv.DictReader(open(path)):
                if r["Counter_Name"] == ctr:
                    agg[r["Kernel_Name"]].append(float(r["Counter_Value"]))
            cp = [v for k, vs in agg.items() if "copyBuffer" in k for v in vs][-3:]
            scale = copy_bytes / (sum(cp) / len(cp) * 1024.0)
            for tag, pat in (("kernel", f"force_line_kernel<float, 5, 3, {gid}, true"),
                             ("skeleton", f"force_line_skeleton_kernel<5, {gid}, true>"),
                             ("sum", "gather_kernel<float, 3")):
                kv = [v for k, vs in agg.items() if pat in k for v in vs]
                if kv:
                    d.setdefault(tag, {})[ctr] = {
                        "kib_per_dispatch": sum(kv) / len(kv), "dispatches": len(kv),
                        "copy_kib_per_dispatch": sum(cp) / len(cp), "scale": scale,
                        "bytes_per_launch": sum(kv) / len(kv) * 1024.0 * scale}
        for tag in d:
            d[tag]["bytes_per_launch"] = sum(d[tag][c]["bytes_per_launch"] for c in ("FETCH_SIZE", "WRITE_SIZE"))
        out[geo] = d["kernel"]
        for tag in ("skeleton", "sum"):
            if tag in d:
                out[f"{geo}_{tag}"] = d[tag]
    out["bytes_per_launch"] = out["trilinear"]["bytes_per_launch"]
    with open(os.path.join(ROOT, "profiles", "force_traffic.json"), "w") as fh:
        json.dump(out, fh, indent=1)
    print(json.dumps({k: (v["bytes_per_launch"] if isinstance(v, dict) else v) for k, v in out.items()}))


def write_acoustic_traffic(run_dir: str):
    """profiles/acoustic_traffic.json from the FETCH_SIZE and WRITE_SIZE runs
    of `bench.py --acoustic-only` (DIR/pmc_ac_<counter>/run_counter_collection.csv):
    KiB per dispatch of the NGLL 5 coloured acoustic force kernel on each
    geometry path, scaled by what the same counter reads for the 1 GiB device
    copies that follow them."""
    import collections
    import csv
    copy_bytes = 1 << 30
    src = b"".join(open(os.path.join(ROOT, "paper_2606_12850_amd", "csrc", f), "rb").read()
                   for f in ("acoustic.hip", "elem_common.hpp"))
    out = {"unit": "bytes per launch",
           "workload": "layered-cube mesh 64^3 jittered, NGLL 5, homogeneous acoustic medium, colored "
                       "(8 launches of 32768 elements), affine node numbering",
           "kernel_source_sha256": hashlib.sha256(src).hexdigest()}
    agg = {}
    for ctr in ("FETCH_SIZE", "WRITE_SIZE"):
        a = collections.defaultdict(list)
        for r in csv.DictReader(open(os.path.join(run_dir, f"pmc_ac_{ctr}", "run_counter_collection.csv"))):
            if r["Counter_Name"] == ctr:
                a[r["Kernel_Name"]].append(float(r["Counter_Value"]))
        agg[ctr] = a
    for geo, gid in (("trilinear", 2), ("stored", 1)):
        d = {}
        for ctr in ("FETCH_SIZE", "WRITE_SIZE"):
            cp = [v for k, vs in agg[ctr].items() if "copyBuffer" in k for v in vs][-3:]
            scale = copy_bytes / (sum(cp) / len(cp) * 1024.0)
            kv = [v for k, vs in agg[ctr].items() if f"force_ac_kernel<5, {gid}, false, true>" in k for v in vs]
            d[ctr] = {"kib_per_dispatch": sum(kv) / len(kv), "dispatches": len(kv),
                      "copy_kib_per_GiB": sum(cp) / len(cp), "scale": scale,
                      "bytes_per_launch": sum(kv) / len(kv) * 1024.0 * scale}
        d["bytes_per_launch"] = d["FETCH_SIZE"]["bytes_per_launch"] + d["WRITE_SIZE"]["bytes_per_launch"]
        out[geo] = d
    with open(os.path.join(ROOT, "profiles", "acoustic_traffic.json"), "w") as fh:
        json.dump(out, fh, indent=1)
    print(json.dumps({k: (v["bytes_per_launch"] if isinstance(v, dict) else v) for k, v in out.items()}))


def cpu_baseline(mesh, lam, mu, budget_s: float = 12.0):
    """FP64 oracle force apply on the first 8 element layers of the same mesh."""
    import numpy as np
    from oracle import oracle as O
    n = mesh.n
    nsub = mesh.nex * mesh.ney * 8
    ibool = mesh.ibool[:nsub]
    gam, jac, _ = O.geometry(n, mesh.elem_vert[:nsub], mesh.vert)
    u = np.random.default_rng(0).uniform(-1, 1, (mesh.nglob, 3))
    O.force(n, ibool, gam, jac, lam[:nsub], mu[:nsub], u, mesh.nglob)  # warm
    reps, t0 = 0, time.perf_counter()
    while True:
        O.force(n, ibool, gam, jac, lam[:nsub], mu[:nsub], u, mesh.nglob)
        reps += 1
        el = time.perf_counter() - t0
        if el >= budget_s or reps >= 200:
            break
    cpu = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            cpu = next((l.split(":", 1)[1].strip() for l in fh if l.startswith("model name")), cpu)
    except OSError:
        pass
    return {"value": nsub * n ** 3 * reps / el, "unit": "GLL-pt force evals/s",
            "cores": O.num_threads(), "cpu_model": cpu, "kind": "oracle",
            "sample": f"FP64 oracle force apply on the first 8 of 64 element layers "
                      f"({nsub} elements, {nsub * n ** 3} GLL points), {reps} applies in {el:.1f} s"}


def cpu_baseline_acoustic(mesh, budget_s: float = 10.0):
    """FP64 oracle acoustic force apply (numpy) on the first 2 of the 64
    element layers of the same mesh, homogeneous 1000 kg/m^3, 1500 m/s."""
    import numpy as np
    from oracle import acoustic as OA
    n = mesh.n
    nsub = mesh.nex * mesh.ney * 2
    ibool = mesh.ibool[:nsub]
    gam, jac, _ = OA.O.geometry(n, mesh.elem_vert[:nsub], mesh.vert)
    rho = np.full((nsub, n ** 3), 1000.0)
    p = np.random.default_rng(0).uniform(-1, 1, mesh.nglob)
    OA.force(n, ibool, gam, jac, rho, p, mesh.nglob)  # warm
    reps, t0 = 0, time.perf_counter()
    while True:
        OA.force(n, ibool, gam, jac, rho, p, mesh.nglob)
        reps += 1
        el = time.perf_counter() - t0
        if el >= budget_s or reps >= 100:
            break
    return {"value": nsub * n ** 3 * reps / el, "unit": "GLL-pt force evals/s", "cores": 1, "kind": "oracle",
            "sample": f"FP64 numpy acoustic oracle force apply on the first 2 of 64 element layers "
                      f"({nsub} elements, {nsub * n ** 3} GLL points), {reps} applies in {el:.1f} s"}


def adjoint_leg(ne: int = 32, nt: int = 1000, every: int = 100, fd_dirs: int = 16, fd_eps: float = 1e-4):
    """Adjoint sensitivity on the layered cube with a -5% Gaussian anomaly:
    forward with checkpoints, then the discrete adjoint; adjoint/forward time
    and a finite-difference check of the FP32 gradient along random model
    directions against central differences of FP64 forward runs (the
    library's FP64 storage mode)."""
    import numpy as np
    import torch

    import paper_2606_12850_amd as P
    import workloads as W
    from paper_2606_12850_amd.autograd import SeismogramOperator

    wl0 = W.adjoint_layered(ne=ne, n=NGLL, nt=nt, anomaly=False)
    wl = W.adjoint_layered(ne=ne, n=NGLL, nt=nt, anomaly=True)
    probe = P.Solver(NGLL)
    probe.upload_mesh(wl.mesh)
    probe.upload_model(wl.lam, wl.mu, wl.rho)
    dt = P.semx_cfl_dt(probe.ctx, 0.4)
    probe.close()
    stf = W.ricker(10.0, 0.12, dt, nt + 1)[None, :]
    op = SeismogramOperator(wl.mesh, wl.src_elem, wl.src_xi, wl.src_dir, stf, wl.rec_elem, wl.rec_xi, dt, nt,
                            checkpoint_every=every)
    data = op.run(wl0.lam, wl0.mu, wl0.rho).clone()
    op.run(wl.lam, wl.mu, wl.rho)  # warm
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    seis = op.run(wl.lam, wl.mu, wl.rho)
    torch.cuda.synchronize()
    t_fwd = time.perf_counter() - t0
    gseis = dt * (seis - data)
    chi = 0.5 * dt * float(torch.sum((seis.double() - data.double()) ** 2))
    op.gradient(gseis)  # warm
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    gl, gm, gr = op.gradient(gseis)
    torch.cuda.synchronize()
    t_adj = time.perf_counter() - t0
    op.solver.close()
    progress(f"adjoint: forward {t_fwd:.3f} s, adjoint {t_adj:.3f} s")
    # FP64 forward runs of the same discrete problem (FP64 storage)
    s64 = P.Solver(NGLL, storage=P.SEMX_F64)
    s64.upload_mesh(wl.mesh)
    s64.upload_model(wl0.lam, wl0.mu, wl0.rho)
    P.semx_set_sources_f64(s64.ctx, wl.src_elem, wl.src_xi, wl.src_dir, stf)
    P.semx_set_receivers(s64.ctx, wl.rec_elem, wl.rec_xi, nt)
    P.semx_set_dt(s64.ctx, dt)
    out64 = np.zeros((1, len(wl.rec_elem), 3, nt))

    def seis64(lam, mu, rho):
        s64.upload_model(lam, mu, rho)  # resets the run
        P.semx_step(s64.ctx, nt)
        P.semx_read_seismograms_f64(s64.ctx, out64, False)
        return out64[0].copy()

    data64 = seis64(wl0.lam, wl0.mu, wl0.rho)
    t0 = time.perf_counter()
    misfit_of = lambda lam, mu, rho: 0.5 * dt * float(np.sum((seis64(lam, mu, rho) - data64) ** 2))
    chi64 = misfit_of(wl.lam, wl.mu, wl.rho)
    t_fwd64 = time.perf_counter() - t0
    # directional derivatives: (chi(+e) - chi(-e)) / (2 e) of FP64 runs along
    # relative directions lambda xi, mu xi', rho xi'' with xi ~ N(0, 1) per point
    rng = np.random.default_rng(0)
    fd = []
    for k in range(fd_dirs):
        dl = wl.lam * rng.standard_normal(wl.lam.shape)
        dm = wl.mu * rng.standard_normal(wl.mu.shape)
        dr = wl.rho * rng.standard_normal(wl.rho.shape)
        cp = misfit_of(wl.lam + fd_eps * dl, wl.mu + fd_eps * dm, wl.rho + fd_eps * dr)
        cm = misfit_of(wl.lam - fd_eps * dl, wl.mu - fd_eps * dm, wl.rho - fd_eps * dr)
        fdv = (cp - cm) / (2 * fd_eps)
        ad = float(np.sum(gl[0].cpu().numpy() * dl) + np.sum(gm[0].cpu().numpy() * dm) + np.sum(gr[0].cpu().numpy() * dr))
        fd.append({"adjoint": ad, "fd_fp64": fdv, "rel": abs(ad - fdv) / max(abs(fdv), 1e-300)})
        progress(f"adjoint: FD direction {k + 1}/{fd_dirs}, rel {fd[-1]['rel']:.2e}")
    s64.close()
    scale = max(abs(d["fd_fp64"]) for d in fd)
    for d in fd:
        d["rel_to_largest"] = abs(d["adjoint"] - d["fd_fp64"]) / scale
    return {"workload": f"layered cube {ne}^3 regular, NGLL {NGLL}, -5% Gaussian anomaly, {nt} steps, "
                        f"checkpoint every {every}, {len(wl.rec_elem)} receivers, FP32",
            "forward_s": round(t_fwd, 4), "adjoint_s": round(t_adj, 4),
            "adjoint_over_forward": round(t_adj / t_fwd, 3), "misfit": chi, "misfit_fp64": chi64,
            "forward_fp64_s": round(t_fwd64, 4),
            "fd": f"central differences of FP64 forward runs, eps {fd_eps:g} (relative model perturbation)",
            "fd_directions": len(fd), "fd_rel_max": max(d["rel"] for d in fd),
            "fd_rel_to_largest_max": max(d["rel_to_largest"] for d in fd),
            "fd_rel_median": sorted(d["rel"] for d in fd)[len(fd) // 2], "fd_check": fd}


def surrogate_leg(f0: float = 10.0, ntrain: int = 4500, nval: int = 500, ntest: int = 4096, epochs: int = 300,
                  members: int = 4, nt: int = 800, nout: int = 512, ne: int = 16, tol: float = 0.05,
                  hidden=(512, 512, 512), batch: int = 128, dt: float | None = None, val_seed0: int | None = None):
    """Learned surrogate on the 16^3 box: batched SEM data for the 64-mode
    lambda/mu perturbations, an ensemble of MLPs trained by the library's
    kernels, the spread indicator calibrated on validation models, SEM
    fallback for flagged test models, SEM as the reference for every test model."""
    import numpy as np
    import torch

    import paper_2606_12850_amd as P
    import workloads as W
    from paper_2606_12850_amd.surrogate import BatchedSEM, Surrogate, rel_err, resample

    log = lambda m: print(f"[surrogate] {m}", file=sys.stderr, flush=True)
    mesh = W.box_mesh(ne, NGLL, 4000.0)
    basis = W.fourier_modes(mesh)
    model_fn = lambda a: W.perturbed_models(mesh, basis, a)
    # common dt: Courant 0.4 at the fastest admissible model (delta = +10 % everywhere)
    if dt is None:
        probe = P.Solver(NGLL)
        probe.upload_mesh(mesh)
        lam0, mu0, rho0 = W.homogeneous_model(mesh)
        probe.upload_model(lam0 * 1.1, mu0 * 1.1, rho0)
        dt = P.semx_cfl_dt(probe.ctx, 0.4)
        probe.close()
    se, sx = W.center_vertex_source(mesh)
    re, rx = W.top_receivers_grid(mesh, 4)
    stf = W.ricker(f0, 1.2 / f0, dt, nt + 1)[None, :]
    sem = BatchedSEM(mesh, se, sx, [[0.0, 0.0, 1.0]], stf, re, rx, dt, nt, batch=64)

    def run(coeffs):
        out = []
        for b0 in range(0, len(coeffs), 512):
            out.append(resample(sem.run_models(model_fn, coeffs[b0:b0 + 512]), nout).astype(np.float32))
        return np.concatenate(out, 0)

    A_tr = W.perturbation_coefficients(basis, range(0, ntrain))
    v0 = ntrain if val_seed0 is None else val_seed0
    A_va = W.perturbation_coefficients(basis, range(v0, v0 + nval))
    A_te = W.perturbation_coefficients(basis, range(10000, 10000 + ntest))
    t0 = time.perf_counter()
    Y_tr = run(A_tr)
    t_data = time.perf_counter() - t0
    log(f"training data {Y_tr.shape} in {t_data:.1f} s")
    Y_va = run(A_va)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    Y_te = run(A_te)
    torch.cuda.synchronize()
    t_sem = time.perf_counter() - t0
    log(f"test data (SEM for all {ntest} models) in {t_sem:.1f} s")
    n_out = Y_tr[0].size
    sur = Surrogate(64, n_out, hidden=tuple(hidden), members=members, max_batch=4096)
    t_train = sur.fit(A_tr, Y_tr, epochs=epochs, batch=batch, log=log)
    cal = sur.calibrate(A_va, Y_va.reshape(len(A_va), -1), tol=tol)
    log(f"trained in {t_train:.1f} s; calibration {cal}")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    pred, ind = sur.predict(A_te)
    flag = ind > sur.threshold
    final = pred.copy()
    if flag.any():
        final[flag] = run(A_te[flag]).reshape(int(flag.sum()), -1)
    torch.cuda.synchronize()
    t_sur = time.perf_counter() - t0
    Yt = Y_te.reshape(ntest, -1)
    e_sur, e_fin = rel_err(pred, Yt), rel_err(final, Yt)
    e_mean = rel_err(np.broadcast_to(Y_tr.reshape(ntrain, -1).mean(0), Yt.shape), Yt)
    bad = e_sur > tol
    recall = float((flag & bad).sum() / max(bad.sum(), 1))
    precision = float((flag & bad).sum() / max(flag.sum(), 1))
    sur.close(); sem.close()
    return {"workload": f"box {ne}^3 regular, NGLL {NGLL}, 64 cosine modes (lambda, mu x (1 +- 10 %)), Ricker {f0:g} Hz, "
                        f"{nt} steps -> {nout} samples, 16 receivers; MLP 64-{'-'.join(str(h) for h in hidden)}-"
                        f"{n_out} x {members}, {epochs} epochs batch {batch}; train {ntrain} / val {nval} / "
                        f"test {ntest}",
            "dt": dt, "sem_data_s": round(t_data, 2), "train_s": round(t_train, 2),
            "surrogate_err_mean": float(e_sur.mean()), "surrogate_err_median": float(np.median(e_sur)),
            "surrogate_err_max": float(e_sur.max()), "mean_seismogram_err_mean": float(e_mean.mean()),
            "frac_true_err_above_tol": float(bad.mean()), "flagged_frac": float(flag.mean()),
            "flag_recall": recall, "flag_precision": precision,
            "final_err_mean": float(e_fin.mean()), "final_err_max": float(e_fin.max()),
            "final_frac_above_tol": float((e_fin > tol).mean()),
            "time_surrogate_plus_fallback_s": round(t_sur, 3), "time_sem_all_s": round(t_sem, 3),
            "gain": round(t_sem / t_sur, 3), "calibration": cal}


def mlp_profile(steps: int = 200, infer_batches: int = 4):
    """The surrogate network's kernels alone (64 -> 512 -> 512 -> 512 -> 24,576,
    SiLU, BF16 matrix-core GEMMs with FP32 accumulation): `steps` training
    steps at batch 128 (forward, MSE, backward, Adam) on synthetic data, then
    `infer_batches` inference batches of 4096.  Time per step and achieved
    TFLOP/s on the GEMM flops (2 x multiply-adds of the three GEMMs per layer
    in training, one in inference), against the 2.5 PFLOP/s dense BF16 peak."""
    import numpy as np
    import torch

    import paper_2606_12850_amd as P
    widths = [64, 512, 512, 512, 24576]
    net = P.semx_mlp_create(widths, 4096)
    nparam = P.semx_mlp_num_params(net)
    rng = np.random.default_rng(0)
    P.semx_mlp_set_params(net, (rng.standard_normal(nparam) * 0.02).astype(np.float32))
    x = torch.randn((4096, widths[0]), device="cuda")
    t = torch.randn((128, widths[-1]), device="cuda")
    y = torch.empty((4096, widths[-1]), device="cuda")
    dy = torch.empty((128, widths[-1]), device="cuda")
    macs = sum(widths[l] * widths[l + 1] for l in range(len(widths) - 1))

    def train(k0, k):
        for i in range(k):
            P.semx_mlp_forward(net, x, 128, y)
            P.semx_mlp_mse(net, y[:128], t, 128 * widths[-1], dy, want_loss=False)
            P.semx_mlp_backward(net, dy, 128)
            P.semx_mlp_adam(net, 1e-4, 0.9, 0.999, 1e-8, k0 + i + 1)
    train(0, 10)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    train(10, steps)
    torch.cuda.synchronize()
    t_step = (time.perf_counter() - t0) / steps
    # training: forward, weight gradient and input gradient (none for layer 0)
    flops_step = 2 * 128 * (3 * macs - widths[0] * widths[1])
    P.semx_mlp_forward(net, x, 4096, y)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(infer_batches):
        P.semx_mlp_forward(net, x, 4096, y)
    torch.cuda.synchronize()
    t_inf = (time.perf_counter() - t0) / infer_batches
    P.semx_mlp_destroy(net)
    return {"widths": widths, "train_batch": 128, "train_ms_per_step": round(t_step * 1e3, 4),
            "train_tflops": round(flops_step / t_step / 1e12, 3),
            "infer_batch": 4096, "infer_ms": round(t_inf * 1e3, 4),
            "infer_tflops": round(2 * 4096 * macs / t_inf / 1e12, 3), "peak_tflops_bf16": 2500.0}


ORDER_SWEEP = [(4, 90), (5, 68), (6, 54), (7, 45), (8, 39), (9, 34), (10, 30), (11, 27), (12, 25), (13, 23),
               (14, 21), (15, 19), (16, 18)]  # (NGLL, elements per side): ~2e7 points


def order_sweep_leg(reps: int = 20, orders=None):
    """Force apply at about 2e7 unique points for NGLL 4..16 (element size
    h = N * 69.3 / 5 m, about five GLL points per minimum wavelength of a
    25 Hz wave at vs = 1732 m/s), homogeneous medium times a +-5 % random
    field, regular hexahedra, coloured assembly: FP32, and BF16 / FP16 matrix
    core contractions where supported, with the relative force difference of
    the mixed paths against FP32 on a smooth field."""
    import numpy as np
    import torch

    import paper_2606_12850_amd as P
    import workloads as W

    log = lambda m: print(f"[order-sweep] {m}", file=sys.stderr, flush=True)
    rows = []
    for n, ne in ORDER_SWEEP:
        if orders is not None and n not in orders:
            continue
        N = n - 1
        h = N * 69.3 / 5
        mesh = W.box_mesh(ne, n, ne * h)
        lam, mu, rho = W.layered_model(mesh, vp_layers=(3000.0,), vpvs=3000.0 / 1732.0, grf_amp=0.05,
                                       grf_seed=12850, grf_corr_elems=4.0)
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        s = P.Solver(n)
        s.upload_mesh(mesh)
        s.upload_model(lam, mu, rho)
        torch.cuda.synchronize()
        device_bytes = free0 - torch.cuda.mem_get_info()[0]  # the library's own allocations
        vp_max = float(np.sqrt((lam + 2.0 * mu) / rho).max())
        del lam, mu, rho
        G = mesh.nglob
        Gx = ne * N + 1
        g = np.arange(G)
        xs = (g % Gx, (g // Gx) % Gx, g // (Gx * Gx))
        k = 2.0 * np.pi / (Gx - 1)
        u_np = np.stack([np.sin(k * xs[0] + 0.3) * np.cos(k * xs[1]), np.cos(k * xs[1] + 0.7) * np.sin(k * xs[2]),
                         np.sin(k * xs[2] + 1.1) * np.cos(k * xs[0])], axis=1).astype(np.float32)
        u = torch.from_numpy(u_np).to("cuda")
        del u_np, xs, g
        f = torch.empty_like(u)
        row = {"ngll": n, "ne": ne, "nspec": mesh.nspec, "nglob": G, "h_m": round(h, 2), "device_bytes": device_bytes}
        b_model = bytes_per_element_model(n, G, mesh.nspec, "regular")
        b_elem = bytes_per_element(n, G, mesh.nspec, "regular", affine=n <= 10 or n == 16)
        # full explicit step (FP32, coloured) from a nonzero state, CFL time step
        dt = P.semx_cfl_dt(s.ctx, 0.4)
        P.semx_set_dt(s.ctx, dt)
        P.semx_set_state(s.ctx, u, torch.zeros_like(u), torch.zeros_like(u), 0)
        s.step(3)
        e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
        e0.record(s.stream)
        s.step(reps)
        e1.record(s.stream)
        e1.synchronize()
        row["step_ms"] = round(e0.elapsed_time(e1) / reps, 4)
        row["dt_cfl"] = dt
        row["hmin_over_h"] = dt * vp_max / 0.4 / h  # smallest GLL spacing over the element size
        # contraction modes: FP32 everywhere; the matrix-core modes where they
        # exist (NGLL 4..8 and 11..16; from 13 the FP32 path is the
        # FP32-operand matrix-core kernel itself, so mf32 is not listed
        # there).  Timed in interleaved rounds (median), so that clock state
        # favours no mode.
        modes = [(c, m) for c, m in (("f32", P.SEMX_C_F32), ("mf32", P.SEMX_C_MFMA_F32), ("bf16", P.SEMX_C_BF16),
                                     ("f16", P.SEMX_C_F16))
                 if c == "f32" or (4 <= n <= 8) or (11 <= n <= 16 and not (n >= 13 and c == "mf32"))]
        ref = None
        for cname, cmode in modes:
            P.semx_set_mode(s.ctx, cmode, P.SEMX_ASM_COLORED)
            for _ in range(3):
                P.semx_apply_force(s.ctx, u, f)
            if ref is None:
                ref = f.clone()
            else:
                row[f"{cname}_rel_diff_vs_f32"] = (torch.linalg.norm(f - ref) / torch.linalg.norm(ref)).item()
        times = {c: [] for c, _ in modes}
        for _ in range(3):
            for cname, cmode in modes:
                P.semx_set_mode(s.ctx, cmode, P.SEMX_ASM_COLORED)
                P.semx_apply_force(s.ctx, u, f)
                e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
                e0.record(s.stream)
                for _ in range(reps):
                    P.semx_apply_force(s.ctx, u, f)
                e1.record(s.stream)
                e1.synchronize()
                times[cname].append(e0.elapsed_time(e1) / reps)
        for cname, _ in modes:
            ms = float(np.median(times[cname]))
            row[f"{cname}_ms"] = round(ms, 4)
            row[f"{cname}_gll_pts_per_s"] = mesh.nspec * n ** 3 / (ms * 1e-3)
            row[f"{cname}_hbm_frac"] = round(b_model * mesh.nspec / (ms * 1e-3) / (HBM_PEAK_GBS * 1e9), 4)
            row[f"{cname}_hbm_frac_impl"] = round(b_elem * mesh.nspec / (ms * 1e-3) / (HBM_PEAK_GBS * 1e9), 4)
            if cname != "f32":
                row[f"{cname}_speedup_vs_f32"] = round(row["f32_ms"] / ms, 3)
        P.semx_set_mode(s.ctx, P.SEMX_C_F32, P.SEMX_ASM_COLORED)
        del u, f, ref
        s.close()
        if n in (5, 8, 16):  # the acoustic experiment's orders: the scalar operator on the same mesh
            torch.cuda.synchronize()
            free0 = torch.cuda.mem_get_info()[0]
            sa = P.Solver(n, physics=P.SEMX_ACOUSTIC)
            sa.upload_mesh(mesh)
            shp = (mesh.nspec, n ** 3)
            sa.upload_model_acoustic(np.full(shp, 1000.0 * 1500.0 ** 2), np.full(shp, 1000.0))
            torch.cuda.synchronize()
            row["acoustic_device_bytes"] = free0 - torch.cuda.mem_get_info()[0]
            pa = torch.rand(G, device="cuda") - 0.5
            fa = torch.empty_like(pa)
            P.semx_set_dt(sa.ctx, P.semx_cfl_dt(sa.ctx, 0.4))
            P.semx_set_state(sa.ctx, pa, torch.zeros_like(pa), torch.zeros_like(pa), 0)
            sa.step(3)
            e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
            e0.record(sa.stream)
            sa.step(reps)
            e1.record(sa.stream)
            e1.synchronize()
            row["acoustic_step_ms"] = round(e0.elapsed_time(e1) / reps, 4)
            for _ in range(3):
                P.semx_apply_force(sa.ctx, pa, fa)
            e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
            e0.record(sa.stream)
            for _ in range(reps):
                P.semx_apply_force(sa.ctx, pa, fa)
            e1.record(sa.stream)
            e1.synchronize()
            ms = e0.elapsed_time(e1) / reps
            ba = bytes_per_element_acoustic(n, G, mesh.nspec, "regular")
            row["acoustic_ms"] = round(ms, 4)
            row["acoustic_gll_pts_per_s"] = mesh.nspec * n ** 3 / (ms * 1e-3)
            row["acoustic_hbm_frac_alg"] = round(ba * mesh.nspec / (ms * 1e-3) / (HBM_PEAK_GBS * 1e9), 4)
            del pa, fa
            sa.close()
        log(json.dumps(row))
        rows.append(row)
    return rows


def launches_of_apply(s, u, f) -> int:
    """Launches of one force apply as the library counts them."""
    import paper_2606_12850_amd as P
    P.semx_set_timing(s.ctx, 1)
    P.semx_apply_force(s.ctx, u, f)
    n, _ = P.semx_force_timing(s.ctx)
    P.semx_set_timing(s.ctx, 0)
    return n


def single_order_apply(n: int, reps: int, mode: str = "f32"):
    """Coloured force applies (contraction `mode`: f32, bf16, f16) on the
    order-sweep mesh of one NGLL (regular hexahedra, about 2e7 unique
    points), event-timed, then three 1 GiB device copies that calibrate
    traffic counters; for profiling."""
    import numpy as np
    import torch

    import paper_2606_12850_amd as P
    import workloads as W
    ne = dict(ORDER_SWEEP)[n]
    h = (n - 1) * 69.3 / 5
    mesh = W.box_mesh(ne, n, ne * h)
    lam, mu, rho = W.homogeneous_model(mesh)
    s = P.Solver(n)
    s.upload_mesh(mesh)
    s.upload_model(lam, mu, rho)
    del lam, mu, rho
    s.set_mode({"f32": P.SEMX_C_F32, "bf16": P.SEMX_C_BF16, "f16": P.SEMX_C_F16}[mode], P.SEMX_ASM_COLORED)
    u = torch.rand((mesh.nglob, 3), device="cuda", generator=torch.Generator("cuda").manual_seed(0)) - 0.5
    f = torch.empty_like(u)
    for _ in range(3):
        P.semx_apply_force(s.ctx, u, f)
    e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
    e0.record(s.stream)
    for _ in range(reps):
        P.semx_apply_force(s.ctx, u, f)
    e1.record(s.stream)
    e1.synchronize()
    ms = e0.elapsed_time(e1) / reps
    launches = launches_of_apply(s, u, f)
    s.set_mode(P.SEMX_C_F32, P.SEMX_ASM_COLORED)
    sk = P.semx_force_skeleton(s.ctx, u, f, reps)  # the memory skeleton of the FP32 pass
    s.close()
    nbytes = 1 << 30
    a = torch.ones(nbytes // 4, device="cuda")
    b = torch.empty_like(a)
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()
    bm = bytes_per_element_model(n, mesh.nglob, mesh.nspec, "regular")
    be = bytes_per_element(n, mesh.nglob, mesh.nspec, "regular", affine=n <= 10 or n == 16)
    return {"ngll": n, "mode": mode, "ne": ne, "nspec": mesh.nspec, "nglob": mesh.nglob, "ms_per_apply": round(ms, 4),
            "launches_per_apply": launches, "bytes_per_element": bm, "bytes_per_element_impl": be,
            "hbm_frac": round(bm * mesh.nspec / (ms * 1e-3) / (HBM_PEAK_GBS * 1e9), 4),
            "hbm_frac_impl": round(be * mesh.nspec / (ms * 1e-3) / (HBM_PEAK_GBS * 1e9), 4),
            "skeleton_ms_per_apply": round(sk, 4), "frac_of_skeleton": round(sk / ms, 4),
            "copy_bytes_each_way": nbytes}


def iso_accuracy_summary(rows, eps: float = 1e-5):
    """Equal-accuracy comparison across orders (the paper's dispersion-based
    (h, p) frontier, Sec. IV-B and V-C): with ppw_p the GLL points per
    wavelength at which an axis plane wave has relative phase-velocity error
    eps (tests/golden/iso_accuracy.json, from the oracle's Bloch analysis),
    a volume of one minimum wavelength cubed holds ppw_p^3 unique nodes.
    The per-node costs come from the order sweep (about 2e7 nodes per order,
    where every order fills the GPU): FP32 step time and device bytes per
    node, and the CFL time step through the smallest GLL spacing.  Reported
    per lambda^3 and relative to NGLL 5 (p = 4)."""
    with open(os.path.join(ROOT, "tests", "golden", "iso_accuracy.json")) as fh:
        tab = json.load(fh)
    ppw_of = dict(zip(tab["ngll"], tab["ppw"][tab["eps"].index(eps)]))
    out = []
    for r in rows:
        n = r["ngll"]
        if n not in ppw_of or "step_ms" not in r:
            continue
        ppw = ppw_of[n]
        nodes = ppw ** 3
        step_ns = r["step_ms"] * 1e6 / r["nglob"] * nodes      # ns per step per lambda^3
        apply_ns = r["f32_ms"] * 1e6 / r["nglob"] * nodes
        mem = r["device_bytes"] / r["nglob"] * nodes
        dt_rel = r["hmin_over_h"] * (n - 1) / ppw              # CFL dt in units of lambda / vp
        out.append({"ngll": n, "p": n - 1, "ppw": ppw, "h_over_lambda": round((n - 1) / ppw, 4),
                    "nodes_per_lambda3": round(nodes, 1), "step_ns_per_lambda3": round(step_ns, 3),
                    "apply_ns_per_lambda3": round(apply_ns, 3), "device_bytes_per_lambda3": round(mem, 1),
                    "cfl_dt_lambda_over_vp": round(dt_rel, 5),
                    "time_to_solution_cfl": step_ns / dt_rel})
    base = next((o for o in out if o["ngll"] == 5), None)
    if base:
        for o in out:
            o["rel_step_cost_fixed_dt"] = round(o["step_ns_per_lambda3"] / base["step_ns_per_lambda3"], 4)
            o["rel_time_cfl_dt"] = round(o["time_to_solution_cfl"] / base["time_to_solution_cfl"], 4)
            o["rel_memory"] = round(o["device_bytes_per_lambda3"] / base["device_bytes_per_lambda3"], 4)
    return {"eps": eps, "rows": out}


def bytes_per_element_acoustic(n: int, nglob: int, nspec: int, geometry: str = "trilinear") -> float:
    """Algorithmic HBM bytes per element per apply of the scalar (acoustic)
    force: ibool 4 n^3, geometry as for the elastic operator, W / rho 4 n^3,
    p read once and f written once per unique node (4 G/E each)."""
    n3 = n ** 3
    geo = {"stored": 36 * n3, "trilinear": 96, "regular": 36}[geometry]
    return 4 * n3 + geo + 4 * n3 + 2 * 4.0 * nglob / nspec


def acoustic_traffic(geometry: str):
    """HBM bytes per launch of the acoustic force kernel from rocprofv3 PMC
    counters (profiles/acoustic_traffic.json), if they were taken on the
    current kernel source; else None."""
    p = os.path.join(ROOT, "profiles", "acoustic_traffic.json")
    if not os.path.exists(p):
        return None
    try:
        d = json.load(open(p))
    except Exception:
        return None
    src = b"".join(open(os.path.join(ROOT, "paper_2606_12850_amd", "csrc", f), "rb").read()
                   for f in ("acoustic.hip", "elem_common.hpp"))
    if d.get("kernel_source_sha256") != hashlib.sha256(src).hexdigest():
        return None
    return d.get(geometry, {}).get("bytes_per_launch")


def acoustic_leg(mesh, reps: int = 50, rods: bool = True):
    """The scalar (acoustic) operator.  (1) Force apply on the bench mesh
    (homogeneous 1000 kg/m^3, 1500 m/s), coloured, trilinear and stored
    geometry, event-timed on the library stream: GLL-pt/s and the fraction of
    8 TB/s for its own byte model.  (2) The paper's equal-accuracy runs
    (Sec. V-C): a 20 Hz Ricker plane source on the end of a rod, the trace at
    12 km (8 s of travel), dt = 1e-4 s, at each degree's equal-accuracy
    element size (tests/golden/acoustic_iso.json): the library's waveform
    error against the closed form p = rho c S(t - x/c), S(tau) = (tau - t0)
    exp(-(pi f0 (tau - t0))^2), and the run's wall time."""
    import numpy as np
    import torch

    import paper_2606_12850_amd as P
    import workloads as W

    rho, vp, f0 = 1000.0, 1500.0, 20.0
    out = {"force_apply": {}}
    s = P.Solver(mesh.n, physics=P.SEMX_ACOUSTIC)
    info = s.upload_mesh(mesh)
    shape = (mesh.nspec, mesh.n ** 3)
    s.upload_model_acoustic(np.full(shape, rho * vp * vp), np.full(shape, rho))
    p = torch.rand(mesh.nglob, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) - 0.5
    f = torch.empty_like(p)
    for gname, gmode in (("trilinear", P.SEMX_GEOM_TRILINEAR), ("stored", P.SEMX_GEOM_STORED)):
        P.semx_set_geometry(s.ctx, gmode)
        for _ in range(5):
            P.semx_apply_force(s.ctx, p, f)
        e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
        e0.record(s.stream)
        for _ in range(reps):
            P.semx_apply_force(s.ctx, p, f)
        e1.record(s.stream)
        e1.synchronize()
        ms = e0.elapsed_time(e1) / reps
        geo = gname if info["nirregular"] > 0 else "regular"
        b = bytes_per_element_acoustic(mesh.n, mesh.nglob, mesh.nspec, geo)
        out["force_apply"][f"acoustic_{gname}_colored"] = {
            "ms_per_apply": round(ms, 4), "gll_pts_per_s": mesh.nspec * mesh.n ** 3 / (ms * 1e-3),
            "bytes_per_element": b, "hbm_frac_alg": round(b * mesh.nspec / (ms * 1e-3) / (HBM_PEAK_GBS * 1e9), 4),
            "traffic": acoustic_traffic(gname)}
    s.close()
    del p, f
    progress("acoustic force apply done")
    if not rods:
        return out

    with open(os.path.join(ROOT, "tests", "golden", "acoustic_iso.json")) as fh:
        tab = json.load(fh)
    x_rec = tab["x_rec"]
    t0 = 1.2 / f0
    t_end = x_rec / vp + t0 + 1.2 / f0 + 1.0 / f0
    runs = []
    for key, o in sorted(tab["orders"].items(), key=lambda kv: int(kv[0])):
        n, h = int(key), o["h_max"]
        xi, w = P.semx_gll(n)
        rod = W.acoustic_rod(n, h, x_rec, t_end, xi, w, dt=tab["dt"], c=vp, f0=f0)
        s = P.Solver(n, physics=P.SEMX_ACOUSTIC)
        s.upload_mesh(rod.mesh)
        shp = (rod.mesh.nspec, n ** 3)
        s.upload_model_acoustic(np.full(shp, rho * vp * vp), np.full(shp, rho))
        P.semx_set_sources(s.ctx, rod.src_elem, rod.src_xi, None, rod.stf.astype(np.float32))
        P.semx_set_receivers(s.ctx, rod.rec_elem, rod.rec_xi, rod.nt)
        s.nrec, s.nt_max = 1, rod.nt
        P.semx_set_dt(s.ctx, rod.dt)
        # a few hundred elements: the step is bound by kernel launches, which
        # graph-captured chunks cut at NGLL 5 and 8 (not at 16, where the
        # element kernels dominate)
        chunk = 256 if n <= 10 else 0
        P.semx_set_graphs(s.ctx, chunk)
        P.semx_reset(s.ctx)
        torch.cuda.synchronize()
        w0 = time.perf_counter()
        s.step(rod.nt)
        torch.cuda.synchronize()
        wall = time.perf_counter() - w0
        tr = s.seismograms()[0, 0].astype(np.float64)
        s.close()
        t = (np.arange(rod.nt) + 1) * rod.dt
        tau = t - x_rec / vp - t0
        ref = rho * vp * tau * np.exp(-(np.pi * f0 * tau) ** 2)
        err = float(np.sum((tr - ref) ** 2) / np.sum(ref ** 2))
        runs.append({"p": n - 1, "ngll": n, "h_m": round(h, 3), "steps": rod.nt, "nspec": rod.mesh.nspec,
                     "error_ratio": err, "rel_l2_error_pct": round(100 * np.sqrt(err), 4),
                     "oracle_rel_l2_error_pct": round(100 * np.sqrt(o["error_at_h_max"]), 4),
                     "wall_s": round(wall, 2), "us_per_step": round(wall / rod.nt * 1e6, 2),
                     "graph_chunk": chunk})
        progress(f"acoustic rod p={n - 1} h={h:.2f}: error {100 * np.sqrt(err):.4f} % in {wall:.1f} s")
    out["equal_accuracy_rod"] = {"x_rec_m": x_rec, "dt": tab["dt"], "bound_rel_l2_pct": 1.0, "runs": runs,
                                 "paper_h_m": {"4": 20.0, "7": 50.0, "15": 130.0}}
    return out


def acoustic_frontier_summary(rows):
    """The paper's cost comparison on its equal-accuracy frontier (Sec. V-C):
    element sizes h_p from the acoustic rod experiment
    (tests/golden/acoustic_iso.json), elastic FP32 costs per element from the
    order sweep (step time and device bytes at about 2e7 nodes, where each
    order fills the GPU), a fixed domain and the same dt for every order, so
    time to solution and memory scale as cost per element / h_p^3.  The
    acoustic operator's own ratios (same meshes, NGLL 5, 8, 16) come with
    them."""
    with open(os.path.join(ROOT, "tests", "golden", "acoustic_iso.json")) as fh:
        tab = json.load(fh)
    by_n = {r["ngll"]: r for r in rows if "step_ms" in r}
    per = {}
    for key, o in tab["orders"].items():
        n = int(key)
        if n not in by_n:
            continue
        r = by_n[n]
        h = o["h_max"]
        per[n - 1] = {"h_m": round(h, 3), "step_s_per_km3": r["step_ms"] * 1e-3 / r["nspec"] * 1e9 / h ** 3,
                      "device_bytes_per_km3": r["device_bytes"] / r["nspec"] * 1e9 / h ** 3}
        if "acoustic_step_ms" in r:
            per[n - 1]["acoustic_step_s_per_km3"] = r["acoustic_step_ms"] * 1e-3 / r["nspec"] * 1e9 / h ** 3
            per[n - 1]["acoustic_device_bytes_per_km3"] = r["acoustic_device_bytes"] / r["nspec"] * 1e9 / h ** 3
    pairs = []
    for a, b, paper_t, paper_m in ((4, 7, 3.85, 3.18), (7, 15, 1.4, 1.8)):
        if a in per and b in per:
            pr = {"from_p": a, "to_p": b,
                  "time_ratio": round(per[a]["step_s_per_km3"] / per[b]["step_s_per_km3"], 3),
                  "memory_ratio": round(per[a]["device_bytes_per_km3"] / per[b]["device_bytes_per_km3"], 3),
                  "paper_time_ratio": paper_t, "paper_memory_ratio": paper_m}
            if "acoustic_step_s_per_km3" in per[a] and "acoustic_step_s_per_km3" in per[b]:
                pr["acoustic_time_ratio"] = round(per[a]["acoustic_step_s_per_km3"] / per[b]["acoustic_step_s_per_km3"], 3)
                pr["acoustic_memory_ratio"] = round(per[a]["acoustic_device_bytes_per_km3"]
                                                    / per[b]["acoustic_device_bytes_per_km3"], 3)
            pairs.append(pr)
    return {"per_order": per, "pairs": pairs}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2000)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-adjoint", action="store_true")
    ap.add_argument("--no-acoustic", action="store_true")
    ap.add_argument("--sweep-order", type=int, default=0,
                    help="time only the force apply (--sweep-mode) on the order-sweep mesh of this NGLL, then a 1 GiB "
                         "device copy (for counter runs); prints one JSON line")
    ap.add_argument("--acoustic-only", action="store_true",
                    help="time only the acoustic force apply on the bench mesh (no time loop, no rod runs); "
                         "prints one JSON line")
    ap.add_argument("--geometry", choices=["stored", "trilinear"], default="trilinear")
    ap.add_argument("--assembly", choices=["colored", "atomic"], default="colored")
    ap.add_argument("--apply-reps", type=int, default=50)
    ap.add_argument("--sweep-mode", choices=("f32", "bf16", "f16"), default="f32",
                    help="contraction mode of --sweep-order")
    ap.add_argument("--profile-force", action="store_true",
                    help="time only the force apply of --contraction/--geometry/--assembly, then a 1 GiB "
                         "device copy (calibration for HBM traffic counters); prints one JSON line")
    ap.add_argument("--contraction", choices=["f32", "mf32", "bf16", "f16"], default="f32")
    ap.add_argument("--profile-mlp", action="store_true",
                    help="time only the surrogate network's training and inference kernels (for counter runs)")
    ap.add_argument("--surrogate", action="store_true",
                    help="run the learned-surrogate leg at its full model counts (several minutes)")
    ap.add_argument("--surrogate-f0", type=float, default=10.0)
    ap.add_argument("--surrogate-scale", type=float, default=1.0,
                    help="fraction of the surrogate leg's model counts and epochs (quick checks)")
    ap.add_argument("--no-order-sweep", action="store_true",
                    help="skip the order sweep (NGLL 4..9 at ~2e7 points, FP32 and mixed)")
    ap.add_argument("--order-sweep-full", action="store_true",
                    help="extend the order sweep to NGLL 16 (the column kernels) with the equal-accuracy summaries")
    ap.add_argument("--no-surrogate", action="store_true",
                    help="skip the bounded surrogate leg (16^3 box at 10 Hz, reduced model counts)")
    ap.add_argument("--write-traffic", metavar="DIR",
                    help="no GPU: read the two rocprofv3 --pmc runs of --profile-force (DIR/pmc_<geometry>_"
                         "<counter>/run_counter_collection.csv) and write profiles/force_traffic.json")
    ap.add_argument("--write-acoustic-traffic", metavar="DIR",
                    help="no GPU: read the two rocprofv3 --pmc runs of --acoustic-only (DIR/pmc_ac_<counter>/"
                         "run_counter_collection.csv) and write profiles/acoustic_traffic.json")
    args = ap.parse_args()
    if args.write_traffic:
        write_traffic(args.write_traffic)
        return
    if args.write_acoustic_traffic:
        write_acoustic_traffic(args.write_acoustic_traffic)
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}): the library has no "
              "multi-GPU path; the operator would shard by mesh blocks with a halo exchange.",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2606_12850_amd as P
    import workloads as W

    GEOM = {"stored": P.SEMX_GEOM_STORED, "trilinear": P.SEMX_GEOM_TRILINEAR}
    CONTRACTION = {"f32": P.SEMX_C_F32, "mf32": P.SEMX_C_MFMA_F32, "bf16": P.SEMX_C_BF16, "f16": P.SEMX_C_F16}
    ASSEMBLY = {"colored": P.SEMX_ASM_COLORED, "atomic": P.SEMX_ASM_ATOMIC}
    torch.cuda.set_device(0)
    if args.profile_mlp:
        print(json.dumps({"mlp": mlp_profile()}))
        return
    if args.sweep_order:
        print(json.dumps({"sweep_order": single_order_apply(args.sweep_order, args.apply_reps, args.sweep_mode)}))
        return
    t_setup = time.perf_counter()
    nt_total = args.warmup + args.steps
    wl = W.layered_jittered(ne=NE, n=NGLL, nt=nt_total, dt=1.0, jitter=0.10, seed=2606,
                            grf_seed=12850, grf_amp=0.05, nrec=8)
    mesh = wl.mesh
    if args.acoustic_only:
        ac = acoustic_leg(mesh, reps=args.apply_reps, rods=False)
        # calibration for the traffic counters: a plain device copy of known size
        nbytes = 1 << 30
        a = torch.ones(nbytes // 4, device="cuda")
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"acoustic": ac, "nspec": mesh.nspec, "nglob": mesh.nglob, "copy_bytes_each_way": nbytes}))
        return
    s = P.Solver(NGLL)
    info = s.upload_mesh(mesh)
    s.upload_model(wl.lam, wl.mu, wl.rho)
    asm = P.SEMX_ASM_COLORED if args.assembly == "colored" else P.SEMX_ASM_ATOMIC
    s.set_mode(P.SEMX_C_F32, asm)
    dt = P.semx_cfl_dt(s.ctx, 0.4)
    wl.dt = dt
    wl.stf = W.ricker(10.0, 0.12, dt, nt_total + 1)[None, :]
    s.setup_run(wl)
    setup_s = time.perf_counter() - t_setup
    stream = s.stream
    E, n3 = mesh.nspec, NGLL ** 3
    geo_of = (lambda g: g if info["nirregular"] > 0 else "regular")
    # the roofline's byte model (per-point inverse Jacobian) and what this path reads
    b_model = bytes_per_element_model(NGLL, mesh.nglob, E, geo_of(args.geometry))
    b_elem = bytes_per_element(NGLL, mesh.nglob, E, geo_of(args.geometry), affine=True)

    # ---- force apply alone (FP32 and mixed contractions, coloured and atomic):
    #      median over `apply_reps` applies after 10 warm-ups, each apply
    #      bracketed by an event pair on the library stream; the mixed modes
    #      carry their relative L2 difference from the FP32 force on a random
    #      and on a smooth displacement
    u = (torch.rand((mesh.nglob, 3), device="cuda", generator=torch.Generator("cuda").manual_seed(0)) - 0.5)
    f = torch.empty_like(u)
    g_idx = torch.arange(mesh.nglob, device="cuda", dtype=torch.float64)
    Gx = mesh.nex * (NGLL - 1) + 1
    kx = 2.0 * np.pi / (Gx - 1)
    xs = (g_idx % Gx, (g_idx // Gx) % Gx, g_idx // (Gx * Gx))
    u_smooth = torch.stack([torch.sin(kx * xs[0] + 0.3) * torch.cos(kx * xs[1]),
                            torch.cos(kx * xs[1] + 0.7) * torch.sin(kx * xs[2]),
                            torch.sin(kx * xs[2] + 1.1) * torch.cos(kx * xs[0])], dim=1).float().contiguous()
    del g_idx, xs
    combos = [(c, g, a) for c in ("f32", "mf32", "bf16", "f16") for g in ("stored", "trilinear")
              for a in ("colored", "atomic") if c == "f32" or a == "colored"]
    if args.profile_force:
        combos = [(args.contraction, args.geometry, args.assembly)]
    apply = {}
    ref_f32 = {}
    for cname, gname, aname in combos:
        P.semx_set_geometry(s.ctx, GEOM[gname])
        P.semx_set_mode(s.ctx, CONTRACTION[cname], ASSEMBLY[aname])
        bm = bytes_per_element_model(NGLL, mesh.nglob, E, geo_of(gname))
        bg = bytes_per_element(NGLL, mesh.nglob, E, geo_of(gname),
                               affine=cname == "f32")
        for _ in range(10):
            P.semx_apply_force(s.ctx, u, f)
        ts = []
        for _ in range(args.apply_reps):
            e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            P.semx_apply_force(s.ctx, u, f)
            e1.record(stream)
            e1.synchronize()
            ts.append(e0.elapsed_time(e1))
        ms = float(np.median(ts))
        row = {"ms_per_apply": round(ms, 4), "ms_min": round(float(np.min(ts)), 4),
               "gll_pts_per_s": E * n3 / (ms * 1e-3),
               "hbm_frac": round((bm * E / (ms * 1e-3)) / (HBM_PEAK_GBS * 1e9), 4),
               "bytes_per_element_impl": bg,
               "hbm_frac_impl": round((bg * E / (ms * 1e-3)) / (HBM_PEAK_GBS * 1e9), 4)}
        if not args.profile_force:
            outs = []
            for uu in (u, u_smooth):
                P.semx_apply_force(s.ctx, uu, f)
                outs.append(f.clone())
            if cname == "f32" and aname == "colored":
                ref_f32[gname] = outs
            elif gname in ref_f32:
                for lab, a_, b_ in zip(("random", "smooth"), outs, ref_f32[gname]):
                    row[f"rel_diff_vs_f32_{lab}"] = (torch.linalg.norm(a_ - b_) / torch.linalg.norm(b_)).item()
        apply[f"{cname}_{gname}_{aname}"] = row
    del u_smooth
    fa = apply.get(f"f32_{args.geometry}_{args.assembly}")
    for cname in ("bf16", "f16", "mf32"):
        mx = apply.get(f"{cname}_{args.geometry}_colored")
        if fa and mx:
            mx["speedup_vs_f32"] = round(fa["ms_per_apply"] / mx["ms_per_apply"], 3)
    progress(f"force-apply matrix done ({len(apply)} variants)")
    if args.profile_force:
        sk = None
        if args.contraction == "f32" and args.assembly == "colored":
            # the force pass's memory skeleton, for the same counters
            sk = round(P.semx_force_skeleton(s.ctx, u, f, args.apply_reps), 4)
        # calibration for the traffic counters: a plain device copy of known size
        nbytes = 1 << 30
        a = torch.ones(nbytes // 4, device="cuda")
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"profile_force": apply, "skeleton_ms_per_apply": sk, "elements": E,
                          "copy_bytes_each_way": nbytes,
                          "force_launches_per_apply": launches_of_apply(s, u, f)}))
        s.close()
        return
    P.semx_set_mode(s.ctx, P.SEMX_C_F32, asm)
    P.semx_set_geometry(s.ctx, GEOM[args.geometry])

    # ---- time loop: warmup, then exactly `steps` timed steps.  The force
    # kernel's launch duration is measured over the same region: one HIP
    # event pair around the force pass of every second step, divided by its
    # launches (element-local forces run it as one launch, its nodal sum inside
    # the Newmark pass).  An event pair around every launch would add the
    # event-to-kernel latency to each duration and slow the step itself by about
    # 9 %.
    stride = 2
    P.semx_reset(s.ctx)
    s.step(args.warmup)
    torch.cuda.synchronize()
    P.semx_set_timing(s.ctx, stride)
    P.semx_force_timing(s.ctx)  # clear
    e0 = torch.cuda.Event(enable_timing=True); e1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    w0 = time.perf_counter()
    e0.record(stream)
    s.step(args.steps)
    e1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - w0
    launches, force_ms = P.semx_force_timing(s.ctx)
    P.semx_set_timing(s.ctx, 0)
    step_ms = e0.elapsed_time(e1) / args.steps
    progress(f"time loop: {args.steps} steps, {step_ms:.4f} ms per step")
    seis = s.seismograms()
    assert np.all(np.isfinite(seis)), "non-finite seismograms"

    # ---- streaming reference: the library's own 1 GiB copy kernel (read + write)
    bw_copy = P.semx_stream_bandwidth(s.ctx, 1 << 30, 20)

    # ---- roofline of the force kernel (per launch)
    launches_per_apply = launches / ((args.steps + stride - 1) // stride)
    avg_launch_ms = force_ms / launches

    # ---- access-pattern reference: the memory skeleton of a force apply (same
    # launches, grid, loads and stores, no arithmetic; element launches and
    # nodal sum) on scratch fields, against the apply's own time
    skeleton = None
    if args.assembly == "colored":
        uu = torch.zeros((mesh.nglob, 3), device="cuda")
        ff = torch.zeros_like(uu)
        sk_ms = P.semx_force_skeleton(s.ctx, uu, ff, 20)
        del uu, ff
        skeleton = {"skeleton_ms_per_apply": round(sk_ms, 5)}
        if fa:
            skeleton["frac_of_skeleton"] = round(sk_ms / fa["ms_per_apply"], 4)
    # element-local forces: one launch a pass (this box is all of one kind)
    parts = args.assembly == "colored" and launches_per_apply == 1
    b_pass = (bytes_per_element_pass(NGLL, mesh.nglob, E, geo_of(args.geometry), affine=True) if parts else b_elem)
    bytes_per_launch = b_pass * E / launches_per_apply
    achieved = bytes_per_launch / (avg_launch_ms * 1e-3) / 1e9
    achieved_model = b_model * E / launches_per_apply / (avg_launch_ms * 1e-3) / 1e9
    src_hash = kernel_source_hash()
    traffic = traffic_from_profiles(src_hash, args.geometry)
    if skeleton is not None:
        skeleton["skeleton_traffic"] = traffic_from_profiles(src_hash, args.geometry + "_skeleton")

    out = {
        "metric": "GLL-point force evals/s (FP32 vs mixed) + % HBM roofline; adjoint/fwd time",
        "value": E * n3 / (step_ms * 1e-3),
        "unit": "GLL-pt force evals/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(step_ms, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "layered elastic cube 64^3 hex, NGLL 5, jittered +-10% h, 3 layers + 5% GRF, "
                               f"Ricker 10 Hz, Courant 0.4, {args.assembly} assembly, FP32",
                   "nspec": E, "nglob": mesh.nglob, "ngll": NGLL, "dt": dt,
                   "assembly": args.assembly, "contraction": "f32",
                   "nregular": info["nregular"], "nirregular": info["nirregular"], "ncolors": info["ncolors"]},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                     "kernel": f"FP32 force pass, NGLL 5, {args.geometry}, {args.assembly}"
                               + (" (one launch of element-local forces on a box, the nodal sum in the Newmark pass)"
                                  if args.assembly == "colored" and args.geometry == "trilinear" else ""),
                     "note": "achieved and frac price the timed launch at the bytes that it cannot do without (inputs "
                             "and forces once); achieved_model prices it at the byte model, whose Gamma and det J per "
                             "point the trilinear path does not move; the skeleton is that of an apply, nodal sum "
                             "included, and is compared with an apply",
                     "bytes_per_element": b_pass, "bytes_per_launch": bytes_per_launch,
                     "avg_launch_ms": round(avg_launch_ms, 5), "launches": launches, "timed_pass_stride": stride,
                     "bytes_model": "4 n^3 + 10 s n^3 + 2 s n^3 + 6 s G/E (node numbers, Gamma and det J per "
                                    "point, lambda and mu, u read and f written once per unique node; s = 4)",
                     "bytes_per_element_model": b_model, "achieved_model": round(achieved_model, 1),
                     "launch_ms_for_frac_0.6": round(bytes_per_launch / (0.6 * HBM_PEAK_GBS * 1e9) * 1e3, 5),
                     "bw_copy": round(bw_copy, 1), "frac_of_copy": round(achieved / bw_copy, 4),
                     **(skeleton or {})},
        "force_apply_median": {"ms_per_apply": fa["ms_per_apply"], "gll_pts_per_s": fa["gll_pts_per_s"],
                               "hbm_frac": fa["hbm_frac"], "applies": args.apply_reps, "warmup": 10} if fa else None,
        "unique_nodes_per_s": mesh.nglob / (step_ms * 1e-3),
        "force_apply": apply,
        "wall_s_timed": round(wall, 3),
        "setup_s": round(setup_s, 1),
    }
    s.close()
    if not args.no_acoustic:
        out["acoustic"] = acoustic_leg(mesh)
    if not args.no_adjoint:
        out["adjoint"] = adjoint_leg()
    if not args.no_order_sweep:
        full = args.order_sweep_full
        out["order_sweep"] = order_sweep_leg(orders=None if full else (4, 5, 6, 7, 8, 9, 12, 16))
        progress("order sweep done")
        # the paper's cost comparison at its equal-accuracy sizes needs
        # NGLL 5, 8 and 16, which the default sweep has
        out["equal_accuracy_acoustic_sizes"] = acoustic_frontier_summary(out["order_sweep"])
        if full:
            out["iso_accuracy"] = [iso_accuracy_summary(out["order_sweep"], e) for e in (1e-4, 1e-5)]
    if args.surrogate or not args.no_surrogate:
        # bounded by default: the 10 Hz workload at reduced model counts and epochs
        k = args.surrogate_scale if args.surrogate else 0.25
        out["surrogate"] = surrogate_leg(f0=args.surrogate_f0, ntrain=max(64, int(4500 * k)), nval=max(64, int(500 * k)),
                                         ntest=max(64, int(4096 * k)), epochs=max(5, int(300 * k)))
        out["surrogate"]["scale"] = k
        progress("surrogate leg done")
        if not args.surrogate:
            # the same pipeline with a source the mesh resolves: the reduced
            # configuration of the GPU test (8^3 box, 3 Hz Ricker, 200 steps ->
            # 100 samples, 4096 training models), where most models are accepted
            out["surrogate_resolved_source"] = surrogate_leg(
                f0=3.0, ne=8, nt=200, nout=100, ntrain=4096, nval=128, ntest=256, epochs=120, hidden=(256, 256, 256),
                batch=64, dt=0.01, val_seed0=5000)
            progress("resolved-source surrogate leg done")
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(mesh, wl.lam, wl.mu)
        if "acoustic" in out:
            out["acoustic"]["cpu_baseline"] = cpu_baseline_acoustic(mesh)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
