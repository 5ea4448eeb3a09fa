#!/usr/bin/env python
"""Benchmark: FMM-BEM solve seconds per time step on the 1000-bubble cluster.

One step = one BEM solve as inside a time step of the paper's method: the
vertices move (device-to-device copy of positions, which invalidates the
geometry and the octree), then geometry, octree build, the five-channel
pass for the singular diagonals and b, and GMRES for q = dphi/dn. Inputs
(mesh, positions, phi) are resident in HBM before the timed region.

Prints one JSON line (see the keys below). Kernel times come from HIP
events recorded by the library on its stream around every launch inside
the timed region.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "FMM-BEM solve s/step at 1.28M tris: tuned vs plain FP64, dphi/dn rel err<=1e-6"
PEAK_FP64_TFLOPS = 78.6  # MI355X FP64 vector and FP64 matrix (dense)
# HBM bytes per launch measured with hardware counters (FETCH_SIZE and
# WRITE_SIZE, scaled by a copy of known size), one line per kernel, workload,
# octree depth and order; a line counts only while the kernels' sources hash
# to the value it was measured with.
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "hbm_traffic_c1000.txt")
KERNEL_SOURCES = {"p2p": ("fmm_near.hip", "fmm_kernels.h", "fmm.h", "tree.h", "common.h"),
                  "m2l": ("fmm.hip", "fmm_rot.hip", "fmm_azim.hip", "fmm.h", "common.h"),
                  "leaf": ("fmm_leaf.hip", "fmm_kernels.h", "fmm.h", "tree.h", "common.h")}


def parse():
    """Command line. Solver options left unset take the values of the form
    (paper_1905_01341_amd/forms.py), which the oracle tests use too."""
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="c1000")
    ap.add_argument("--p", type=int, default=None)
    ap.add_argument("--p-diag", type=int, default=None)
    ap.add_argument("--p-lo", type=int, default=None, help="order of the low-precision products (autotuned if unset)")
    ap.add_argument("--leaf", type=int, default=None)
    ap.add_argument("--lmax", type=int, default=None)
    ap.add_argument("--m2l-shape", type=int, default=None, help="M2L launch shape 0..2, 3 (rotation-factored); -1: by size")
    ap.add_argument("--tol", type=float, default=None, help="GMRES tolerance of the tuned form")
    ap.add_argument("--plain-tol", type=float, default=None,
                    help="GMRES tolerance of the plain form (unpreconditioned GMRES needs 1e-8 to bring "
                         "the solution within 1e-6 of the oracle's; at 1e-7 it stops at 2.5e-6)")
    ap.add_argument("--restart", type=int, default=None)
    ap.add_argument("--near-corr", type=int, default=None,
                    help="1: near-field correction matrices in every product (a different discrete system: "
                         "the error is then taken against an FP64 GPU solve of the corrected system)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-rows", type=int, default=40000)
    ap.add_argument("--no-profile", action="store_true")
    ap.add_argument("--no-probe", action="store_true", help="skip the ceiling probes (measured peaks of each mix)")
    ap.add_argument("--form", choices=["tuned", "plain"], default="tuned")
    ap.add_argument("--precond-degree", type=int, default=None)
    ap.add_argument("--plain-steps", type=int, default=2)
    ap.add_argument("--graph", type=int, default=None, help="tuned form: replay GMRES products from a HIP graph")
    ap.add_argument("--autotune", type=int, default=1, help="tuned form: autotune p, octree depth, M2L shape")
    ap.add_argument("--tune-tol", type=float, default=None)
    ap.add_argument("--learned-steps", type=int, default=0,
                    help="run the learned-guess study instead: this many time steps collect training "
                         "pairs, then the same number of steps are run with zero, previous-step and "
                         "learned initial guesses")
    ap.add_argument("--ref-gpu", type=int, default=-1,
                    help="also solve the workload in FP64 on the GPU at order 20, every translation at full order, "
                         "tolerance 1e-10, and report the timed solve's error against it (-1: only when there "
                         "is no stored oracle solution for the workload)")
    ap.add_argument("--calib-copy-mib", type=int, default=0,
                    help="before the timed region, copy a buffer of this many MiB once (reference "
                         "dispatch for hardware byte counters)")
    return ap.parse_args()


def kernel_source_sha(cls):
    """First 16 hex digits of the SHA-256 of the sources of a kernel class
    ("p2p" or "m2l")."""
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[cls]:
        with open(os.path.join(ROOT, "paper_1905_01341_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(cls, kernel, workload, lmax, p):
    """(bytes per launch, fetch KiB, write KiB) of the line for this kernel,
    workload, depth and order measured on the kernel class's current
    sources, else None.
    Lines: kernel, workload, lmax, p, source hash, launches, FETCH_SIZE KiB,
    WRITE_SIZE KiB, fetch scale, write scale, bytes per launch (tab separated)."""
    if not os.path.exists(TRAFFIC_FILE):
        return None
    sha = kernel_source_sha(cls)
    with open(TRAFFIC_FILE) as fh:
        for line in fh:
            if line.startswith("#") or not line.strip():
                continue
            f = line.rstrip("\n").split("\t")
            if (len(f) == 11 and f[0] == kernel and f[1] == workload and int(f[2]) == lmax
                    and int(f[3]) == p and f[4] == sha):
                return float(f[10]), float(f[6]), float(f[7])
    return None


def m2l_kernel_name(p, shape, orders=0):
    """Instantiation(s) of the FP64 M2L kernels for order p and launch shape:
    the azimuth-reduced translation (template arguments: applied order, stored
    order, row-block pairs, waves, kind) and the sum per target box of each
    order group (reduced orders for distant offsets make two or three), or
    the rotation-factored form (applied order, stored order), joined by
    ' + '."""
    orders_p = [p] if not orders else list(dict.fromkeys([p, 4 * ((p + 4) // 5), 4 * ((3 * p + 19) // 20)]))
    names = []
    for k, po in enumerate(orders_p):
        if shape == 3:
            names.append(f"bfm::k_m2l_rot<{po}, {p}>")
            continue
        pairs, waves = {0: (None, 8), 1: (None, 4), 2: (1, 1)}[shape]
        pairs = pairs or (1 if po <= 4 else (5 if po == 12 else 3))
        names.append(f"bfm::k_translate_az<{po}, {p}, {pairs}, {waves}, 0> + "
                     f"bfm::k_az_reduce<{po}, {'true' if k == 0 else 'false'}>")
    return " + ".join(names)


def cpu_baseline(cl, phi, matvecs, rows_n):
    """The oracle (unchanged) on a bounded receiver sample of the same
    workload, scaled to one solve: one pass of the diagonal/RHS sums plus
    `matvecs` direct products (the plain solve's count; the oracle's GMRES is
    unpreconditioned), each costing N receivers."""
    import oracle
    oracle.build(force=False)
    rows = np.arange(0, cl.nv, max(1, cl.nv // rows_n), dtype=np.int64)[:rows_n]
    s, n, _ = oracle.geometry(cl.xyz, cl.tri)
    t0 = time.perf_counter()
    oracle.sums(cl.xyz, s, n, phi, rows=rows)
    t1 = time.perf_counter()
    oracle.offdiag_mvp(cl.xyz, s, n, 1.0, phi, rows=rows)
    t2 = time.perf_counter()
    per_row_sums = (t1 - t0) / len(rows)
    per_row_mvp = (t2 - t1) / len(rows)
    est = cl.nv * (per_row_sums + matvecs * per_row_mvp)
    return {
        "value": est, "unit": "s/step", "cores": oracle.num_threads(), "cpu": cpu_model(), "kind": "oracle",
        "sample": (f"direct sums and one direct product for {len(rows)} evenly spaced receivers x "
                   f"{cl.nv} sources ({t2 - t0:.1f} s), scaled to {cl.nv} receivers and "
                   f"{matvecs} products (the GPU solve's count)"),
    }


def learned_study(a):
    """Time-stepped cluster (the 1000-bubble cluster, phi = 0 at rest,
    p_inf = 1 + 0.5 sin(2 pi t / 5), surface tension 0.073, kappa 1.4, shape
    filter p_f = 9, dt = 0.1 min edge (rho / P_a)^(1/2)): the first
    `learned_steps` steps collect (features, targets) of every solve and the
    network is trained on them; then the same number of steps is run from
    that state three times, starting GMRES from zero, from the previous
    solve's q, and from the learned guess. Prints one JSON line."""
    import torch
    from paper_1905_01341_amd import bfm
    from paper_1905_01341_amd import workload as wl
    cl, _ = wl.make(a.workload)
    t0 = time.perf_counter()
    edges = np.concatenate([np.linalg.norm(cl.xyz[cl.tri[:, i]] - cl.xyz[cl.tri[:, (i + 1) % 3]], axis=1)
                            for i in range(3)])
    dt = 0.1 * float(edges.min()) * (1.0 / 0.5) ** 0.5
    from paper_1905_01341_amd import forms
    sv = bfm.Solver(device=0, **forms.options("tuned", p=a.p, leaf_target=a.leaf, gmres_tol=a.tol,
                                              gmres_restart=a.restart, precond_degree=a.precond_degree,
                                              use_graph=0))
    sv.set_cluster(cl)
    phys = dict(sigma=0.073, kappa=1.4, p0=1.0, pa=0.5, period=5.0, forcing_sign=1.0, filter_degree=9)
    sv.set_physics(guess=bfm.GUESS_GIVEN, collect=1, **phys)
    sv.state_set(cl.xyz, np.zeros(cl.nv), 0.0)
    train = []
    for _ in range(a.learned_steps):
        train.append(sv.step(dt))
    xyz, phi, t = sv.state_get()
    rows = sv.mlp_dataset()
    torch.cuda.synchronize()
    tf = time.perf_counter()
    loss1 = sv.mlp_fit(1, batch=256, lr=1e-3, seed=1)
    loss = sv.mlp_fit(30, batch=256, lr=1e-3, seed=2)
    t_fit = time.perf_counter() - tf
    runs = {}
    for name, guess in (("zero", bfm.GUESS_ZERO), ("previous", bfm.GUESS_GIVEN), ("learned", bfm.GUESS_LEARNED)):
        sv.set_physics(guess=guess, collect=0, **phys)
        sv.state_set(xyz, phi, t)
        infos = [sv.step(dt) for _ in range(a.learned_steps)]
        solves = sum(i["solves"] for i in infos)
        runs[name] = {"iterations_per_solve": round(sum(i["iterations"] for i in infos) / solves, 3),
                      "ms_per_step": round(sum(i["ms"] for i in infos) / len(infos), 3), "solves": solves}
    out = {"study": "learned initial guess", "workload": f"{a.workload} time-stepped, dt={dt:.5f}",
           "train_steps": a.learned_steps, "train_rows": rows, "fit_seconds": round(t_fit, 3),
           "loss_first_epoch": loss1, "loss_last_epoch": loss, "eval_steps": a.learned_steps,
           "runs": runs, "seconds": round(time.perf_counter() - t0, 1)}
    print(json.dumps(out), flush=True)


def form_text(opt):
    """One line describing the tuned form's arithmetic and solver."""
    if opt.precision == 0:
        arith = "FP64 FMM products"
    else:
        kind = {1: "FP32", 2: "split-BF16 (hi + lo, three products, FP32 accumulation)"}[opt.precision]
        arith = (f"mixed-precision iterative refinement: GMRES Arnoldi products with {kind} "
                 f"translations and an FP32 near field at order {opt.p_lo}, FP64 residuals at order {opt.p}, "
                 f"cycles ending at a {opt.ir_tol:g} residual reduction")
    if opt.precond == 0:
        return f"tuned: {arith}; GMRES without a preconditioner (toroidal bubbles: no spherical template)"
    return (f"tuned: {arith}; GMRES right-preconditioned by a two-level method (per-bubble spherical "
            f"harmonics to degree {opt.precond_degree}, then a coarse correction with one unknown per bubble)")


def cpu_model():
    """CPU model name of the host (from /proc/cpuinfo), or None."""
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


PEAK_BF16_TFLOPS = 2500.0  # MI355X dense BF16 MFMA
PEAK_FP32_TFLOPS = 157.3   # MI355X FP32 vector (packed; plain FP32 issues at half of it)


def p2p_kernel_name(group):
    return {"": "bfm::k_p2p_sym", "diag_": "bfm::k_p2p_diag<true>", "lo_": "bfm::k_p2p_sym32"}.get(group)


def roofline_entry(cls, prof, prof_steps, stats, opt, p_diag, nv, workload):
    """Roofline line of one kernel class: algorithmic flops of its launches
    over their summed event time against the peak of the arithmetic the
    kernel runs on (FP64 MFMA for the FP64 M2L, BF16 MFMA / 3 for the
    split-BF16 M2L, which issues three BF16 products per FP32-equivalent
    product; FP64 or FP32 vector peak for the near field, which is bound by
    plain ALU work), with the HBM traffic measured for that kernel where the
    traffic table holds a line for it on the current sources."""
    d = prof[cls]
    if d["launches"] == 0 or d["ms"] <= 0:
        return None
    group = next((g for g in ("diag_", "lo_") if cls.startswith(g)), "")
    kind = cls[len(group):]
    p = {"": opt.p, "diag_": p_diag, "lo_": opt.p_lo or opt.p}[group]
    lo_prec = opt.precision if group == "lo_" else 0
    if kind == "m2l":
        pp = p * p
        if lo_prec == 2:
            orders_p = [p] if not opt.m2l_orders else [p, 4 * ((p + 4) // 5), 4 * ((3 * p + 19) // 20)]
            kname = " + ".join(f"bfm::k_translate_bf3<{q * q}, {q * q if q * q <= 144 else (128 if q * q == 256 else 80)}, "
                               f"0, true, {pp}>" for q in dict.fromkeys(orders_p)) + f" + bfm::k_m2l_reduce<{pp}>"
            peak, unit_bytes = PEAK_BF16_TFLOPS / 3.0, 4.0
        elif lo_prec == 1:
            kname, peak, unit_bytes = None, PEAK_FP32_TFLOPS, 4.0
        else:
            shape = stats["diag_m2l_shape" if group else "m2l_shape"]
            kname = m2l_kernel_name(p, shape, opt.m2l_orders) if shape >= 0 else None
            peak, unit_bytes = PEAK_FP64_TFLOPS, 8.0
        bound, tcls = "mfma", "m2l"
        nch = 5 if group == "diag_" else 1
        # every operator read once, every box's multipole read and local
        # expansion written once (FP64: 34 operators of a cosine and a sine
        # block; rotation-factored: two rotations of sum (2n+1)^2 and a
        # translation along the axis of sum (p-m)^2 per offset)
        shape_used = stats["diag_m2l_shape" if group else "m2l_shape"] if not lo_prec else -1
        if lo_prec:
            op_words = 316 * pp * pp
        elif shape_used == 3:
            op_words = 316 * (2 * p * (4 * p * p - 1) // 3 + p * (p + 1) * (2 * p + 1) // 6)
        else:
            op_words = 34 * (pp * pp + pp) // 2
        alg_bytes = unit_bytes * (op_words + 2 * stats["boxes"] * pp * nch)
    elif kind == "p2p":
        kname = p2p_kernel_name(group)
        bound, tcls = "alu", "p2p"
        peak = PEAK_FP32_TFLOPS if group == "lo_" else PEAK_FP64_TFLOPS
        # positions (24 B) and strengths of every point read once, its sums
        # written once (one channel: 8 + 8 B; five packed channels: a 128-byte
        # record read, five sums written)
        alg_bytes = (168.0 if group == "diag_" else 40.0) * nv
    else:
        return None
    # the ceiling probe of the same instruction mix (bench.py --probe runs)
    if kind == "m2l":
        probe = {0: ("fp64_mfma", 1.0), 2: ("bf16_mfma", 3.0)}.get(lo_prec)
    else:
        probe = {"": ("fp64_pair", 1.0), "lo_": ("fp32_pair", 1.0)}.get(group)
    avg_ms = d["ms"] / d["launches"]
    ach = d["flops"] / (d["ms"] * 1e-3) / 1e12
    tr = measured_traffic(tcls, kname, workload, stats["lmax"], p) if kname else None
    return {"kernel": kname or cls, "class": cls, "bound": bound,
            "achieved": round(ach, 3), "peak": round(peak, 1), "unit": "TFLOP/s",
            "frac": round(ach / peak, 4),
            "traffic": None if tr is None else round(tr[0]),
            "traffic_unit": "HBM bytes per launch (rocprofv3 FETCH_SIZE and WRITE_SIZE, copy-calibrated)",
            "traffic_GBps": None if tr is None else round(tr[0] / (avg_ms * 1e-3) / 1e9, 1),
            "algorithmic_bytes": alg_bytes,
            "avg_launch_ms": round(avg_ms, 4), "launches": d["launches"],
            "ms_per_step": round(d["ms"] / prof_steps, 4),
            "flops_per_launch": d["flops"] / d["launches"],
            "probe": None if probe is None else {"mix": probe[0], "divisor": probe[1]}}


# ceiling probes (include/bfm_debug.h bfm_debug_probe): kind, iterations per
# lane (each launch takes a few milliseconds)
PROBES = {"fp64_mfma": (0, 100), "fp64_fma": (1, 10000), "fp32_fma": (2, 10000), "fp64_pair": (3, 30),
          "fp32_pair": (4, 60), "bf16_mfma": (5, 400)}


def run_probes():
    """Achieved TFLOP/s of every ceiling probe (pair probes: 11 flops per pair)."""
    from paper_1905_01341_amd import bfm
    out = {}
    for name, (kind, iters) in PROBES.items():
        ms, ops = bfm.debug_probe(kind, iters)
        out[name] = {"tflops": round(ops / (ms * 1e-3) / 1e12, 2), "ms": round(ms, 3)}
    return out


def attach_probe(entry, probes):
    """probe_peak / probe_frac of a roofline entry from the measured ceilings."""
    if entry is None:
        return entry
    pr = entry.pop("probe", None)
    if pr is None or probes is None or pr["mix"] not in probes:
        entry["probe_peak"] = entry["probe_frac"] = None
        return entry
    peak = probes[pr["mix"]]["tflops"] / pr["divisor"]
    entry["probe_mix"] = pr["mix"] + (f" / {pr['divisor']:g}" if pr["divisor"] != 1.0 else "")
    entry["probe_peak"] = round(peak, 2)
    entry["probe_frac"] = round(entry["achieved"] / peak, 4) if peak > 0 else None
    return entry


def main():
    a = parse()
    if a.gpus != 1:
        print("bench.py: this build measures one GPU; multi-GPU runs are not part of it "
              f"(asked for --gpus {a.gpus})", file=sys.stderr)
        sys.exit(2)
    if a.learned_steps > 0:
        return learned_study(a)
    import torch
    from paper_1905_01341_amd import bfm
    from paper_1905_01341_amd import forms
    from paper_1905_01341_amd import workload as wl

    cl, phi = wl.make(a.workload)
    dev = torch.device("cuda:0")
    if a.calib_copy_mib > 0:
        src = torch.ones(a.calib_copy_mib * (1 << 20) // 8, dtype=torch.float64, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    xyz_t = torch.tensor(cl.xyz, dtype=torch.float64, device=dev).contiguous()
    phi_t = torch.tensor(phi, dtype=torch.float64, device=dev).contiguous()
    q_t = torch.zeros_like(phi_t)
    overrides = dict(p=a.p, p_diag=a.p_diag, leaf_target=a.leaf, lmax=a.lmax, m2l_shape=a.m2l_shape,
                     gmres_restart=a.restart, precond_degree=a.precond_degree, near_corr=a.near_corr)
    tuned_only = dict(p_lo=a.p_lo)
    # the harmonic preconditioners work in a sphere template's harmonics:
    # toroidal clusters are solved without one
    toroidal = getattr(cl, "angles", None) is not None
    if toroidal:
        tuned_only["precond"] = bfm.PRECOND_NONE
        if a.tol is None:  # unpreconditioned, 1e-7 leaves 2.3e-6 of error on the 1000-torus cluster
            a.tol = 1e-8

    def run(sv, steps, warmup, profile):
        def step():
            bfm._check(sv.lib.bfm_set_positions_dev(sv.h, bfm.ctypes.c_void_p(xyz_t.data_ptr())))
            return sv.solve_dev(phi_t, q_t)
        for _ in range(warmup):
            step()
        torch.cuda.synchronize()
        if profile:
            sv.profile(True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        infos = [step() for _ in range(steps)]
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        prof = sv.profile_read() if profile else None
        sv.profile(False)
        return (t1 - t0) * 1e3 / steps, infos[-1], prof

    def error_vs_oracle():
        """Relative 2-norm error of the solution now in q_t against the
        oracle's stored solution of this workload (None if there is none)."""
        gold = os.path.join(ROOT, "tests", "golden", f"{a.workload}_q_oracle.npy")
        if not os.path.exists(gold) or a.near_corr:  # the stored solution is the nodal system's
            return None
        qo = np.load(gold).astype(np.float64)
        return float(np.linalg.norm(q_t.cpu().numpy() - qo) / np.linalg.norm(qo))

    # plain FP64 (the paper's unpreconditioned GMRES from a zero guess)
    ms_plain, info_plain, err_plain = None, None, None
    if a.plain_steps > 0:
        sv_plain, _ = forms.make_solver(cl, "plain", gmres_tol=a.plain_tol, **overrides)
        plain_tol = sv_plain.opt.gmres_tol
        ms_plain, info_plain, _ = run(sv_plain, a.plain_steps, a.warmup, False)
        err_plain = error_vs_oracle()
        sv_plain.close()
    # the reported form, timed for the value
    tuned = a.form == "tuned"
    t0 = time.perf_counter()
    if tuned:
        sv, tune = forms.make_solver(cl, "tuned", autotune=bool(a.autotune),
                                     tune_tol=forms.TUNE_TOL if a.tune_tol is None else a.tune_tol,
                                     gmres_tol=a.tol, use_graph=a.graph, **overrides, **tuned_only)
    else:
        sv, tune = forms.make_solver(cl, "plain", gmres_tol=a.plain_tol, **overrides)
    if tune is not None:
        tune["seconds"] = round(time.perf_counter() - t0, 3)
    graph_on = bool(sv.opt.use_graph)
    # kernel classes are timed with HIP events around every launch, which
    # runs every product eagerly and each near field in line with its far
    # field; so the timed steps run without it and the same solve is
    # profiled again afterwards
    ms, info, _ = run(sv, a.steps, a.warmup, False)
    # the error of the timed solve's result, before the profiling re-run
    err = error_vs_oracle()
    prof, prof_steps = None, 0
    if not a.no_profile:
        prof_steps = max(1, min(a.steps, 3))
        _, _, prof = run(sv, prof_steps, 0, True)
    stats = sv.tree_stats()
    p_diag = sv.opt.p_diag or min(20, sv.opt.p + 4)
    # reference FP64 GPU solve (the direct oracle is out of reach at millions of nodes)
    err_ref = None
    if a.ref_gpu == 1 or (a.ref_gpu == -1 and err is None):
        q_timed = q_t.clone()
        sv_ref, _ = forms.make_solver(cl, "tuned", autotune=False, use_graph=0, precision=bfm.PREC_FP64,
                                      m2l_orders=0, p=20, p_diag=20, gmres_tol=1e-10, near_corr=a.near_corr,
                                      **({"precond": bfm.PRECOND_NONE, "gmres_maxit": 2000} if toroidal else {}))
        info_ref = sv_ref.solve_dev(phi_t, q_t)
        q_ref = q_t.clone()
        sv_ref.close()
        err_ref = {"error": float(torch.linalg.norm(q_timed - q_ref) / torch.linalg.norm(q_ref)),
                   "reference": "FP64 GPU solve, p = p_diag = 20, full-order translations, GMRES tolerance 1e-10",
                   "reference_iterations": info_ref["iterations"]}
        q_t.copy_(q_timed)

    # measured ceilings of the hot kernels' instruction mixes, after the timed
    # region (a few milliseconds of probe kernels)
    probes = None if a.no_probe else run_probes()
    roof, roof_p2p = None, None
    if prof:
        named = [c for c in ("m2l", "p2p", "diag_m2l", "diag_p2p", "lo_m2l", "lo_p2p") if prof[c]["launches"] > 0]
        entries = {c: attach_probe(roofline_entry(c, prof, prof_steps, stats, sv.opt, p_diag, cl.nv, a.workload),
                                   probes)
                   for c in named}
        entries = {c: e for c, e in entries.items() if e is not None}
        if entries:
            # the kernel with the largest time per step across every product
            # group (GMRES products and the diagonal/right-hand-side pass)
            dom = max(entries, key=lambda c: prof[c]["ms"])
            roof = entries[dom]
            # the near field of the GMRES products (the low-precision one when
            # the solve refines)
            roof_p2p = entries.get("lo_p2p") or entries.get("p2p")
    out = {
        "metric": METRIC, "value": round(ms / 1e3, 6), "unit": "s/step", "n_gpus": 1,
        "steps": a.steps, "warmup": a.warmup, "ms_per_step": round(ms, 3),
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": {0: "f64", 1: "f64+f32", 2: "f64+bf16x3"}[sv.opt.precision] if tuned else "f64",
        "data": "synthetic",
        "config": {
            "workload": (f"{a.workload}: {cl.nb} {'toroidal' if toroidal else 'icosphere'} bubbles, "
                         f"{cl.nv} nodes, {cl.nt} triangles"),
            "form": form_text(sv.opt) if tuned else "plain FP64",
            "p": sv.opt.p, "p_lo": sv.opt.p_lo if sv.opt.precision else None, "p_diag": p_diag,
            "graph": graph_on, "autotune": tune, "near_corr": bool(sv.opt.near_corr),
            "lmax": stats["lmax"], "leaves": stats["leaves"], "near_pairs": stats["near_pairs"],
            "m2l_pairs": stats["m2l_pairs"], "gmres_tol": sv.opt.gmres_tol, "gmres_restart": sv.opt.gmres_restart,
            "iterations": info["iterations"], "matvecs": info["matvecs"],
            "rel_residual": info["rel_residual"], "err_vs_oracle": err, "err_vs_fp64_gpu": err_ref,
            "phase_ms": {"tree": round(info["t_tree_ms"], 3), "diag": round(info["t_diag_ms"], 3),
                         "gmres": round(info["t_solve_ms"], 3)},
            "plain_fp64": None if info_plain is None else {
                "s_per_step": round(ms_plain / 1e3, 6), "gmres_tol": plain_tol,
                "iterations": info_plain["iterations"],
                "matvecs": info_plain["matvecs"], "err_vs_oracle": err_plain, "steps": a.plain_steps},
            "speedup_vs_plain": None if ms_plain is None else round(ms_plain / ms, 3),
        },
        "roofline": roof,
        "roofline_p2p": roof_p2p,
        "probes_tflops": None if probes is None else {k: v["tflops"] for k, v in probes.items()},
    }
    if prof:
        out["kernels_ms_per_step"] = {k: round(v["ms"] / prof_steps, 3) for k, v in prof.items()
                                      if v["launches"] > 0}
    if not a.no_cpu_baseline:
        mv = info_plain["matvecs"] if info_plain is not None else info["matvecs"]
        out["cpu_baseline"] = cpu_baseline(cl, phi, mv, a.cpu_rows)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
