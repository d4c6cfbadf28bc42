#!/usr/bin/env python3
"""Throughput of the local Hamiltonian on one MI355X, in orbital-gridpoints/s.

One step is the whole hot path over one batch: wavelet synthesis, magic
filter, density and potential product, transposed magic filter, kinetic
operator, wavelet analysis (the local H*psi of Sec. 2.4, with the density of
Sec. 2.5 and the float64 energy reductions), then the float64 overlap matrix
and the Cholesky orthonormalisation of the batch (Sec. 5 step VIII).

Workload: 256 orbitals on a periodic coarse grid of 48^3 (fine 96^3), the
precision form of the method; float64 is the headline, plain float32 and
compensated float32 (hi + lo planes) are reported beside it, each with the
error of every result (H*psi, rho, E_loc, E_kin, per-orbital energies)
against the float64 oracle run over the whole batch on the host cores, which
also gives the CPU baseline.  Inputs are seeded and synthetic and already
resident in device memory when the timed region starts.  The uneven batch
(512 orbitals, coarse dims uniform in 16..64 per axis, one potential per
orbital, compensated float32, persistent launches replayed from a hipGraph,
launch sequence and tile shape picked by the tuner) is measured after it,
with its error on sampled orbitals.

Prints one JSON line.  Options: --steps K --warmup W --gpus 1.
"""

import argparse
import ctypes
import hashlib
import json
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "orbital-gridpoints/s for local H*psi (HBM GB/s % peak), FP64 vs FP32-comp at 1e-10"
HBM_PEAK_GBS = 8000.0
FP64_PEAK_TFLOPS = 78.6      # MI355X float64, vector and matrix cores alike
ESIZE = {"f64": 8, "f32": 4, "f32c": 8}
TOL = {"f64": 1e-12, "f32": 2e-6, "f32c": 1e-10}

# Operation count of the method per orbital-gridpoint and axis (flop): the
# 16-tap synthesis, magic filter, its transpose and analysis (16 FMA each)
# and the 29-tap kinetic filter plus its accumulation (59 flop).
FLOP_AXIS = 4 * 32 + 59
FLOP_POINTWISE = 4           # rho += f psi^2, V psi


VARIANT_NAMES = {0: "pass-by-pass", 1: "plane-resident",
                 2: "plane-resident (float64)",
                 3: "plane-resident (float pairs, last z step fused)"}
NCAND = 15      # tuner candidates: 5 launch sequences x 3 tile shapes


def stage_model(stage, prec, variant):
    """(bound, algorithmic bytes per orbital-gridpoint, algorithmic flop per
    orbital-gridpoint) of one profiled stage.  Bytes: each value the stage
    must read or write once (plane kernel: u and c in, t and kxy out; a z
    pass that accumulates also reads the accumulator); flop: the method's
    operation count for the axes the stage covers."""
    es = ESIZE[prec]
    if stage == "xy_plane":
        return "alu", 4 * es, 2 * FLOP_AXIS + FLOP_POINTWISE
    if stage == "z_final":       # t, c, kxy in; H*psi out
        return "hbm", 4 * es, None
    if stage.endswith("_z") and stage.startswith(("ck", "cwt")) and variant >= 1:
        return "hbm", 3 * es, None
    if stage.startswith(("kin_", "ck_")):
        return "hbm", 3 * es, None
    if stage[:3] in ("mf_", "mft", "syn", "ana", "cw_", "cwt"):
        return "hbm", 2 * es, None
    if stage == "potential":
        return "hbm", 2 * es, None
    if stage in ("overlap", "trmm"):
        return "mfma", None, None
    return None, None, None


# the sources each profiled kernel is built from
STAGE_SOURCES = {
    "xy_plane": ["wvl_xy.hip", "wvl_line.h", "wvl_line_f64_sh.hip", "wvl_plane.h", "wvl_kernels.h",
                 "wvl_internal.h", "filters_gen.h"],
}


def kernel_sources_hash(stage):
    """Hash of the sources of a stage's kernel: a stored counter reading is
    only used while the kernel is the one it was taken on."""
    h = hashlib.sha256()
    cdir = os.path.join(ROOT, "paper_0904_1543_amd", "csrc")
    for name in STAGE_SOURCES[stage]:
        with open(os.path.join(cdir, name), "rb") as f:
            h.update(name.encode() + b"\0" + f.read())
    return h.hexdigest()[:16]


def stored_traffic(stage):
    """HBM bytes per launch of `stage` from the committed counter summary
    (FETCH_SIZE + WRITE_SIZE, scaled by the copy-kernel calibration), or None
    if there is none for the current kernel sources."""
    path = os.path.join(ROOT, "profiles", f"{stage}_traffic.txt")
    if stage not in STAGE_SOURCES or not os.path.exists(path):
        return None
    text = open(path).read()
    m = re.search(r"^sources_hash:\s*(\S+)", text, re.M)
    b = re.search(r"^hbm_bytes_per_launch:\s*([0-9.eE+]+)", text, re.M)
    if not m or not b or m.group(1) != kernel_sources_hash(stage):
        return None
    return float(b.group(1))


def run_precision(prec, C, V, dims, steps, warmup, keep_outputs):
    import torch
    from paper_0904_1543_amd import lib, ops

    plan = ops.Plan(dims, prec=prec)
    c = plan.pack(C)
    Vt = plan.pack_potential(V)
    out = plan.empty()
    rho = torch.empty(plan.M[0], dtype=torch.float64, device=plan.dev)
    en = torch.empty(2, dtype=torch.float64, device=plan.dev)
    eorb = torch.empty(2 * plan.norb, dtype=torch.float64, device=plan.dev)

    def hpsi():
        lib.wvl_local_hpsi(plan.h, ops.ptr(c), ops.ptr(Vt), 1.0, 1.0, ops.ptr(out), ops.ptr(rho),
                           ctypes.c_void_p(en.data_ptr()), ctypes.c_void_p(en.data_ptr() + 8),
                           ops.ptr(eorb), ops.ptr(plan.ws), ops.stream_handle())

    def step():
        # local H*psi of the orbitals, then their orthonormalisation (Sec. 5,
        # steps III and VIII)
        hpsi()
        plan.orthonormalize(c)

    # results of this precision for the accuracy check (untimed)
    hpsi()
    torch.cuda.synchronize()
    got = None
    if keep_outputs:
        got = dict(hpsi=np.stack(plan.unpack(out)), rho=rho.cpu().numpy().copy(),
                   e_orb=eorb.cpu().numpy().copy())
    energies = en.cpu().numpy().copy()

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    plan.profile(64 * (steps + 1))
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    w0 = time.perf_counter()
    t0.record()
    for _ in range(steps):
        step()
    t1.record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - w0
    ms = t0.elapsed_time(t1) / steps
    recs = plan.profile_read()
    plan.profile(0)
    plan.sync()
    # per-stage launch durations over the timed region (hipEvents on the
    # launches' own stream)
    stages = {}
    for name, t in recs:
        s = stages.setdefault(name, [0.0, 0])
        s[0] += t
        s[1] += 1
    table = {k: {"avg_ms": v[0] / v[1], "launches": v[1], "per_step": v[1] / steps,
                 "total_ms_per_step": v[0] / steps} for k, v in stages.items()}
    hpsi_ms = sum(v[0] for k, v in stages.items()
                  if k not in ("overlap", "cholesky", "trmm")) / steps
    v = ctypes.c_int32()
    lib.wvl_plan_tuning(plan.h, ctypes.byref(v), None, 0)
    res = dict(plan=plan, ms_per_step=ms, wall_s=wall, stages=table, hpsi_ms=hpsi_ms, got=got,
               energies=energies, variant=v.value)
    del c, Vt, out, rho
    return res


def host_cpu():
    """(threads the oracle leg uses, logical CPUs, CPU model) of this host."""
    n = os.cpu_count() or 1
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return min(16, n), n, model


def oracle_batch(C, V, occ, threads):
    """The float64 oracle over every orbital of a shared-potential batch, in a
    thread pool over orbitals (numpy releases the interpreter lock inside its
    array operations).  Returns the reference results and the wall time of
    the computation."""
    from concurrent.futures import ThreadPoolExecutor
    from oracle import wavelet as W

    B = len(C)
    hp = np.empty_like(C)
    ekin = np.zeros(B)
    epot = np.zeros(B)
    parts = {}

    def one(b):
        h, psi, s = W.local_hpsi_orbital(C[b], V)
        hp[b] = h
        ekin[b] = float(np.sum(s * W.kinetic(s)))
        p2 = psi * psi
        epot[b] = float(np.sum(V * p2))
        return b, occ[b] * p2

    t = time.perf_counter()
    with ThreadPoolExecutor(threads) as ex:
        for b, contrib in ex.map(one, range(B)):
            # density summed in orbital order (map returns results in order)
            parts["rho"] = contrib if b == 0 else parts["rho"] + contrib
    wall = time.perf_counter() - t
    rho = parts["rho"]
    return dict(hpsi=hp, rho=rho, e_loc=float(np.sum(V * rho)), e_kin=float(np.dot(occ, ekin)),
                e_loc_orb=epot, e_kin_orb=ekin), wall


def errors_vs_oracle(got, energies, ref):
    """Per-result error of one precision: normwise ||d|| / ||ref|| and
    elementwise max|d| / max|ref| for H*psi and rho, |d| / |ref| for E_loc and
    E_kin and the per-orbital energies (normwise over the batch)."""
    def pair(a, b):
        d = a - b
        return {"normwise": float(np.linalg.norm(d) / np.linalg.norm(b)),
                "elementwise": float(np.max(np.abs(d)) / np.max(np.abs(b)))}
    n = len(ref["e_kin_orb"])
    eo = got["e_orb"]
    return {"hpsi": pair(got["hpsi"], ref["hpsi"]),
            "rho": pair(got["rho"], ref["rho"].ravel()),
            "e_loc": abs(float(energies[0]) - ref["e_loc"]) / abs(ref["e_loc"]),
            "e_kin": abs(float(energies[1]) - ref["e_kin"]) / abs(ref["e_kin"]),
            "e_pot_orb": pair(eo[:n], ref["e_loc_orb"]),
            "e_kin_orb": pair(eo[n:], ref["e_kin_orb"])}


PRECOND_ITERS = 5
PRECOND_FORMS = {0: "combined filter, one pass per axis",
                 1: "z pass + plane-resident in-plane kernel",
                 2: "z pass + plane-resident in-plane kernel (float pairs)"}


def run_precond(C, dims, steps, warmup, check):
    """The preconditioner (Sec. 2, Eq. "precon") on the same batch: 5 steps of
    preconditioned conjugate gradients per call, float64 and compensated
    float32, in three forms: the fused wavelet + kinetic operator with both
    in-plane axes in one plane-resident kernel, the combined filter one pass
    per axis, and the separate synthesis / kinetic / analysis passes of the
    paper's GPU design.  Inputs: the batch's coefficients as gradients, one
    orbital energy per orbital uniform in [-1, -0.1]."""
    import torch
    from paper_0904_1543_amd import inputs, lib, ops

    norb = len(dims)
    pts = norb * int(np.prod(inputs.fine_shape(dims[0])))
    eps = -inputs.rng_for(31).uniform(0.1, 1.0, size=norb)
    out = {"workload": f"{norb} orbitals, coarse 48^3 (fine 96^3), {PRECOND_ITERS} conjugate-"
                       "gradient steps per call, eps_b uniform in [-1, -0.1]",
           "iters": PRECOND_ITERS}
    sample = [0, norb - 1]
    refs = None
    if check:
        from oracle import precond as PC
        refs = {b: PC.pcg(C[b], eps[b], PRECOND_ITERS)[0] for b in sample}
    for prec in ("f64", "f32c"):
        plan = ops.Plan(dims, prec=prec)
        g = plan.pack(C)
        gt = plan.empty()
        for name, form in (("fused_plane_kernel", None), ("combined_filter_passes", "passes"),
                           ("separate_passes", "separate")):
            for _ in range(max(1, warmup)):
                plan.precondition(g, eps, PRECOND_ITERS, form=form, out=gt)
            torch.cuda.synchronize()
            t0 = torch.cuda.Event(enable_timing=True)
            t1 = torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(steps):
                plan.precondition(g, eps, PRECOND_ITERS, form=form, out=gt)
            t1.record()
            torch.cuda.synchronize()
            ms = t0.elapsed_time(t1) / steps
            rec = {"ms_per_call": ms, "ms_per_cg_step": ms / PRECOND_ITERS,
                   "orbital_gridpoints_per_s_per_step": pts / (ms / PRECOND_ITERS * 1e-3)}
            if form is None:
                rec["operator"] = PRECOND_FORMS[plan.query(lib.WVL_Q_PRECOND_FORM)]
            if refs is not None:
                got = plan.to_f64(gt)
                M = plan.M[0]
                num = den = 0.0
                for b in sample:
                    d = got[b * M:(b + 1) * M].cpu().numpy().reshape(refs[b].shape) - refs[b]
                    num += float(np.sum(d * d))
                    den += float(np.sum(refs[b] ** 2))
                rec["rel_err_vs_oracle"] = {"orbitals": sample, "normwise": (num / den) ** 0.5,
                                            "tolerance": TOL[prec]}
            out[f"{prec}/{name}"] = rec
        del plan, g, gt
        torch.cuda.empty_cache()
    return out


def run_compressed(C, V, dims, steps, warmup, check):
    """Local H*psi on compressed orbitals (steps 1-7 of Sec. 2.4) on the same
    batch, float64: coarse and fine regions of 4 atom-like spheres (radius
    0.3 and 0.15 of the box, periodic), the coefficients outside the regions
    dropped."""
    import torch
    from paper_0904_1543_amd import inputs, ops

    norb = len(dims)
    d0 = dims[0]
    seg_c, seg_f = inputs.sphere_regions(33, d0, natoms=4, rc=0.3, rf=0.15)
    plan = ops.Plan(dims, prec="f64")
    nvc, nvf = plan.set_regions(seg_c, seg_f)
    psi_c = plan.compress(plan.pack(C))
    Vt = plan.pack_potential(V)
    out = plan.empty_compressed()

    def call():
        plan.local_hpsi_compressed(psi_c, Vt, out=out, rho=False, energies=False)

    for _ in range(max(1, warmup)):
        call()
    torch.cuda.synchronize()
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    t0.record()
    for _ in range(steps):
        call()
    t1.record()
    torch.cuda.synchronize()
    ms = t0.elapsed_time(t1) / steps
    pts = norb * int(np.prod(inputs.fine_shape(d0)))
    res = {"workload": f"{norb} orbitals, coarse {d0[0]}^3, 4 spherical coarse/fine regions "
                       "(radius 0.3 / 0.15 of the box), float64",
           "nvctr_c": nvc, "nvctr_f": nvf, "compressed_fraction": (nvc + 7 * nvf) / (pts / norb),
           "ms_per_hpsi": ms, "orbital_gridpoints_per_s": pts / (ms * 1e-3)}
    if check:
        from oracle import compress as CP
        got = plan.unpack_compressed(out)
        num = den = 0.0
        for b in (0, norb - 1):
            v = CP.compress(C[b], seg_c, seg_f, d0)
            ref, _ = CP.local_hpsi_compressed(v, V, seg_c, seg_f, d0)
            num += float(np.sum((got[b] - ref) ** 2))
            den += float(np.sum(ref ** 2))
        res["rel_err_vs_oracle"] = {"orbitals": [0, norb - 1], "normwise": (num / den) ** 0.5,
                                    "tolerance": TOL["f64"]}
    del plan, psi_c, Vt, out
    torch.cuda.empty_cache()
    return res


def run_uneven(steps, warmup):
    """The 512-orbital uneven batch, compensated float32, persistent launches
    in a replayed hipGraph, launch sequence chosen by the tuner."""
    import torch
    from paper_0904_1543_amd import inputs, lib, ops

    wl = inputs.workload(5)
    dims = wl["dims"]
    t = time.perf_counter()
    plan = ops.Plan(dims, prec="f32c", shared_v=False, persistent=True, graph=True,
                    autotune=True)
    tune_s = time.perf_counter() - t
    c = plan.pack(wl["C"])
    Vt = plan.pack_potential(wl["V"])
    C_host, V_host = wl["C"], wl["V"]
    del wl
    out = plan.empty()
    eorb = torch.empty(2 * plan.norb, dtype=torch.float64, device=plan.dev)

    def hpsi():
        lib.wvl_local_hpsi(plan.h, ops.ptr(c), ops.ptr(Vt), 1.0, 1.0, ops.ptr(out), None, None,
                           None, ops.ptr(eorb), ops.ptr(plan.ws), ops.stream_handle())

    for _ in range(max(warmup, 1)):
        hpsi()
    torch.cuda.synchronize()
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    t0.record()
    for _ in range(steps):
        hpsi()
    t1.record()
    torch.cuda.synchronize()
    ms = t0.elapsed_time(t1) / steps
    v = ctypes.c_int32()
    tm = (ctypes.c_double * NCAND)()
    lib.wvl_plan_tuning(plan.h, ctypes.byref(v), tm, NCAND)
    pts = int(sum(np.prod(inputs.fine_shape(d)) for d in dims))
    seqs = ["pass_by_pass", "plane", "plane_workgroup_wide", "plane_workgroup_wide_vector", "float_pairs"]
    shapes = ["default_tiles", "half_axis1_tiles", "persistent_4_per_cu"]
    names = [f"{a}/{b}" for a in seqs for b in shapes]
    best = plan.query(lib.WVL_Q_TUNE_BEST)
    # accuracy of the replayed sequence on sampled orbitals: the largest, the
    # smallest and two others, each against the float64 oracle
    from oracle import wavelet as W
    got = plan.to_f64(out)
    torch.cuda.synchronize()
    sizes = [int(np.prod(d)) for d in dims]
    sample = sorted({int(np.argmax(sizes)), int(np.argmin(sizes)), 0, 311})
    num = den = 0.0
    emax = 0.0
    for b in sample:
        o, m = int(plan.offsets[b]), plan.M[b]
        g = got[o:o + m].cpu().numpy().reshape(inputs.fine_shape(dims[b]))
        ref = W.local_hpsi_orbital(C_host[b], V_host[b])[0]
        num += float(np.sum((g - ref) ** 2))
        den += float(np.sum(ref ** 2))
        emax = max(emax, float(np.max(np.abs(g - ref)) / np.max(np.abs(ref))))
    return {"workload": "512 orbitals, coarse dims uniform in 16..64 per axis (seed 5), "
                        "one 16-Gaussian potential per orbital, compensated float32, "
                        "replayed from a hipGraph",
            "orbital_gridpoints": pts, "ms_per_hpsi": ms,
            "orbital_gridpoints_per_s": pts / (ms * 1e-3),
            "variant": VARIANT_NAMES[v.value],
            "persistent_launches": bool(plan.query(lib.WVL_Q_PERSISTENT)),
            "tuner_choice": names[best] if best >= 0 else None,
            "axis1_tile_divisor": plan.query(lib.WVL_Q_XDIV),
            "persistent_workgroups_per_cu": plan.query(lib.WVL_Q_PGRID),
            "tuner_ms": {names[i]: tm[i] for i in range(NCAND) if tm[i] >= 0},
            "tuning_s": tune_s,
            "rel_err_vs_oracle": {"orbitals": sample, "normwise": (num / den) ** 0.5,
                                  "elementwise": emax, "tolerance": TOL["f32c"]}}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--precs", default="f64,f32c,f32")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-uneven", action="store_true")
    ap.add_argument("--no-precond", action="store_true")
    ap.add_argument("--no-compressed", action="store_true")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: this build runs on one GPU; --gpus {args.gpus} is not supported "
              "(the orbital batch would be split across GPUs by orbitals, see the design notes)",
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_0904_1543_amd import inputs

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    # known-size copy before the measured work: the counter runs of the
    # profiles calibrate FETCH_SIZE / WRITE_SIZE against it (2 x 1 GiB moved)
    src = torch.ones(1 << 27, dtype=torch.float64, device="cuda:0")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst

    wl = inputs.workload(3)
    C, V, dims = wl["C"], wl["V"], wl["dims"]
    norb = len(dims)
    pts = norb * int(np.prod(inputs.fine_shape(dims[0])))

    precs = [p for p in args.precs.split(",") if p]
    results = {}
    for prec in precs:
        print(f"[bench] {prec}: {norb} orbitals x {inputs.fine_shape(dims[0])}", file=sys.stderr,
              flush=True)
        results[prec] = run_precision(prec, C, V, dims, args.steps, args.warmup,
                                      not args.no_cpu_baseline)
        torch.cuda.empty_cache()

    compressed = precond = None
    if not args.no_compressed:
        print("[bench] compressed orbitals", file=sys.stderr, flush=True)
        compressed = run_compressed(C, V, dims, args.steps, 2, not args.no_cpu_baseline)
    if not args.no_precond:
        print("[bench] preconditioner", file=sys.stderr, flush=True)
        precond = run_precond(C, dims, max(3, args.steps // 4), 1, not args.no_cpu_baseline)

    uneven = None
    if not args.no_uneven:
        print("[bench] uneven batch: 512 orbitals, f32c, persistent + graph + tuner",
              file=sys.stderr, flush=True)
        uneven = run_uneven(args.steps, args.warmup)
        torch.cuda.empty_cache()

    # oracle over the whole batch on the host cores: the CPU baseline, and the
    # error of every result of every precision
    cpu = None
    errors = {}
    if not args.no_cpu_baseline:
        threads, ncpu, model = host_cpu()
        print(f"[bench] oracle on all {norb} orbitals, {threads} host threads", file=sys.stderr,
              flush=True)
        ref, tcpu = oracle_batch(C, V, wl["occ"], threads)
        cpu = {"value": pts / tcpu, "unit": "orbital-gridpoints/s", "cores": threads,
               "kind": "oracle",
               "sample": f"the whole batch: local H*psi, density and energies of all {norb} "
                         f"orbitals (fine 96^3), plain float64 numpy oracle in a pool of "
                         f"{threads} threads over orbitals, {tcpu:.1f} s wall; host: {ncpu} "
                         f"logical CPUs, {model}; the overlap/Cholesky step is not in the sample",
               "host_logical_cpus": ncpu, "host_cpu_model": model}
        for prec, r in results.items():
            errors[prec] = errors_vs_oracle(r["got"], r["energies"], ref)
            r["got"] = None
        del ref

    head = "f64" if "f64" in results else precs[0]
    r = results[head]
    ms = r["ms_per_step"]
    # dominant kernel of the headline precision, per launch
    dom, dstat = max(r["stages"].items(), key=lambda kv: kv[1]["total_ms_per_step"])
    bound, bpp, fpp = stage_model(dom, head, r["variant"])
    roof = None
    if bound is not None:
        units = pts / dstat["per_step"]            # orbital-gridpoints per launch
        sec = dstat["avg_ms"] * 1e-3
        traffic = stored_traffic(dom)
        if bound == "hbm" and bpp is not None:
            ach = units * bpp / sec / 1e9
            roof = {"bound": "hbm", "achieved": round(ach, 1), "peak": HBM_PEAK_GBS,
                    "unit": "GB/s", "frac": round(ach / HBM_PEAK_GBS, 4)}
        elif fpp is not None:
            ach = units * fpp / sec / 1e12
            roof = {"bound": bound, "achieved": round(ach, 2), "peak": FP64_PEAK_TFLOPS,
                    "unit": "TFLOP/s", "frac": round(ach / FP64_PEAK_TFLOPS, 4)}
        if roof is not None:
            roof.update({"traffic": traffic, "kernel": dom, "avg_launch_ms": round(dstat["avg_ms"], 4),
                         "launches_per_step": dstat["per_step"],
                         "orbital_gridpoints_per_launch": int(units),
                         "algorithmic_bytes_per_launch": int(units * bpp) if bpp else None,
                         "algorithmic_flop_per_launch": int(units * fpp) if fpp else None,
                         "hbm_equivalent_GBps": round(units * bpp / sec / 1e9, 1) if bpp else None})
    line = {
        "metric": METRIC,
        "value": pts / (ms * 1e-3),
        "unit": "orbital-gridpoints/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": head,
        "data": "synthetic",
        "config": {"workload": "256 orbitals, periodic coarse 48^3 (fine 96^3), local H*psi "
                               "with density and energies + float64 overlap/Cholesky "
                               "orthonormalisation", "orbitals": norb,
                   "fine_grid": list(inputs.fine_shape(dims[0])),
                   "potential": "16 periodic Gaussians", "seed": 3},
        "roofline": roof,
        "cpu_baseline": cpu,
        "precisions": {
            p: {"ms_per_step": v["ms_per_step"],
                "hpsi_variant": VARIANT_NAMES[v["variant"]],
                "orbital_gridpoints_per_s": pts / (v["ms_per_step"] * 1e-3),
                "hpsi_ms": v["hpsi_ms"],
                "hpsi_orbital_gridpoints_per_s": pts / (v["hpsi_ms"] * 1e-3),
                "rel_err_vs_oracle": errors.get(p),
                "tolerance": TOL[p],
                "within_tolerance": (None if p not in errors else all(
                    (v <= TOL[p]) if isinstance(v, float) else
                    (v["normwise"] <= TOL[p] and v["elementwise"] <= TOL[p])
                    for v in errors[p].values())),
                "e_loc": float(v["energies"][0]), "e_kin": float(v["energies"][1]),
                "stages": {k: {"avg_ms": round(s["avg_ms"], 4), "per_step": s["per_step"]}
                           for k, s in sorted(v["stages"].items(),
                                              key=lambda kv: -kv[1]["total_ms_per_step"])}}
            for p, v in results.items()},
        "uneven_batch": uneven,
        "preconditioner": precond,
        "compressed_hpsi": compressed,
    }
    print(json.dumps(line))


if __name__ == "__main__":
    main()
