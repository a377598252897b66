#!/usr/bin/env python3
"""Benchmark: 2D Model B (Cahn-Hilliard with conserved noise), 1024x1024, FP32.

One "step" is one full time step of the pseudo-spectral integrator (forward
and inverse transforms, real-space cubic, Philox noise, semi-implicit update)
over the whole lattice.  Prints one JSON line with site-steps/s, the roofline
position of the dominant kernel (the update kernel, HBM-bound), the FP64 CPU
oracle timed on a bounded sample of the same workload, and the two
training-system workloads measured against their plain forms:

* "ensemble": 256 x 128^2 + 64 x 256^2 + 16 x 512^2 independent lattices in
  one batch, against the same lattices stepped one lattice per launch;
* "adjoint": the gradient of a structure-factor loss through 2000 steps of
  256^2 Model B (checkpoints every 45), against the forward run alone;
* "model_h": 2D Model H at 1024^2 (the paper's second benchmark model);
* "mixed_radix": 2D Model B at 960^2, a size that is not a power of two.

Timing: the step graphs are built before any timed region (pss_step_prepare);
the lattice runs on a torch stream, and HIP events recorded on that stream
bracket each timed run of K steps, with a device synchronisation on both
sides; `value` is the median of 5 such runs.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu]
       [--workload modelb1024|ensemble|adjoint|3d|modelh] [--no-extras]
"""

import argparse
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, published
# Summary of the FETCH_SIZE / WRITE_SIZE counter runs of the update kernel on
# this workload; its traffic figure is reported only while the kernel sources
# and the launch geometry are the ones the counters were taken with.
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_update_kernel_modelb_1024.txt")
KERNEL_SOURCES = ("pss_kernels.hip", "pss_device.h", "pss_fft.h", "pss_fft_layout.h", "pss_kernels.h", "pss_plan.h")
N = (1024, 1024)
A, B, K, D, DT, SEED = -1.0, 1.0, 1.0, 0.01, 0.01, 1
REPEATS = 5


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_source_hash():
    import hashlib
    h = hashlib.sha256()
    for name in KERNEL_SOURCES:
        path = os.path.join(ROOT, "paper_2405_02410_amd", "csrc", name)
        if os.path.exists(path):
            with open(path, "rb") as f:
                h.update(f.read())
    return h.hexdigest()


def measured_traffic(geometry):
    """HBM bytes per update-kernel launch from the committed counter summary,
    or None if it is missing or was taken on other kernel code or geometry."""
    try:
        with open(TRAFFIC_FILE) as f:
            kv = dict(l.split(":", 1) for l in f.read().splitlines() if ":" in l)
    except OSError:
        return None
    kv = {k.strip(): v.strip() for k, v in kv.items()}
    if kv.get("source_sha256") != kernel_source_hash():
        return None
    if kv.get("geometry") != json.dumps(geometry, sort_keys=True):
        return None
    return float(kv["traffic_bytes_per_launch"])


def timed_runs(torch, stream, run, repeats=REPEATS):
    """Seconds of each of `repeats` calls of run(), measured with HIP events on
    `stream` and bracketed by device synchronisations."""
    out = []
    for _ in range(repeats):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(stream)
        run()
        e1.record(stream)
        torch.cuda.synchronize()
        out.append(e0.elapsed_time(e1) * 1e-3)
    return out


def cpu_baseline(steps, steps_1core=5):
    """The FP64 oracle on `steps` steps of the same workload (after one warm-up),
    on all host cores, and on `steps_1core` steps with one FFT worker."""
    from oracle import model as om
    from oracle import spectral
    cores = os.cpu_count() or 1
    sites = N[0] * N[1]

    def rate(workers, k):
        spectral.WORKERS = workers
        m = om.model_b(spectral.Lattice(*N), DT, a=A, b=B, k=K, D=D, seed=SEED)
        m.init_uniform(0, -0.1, 0.1)
        m.step(1)
        t0 = time.perf_counter()
        m.step(k)
        return sites * k / (time.perf_counter() - t0)
    value = rate(cores, steps)
    one = rate(1, steps_1core)
    return {"value": value, "unit": "site-steps/s", "cores": cores, "kind": "oracle",
            "sample": f"{steps} steps of the 1024x1024 Model B workload after 1 warm-up step "
                      f"(numpy FP64; the FFTs run on scipy.fft with {cores} workers, the elementwise "
                      f"steps are single-threaded numpy)",
            "single_core": {"value": one, "sample": f"{steps_1core} steps, scipy.fft with 1 worker"}}


def modelb1024(args, pss, torch):
    stream = torch.cuda.Stream()
    lat = pss.Lattice(N, dt=DT, seed=SEED)
    lat.stream(stream.cuda_stream)
    f, _ = pss.model_b(lat, a=A, b=B, k=K, D=D)
    lat.init_uniform(f, -0.1, 0.1)
    lat.prepare(args.warmup)
    lat.prepare(args.steps)
    log(f"bench: 2D Model B {N[0]}x{N[1]}, warmup {args.warmup}, {REPEATS} x {args.steps} steps")
    lat.step(args.warmup)
    lat.sync()
    times = timed_runs(torch, stream, lambda: lat.step(args.steps))
    el = statistics.median(times)
    sites = N[0] * N[1]
    value = sites * args.steps / el
    ms_per_step = 1e3 * el / args.steps
    log(f"bench: {ms_per_step * 1e3:.2f} us/step (runs: {', '.join(f'{1e6 * t / args.steps:.2f}' for t in times)}), "
        f"{value:.4e} site-steps/s")
    mass = lat.mass(f)

    # roofline of the dominant kernel: HIP events around back-to-back launches
    kb = lat.kernel_bytes(pss.KERNEL_UPDATE)
    ms_k, kname = lat.time_kernel(pss.KERNEL_UPDATE, args.kernel_reps)
    xb = lat.kernel_bytes(pss.KERNEL_X)
    ms_x, xname = lat.time_kernel(pss.KERNEL_X, args.kernel_reps)
    achieved = kb / (ms_k * 1e-3) / 1e9
    log(f"bench: {kname} {ms_k * 1e3:.2f} us/launch, {kb / 1e6:.2f} MB -> {achieved:.0f} GB/s; "
        f"{xname} {ms_x * 1e3:.2f} us/launch, {xb / 1e6:.2f} MB -> {xb / (ms_x * 1e-3) / 1e9:.0f} GB/s")
    step_bytes = kb + xb
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": measured_traffic(lat.geometry()),
                "kernel": kname, "bytes_per_launch": kb, "us_per_launch": round(ms_k * 1e3, 3),
                "x_kernel": {"kernel": xname, "bytes_per_launch": xb, "us_per_launch": round(ms_x * 1e3, 3),
                             "frac": round(xb / (ms_x * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)},
                "step_bytes": step_bytes,
                "step_GBs": round(step_bytes / (ms_per_step * 1e-3) / 1e9, 1)}
    return {"value": value, "ms_per_step": ms_per_step, "runs_ms_per_step": [1e3 * t / args.steps for t in times],
            "roofline": roofline, "mass_after": mass, "geometry": lat.geometry()}


ENSEMBLE = ((256, 128), (64, 256), (16, 512))  # (members, side)


def ensemble_cpu_baseline(steps):
    """The FP64 oracle on `steps` steps of one 512^2 member (after one warm-up)."""
    from oracle import model as om
    from oracle import spectral
    cores = os.cpu_count() or 1
    spectral.WORKERS = cores
    m = om.model_b(spectral.Lattice(512, 512), DT, a=A, b=B, k=K, D=D, seed=SEED)
    m.init_uniform(0, -0.1, 0.1)
    m.step(1)
    t0 = time.perf_counter()
    m.step(steps)
    dt = time.perf_counter() - t0
    return {"value": 512 * 512 * steps / dt, "unit": "site-steps/s", "cores": cores, "kind": "oracle",
            "sample": f"{steps} steps of one 512x512 member of the ensemble after 1 warm-up step "
                      f"(numpy FP64, scipy.fft with {cores} workers); members are independent, so the "
                      f"site-step rate carries over to the whole ensemble"}


def ensemble(args, pss, torch, steps):
    """Batched ensemble: every member in one batch against the same members
    stepped one lattice per launch sequence (pss_step on each, each on its own
    stream).  Both forms replay graphs built before the timed region."""
    lats, seed = [], 1000
    for count, side in ENSEMBLE:
        for _ in range(count):
            lat = pss.Lattice((side, side), dt=DT, seed=seed)
            f, _ = pss.model_b(lat, a=A, b=B, k=K, D=D)
            if args.autotune:
                lat.autotune(reps=20)  # measured once per size, then cached
            lat.init_uniform(f, -0.1, 0.1)
            lats.append(lat)
            seed += 1
    sites = sum(c * s * s for c, s in ENSEMBLE)
    batch = pss.Batch(lats)
    ncls = batch.classes()[0]
    per_step, fused, resident = batch.launches()
    log(f"bench: ensemble of {len(lats)} lattices, {sites} sites, {ncls} classes, {per_step} launches per step "
        f"({fused} classes fused), {resident} LDS-resident classes (one launch per chunk of steps)")
    batch.step(steps)  # warm-up; builds the graphs of this chunk length
    batch.sync()

    def run_batch():
        batch.step(steps)
        batch.sync()

    def wall(run):
        out = []
        for _ in range(REPEATS):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            run()
            torch.cuda.synchronize()
            out.append(time.perf_counter() - t0)
        return out
    tb = wall(run_batch)
    el = statistics.median(tb)
    value = sites * steps / el
    log(f"bench: batched {1e6 * el / steps:.1f} us/step, {value:.4e} site-steps/s")

    plain_steps = steps
    for lat in lats:
        lat.prepare(plain_steps)
        lat.step(plain_steps)  # warm-up
    for lat in lats:
        lat.sync()

    def run_plain():
        for lat in lats:
            lat.step(plain_steps)
        for lat in lats:
            lat.sync()
    tp = wall(run_plain)
    pel = statistics.median(tp)
    plain = sites * plain_steps / pel
    log(f"bench: plain {1e6 * pel / plain_steps:.1f} us/step, {plain:.4e} site-steps/s")

    # roofline of the per-step launch with the largest share of the batched
    # step: the fused launches when every other class is fused or resident,
    # else each class's own; the resident launch (state on chip between
    # steps, HBM only at its ends) is reported on its own
    res = None
    if resident:
        ms_r, bytes_r = batch.time_kernel(-2, pss.KERNEL_UPDATE, ens_reps := max(50, args.kernel_reps // 10))
        res_sites = sum(c * s * s for c, s in ENSEMBLE if s <= 128)
        res = {"ms_per_step": ms_r, "steps_per_launch": ens_reps, "sites": res_sites,
               "site_steps_per_s": res_sites / (ms_r * 1e-3), "hbm_bytes_per_step": bytes_r}
        log(f"bench: resident launch: {ms_r * 1e3:.2f} us per step over {ens_reps} steps, "
            f"{res_sites / (ms_r * 1e-3):.4e} site-steps/s")
    best = None
    units = [(-1, w) for w in (pss.KERNEL_UPDATE, pss.KERNEL_X)] if fused + resident == ncls else \
        [(c, w) for c in range(ncls) for w in (pss.KERNEL_UPDATE, pss.KERNEL_X)]
    for cls, which in units:
        ms, nbytes = batch.time_kernel(cls, which, max(50, args.kernel_reps // 10))
        log(f"bench: {'fused' if cls < 0 else f'class {cls}'} kernel {which}: {ms * 1e3:.2f} us/launch, "
            f"{nbytes / 1e6:.2f} MB")
        if best is None or ms > best[0]:
            best = (ms, nbytes, cls, which)
    ms, nbytes, cls, which = best
    achieved = nbytes / (ms * 1e-3) / 1e9
    kname = ("batch_update_kernel" if which == 0 else "batch_xrow_kernel") if cls < 0 else \
        f"{'update_kernel' if which == 0 else 'xrow_kernel'} (batched, size class {cls})"
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None,
                "kernel": kname, "bytes_per_launch": nbytes, "us_per_launch": round(ms * 1e3, 3)}
    out = {"value": value, "unit": "site-steps/s", "steps": steps, "ms_per_step": 1e3 * el / steps,
           "members": len(lats), "sites": sites, "classes": ncls, "launches_per_step": per_step,
           "fused_classes": fused, "resident_classes": resident, "resident": res,
           "plain": {"value": plain, "steps": plain_steps, "ms_per_step": 1e3 * pel / plain_steps,
                     "form": "pss_step on each lattice in turn, each on its own stream"},
           "vs_plain": round(value / plain, 2), "roofline": roofline,
           "geometry": "autotuned per size" if args.autotune else "default"}
    batch.close()
    for lat in lats:
        lat.close()
    return out


def adjoint(args, pss, torch):
    """Adjoint workload: dL/d(a, b, k, D) and dL/dphi_0 of the shell
    structure-factor loss after 2000 steps of 256^2 Model B, checkpoints every
    45 steps; the target spectrum comes from a forward run at (a, b, k, D) =
    (-1, 1, 1, 0.01), the gradient is taken at (-0.9, 1.1, 0.9, 0.012) with
    the same seed and initial field.  Compared with the plain forward run."""
    n, nsteps, ckpt = (256, 256), 2000, 45

    def make(theta):
        lat = pss.Lattice(n, dt=DT, seed=SEED)
        f, _ = pss.model_b(lat, a=theta[0], b=theta[1], k=theta[2], D=theta[3])
        lat.init_uniform(f, -0.1, 0.1)
        return lat
    ref = make((-1.0, 1.0, 1.0, 0.01))
    ref.step(nsteps)
    S_target, _ = ref.structure_factor(0)
    t_fwd, t_adj, t_rec = [], [], []
    for _ in range(3):
        fwd = make((-0.9, 1.1, 0.9, 0.012))
        fwd.prepare(nsteps)
        fwd.sync()
        t0 = time.perf_counter()
        fwd.step(nsteps)
        fwd.sync()
        t_fwd.append(time.perf_counter() - t0)
        lat = make((-0.9, 1.1, 0.9, 0.012))
        lat.prepare(ckpt)
        lat.prepare(nsteps % ckpt)
        lat.sync()
        t0 = time.perf_counter()
        loss, tape = lat.adjoint_forward(nsteps, S_target, ckpt_every=ckpt)
        lat.sync()
        t1 = time.perf_counter()
        grad = tape.backward()
        t2 = time.perf_counter()
        tape.close()
        t_rec.append(t1 - t0)
        t_adj.append(t2 - t0)
    tf, ta, tr = min(t_fwd), min(t_adj), min(t_rec)
    log(f"bench: adjoint {ta * 1e3:.1f} ms for {nsteps} steps (forward alone {tf * 1e3:.1f} ms, "
        f"checkpointed forward {tr * 1e3:.1f} ms); loss {loss:.6g}, grad {grad}")
    sites = n[0] * n[1]
    return {"value": sites * nsteps / ta, "unit": "site-steps/s", "steps": nsteps, "ckpt_every": ckpt,
            "ms": ta * 1e3, "forward_ms": tf * 1e3, "checkpointed_forward_ms": tr * 1e3,
            "plain": {"value": sites * nsteps / tf, "form": "the forward run alone (pss_step)"},
            "cost_vs_plain": round(ta / tf, 3), "vs_plain": round(tf / ta, 3),
            "loss": loss, "grad": list(grad)}


def three_d(args, pss, torch):
    """3D two-field system, 256^3 FP32: Model B phi (a, b, k = -1, 1, 1, conserved
    noise 0.005 q^2) coupled to non-conserved psi with
    d/dt psi = -(c psi + psi^3 - lap psi) - g phi psi + noise 0.005, and
    (g/2) phi psi^2 inside phi's chemical potential; c = -0.5, g = 0.3,
    dt = 0.005; launch geometry picked by pss_autotune."""
    from paper_2405_02410_amd import Mono
    n, dt, c, g, Dn = (256, 256, 256), 0.005, -0.5, 0.3, 0.005
    stream = torch.cuda.Stream()
    lat = pss.Lattice(n, dt=dt, seed=SEED)
    lat.stream(stream.cuda_stream)
    phi = lat.field("phi")
    psi = lat.field("psi")
    lat.term(phi, [Mono(-A, q2=1), Mono(-K, q2=2)], [(phi, 1)], implicit=True)
    lat.term(phi, [Mono(-B, q2=1)], [(phi, 3)])
    lat.term(phi, [Mono(-0.5 * g, q2=1)], [(phi, 1), (psi, 2)])
    lat.term(psi, [Mono(-c), Mono(-1.0, q2=1)], [(psi, 1)], implicit=True)
    lat.term(psi, [Mono(-1.0)], [(psi, 3)])
    lat.term(psi, [Mono(-g)], [(phi, 1), (psi, 1)])
    lat.noise(phi, [Mono(Dn, q2=1)])
    lat.noise(psi, [Mono(Dn)])
    us_tuned = lat.autotune(reps=20)
    lat.init_uniform(phi, -0.1, 0.1)
    lat.init_uniform(psi, -0.1, 0.1)
    steps = min(args.steps, 400)
    lat.prepare(args.warmup)
    lat.prepare(steps)
    lat.step(args.warmup)
    lat.sync()
    times = timed_runs(torch, stream, lambda: lat.step(steps))
    el = statistics.median(times)
    sites = n[0] * n[1] * n[2]
    names = ("update_kernel", "xrow_kernel", "ypass_kernel(inverse)", "ypass_kernel(forward)")
    best = None
    for w in range(lat.kernels_per_step()):
        ms, _ = lat.time_kernel(w, max(10, args.kernel_reps // 20))
        nb = lat.kernel_bytes(w)
        log(f"bench: {names[w]} {ms * 1e3:.1f} us/launch, {nb / 1e6:.1f} MB -> {nb / (ms * 1e-3) / 1e9:.0f} GB/s")
        if best is None or ms > best[0]:
            best = (ms, nb, names[w])
    ms, nb, kname = best
    achieved = nb / (ms * 1e-3) / 1e9
    log(f"bench: 3d {1e6 * el / steps:.1f} us/step, {sites * steps / el:.4e} site-steps/s")
    return {
        "metric": "site-steps/s", "value": sites * steps / el, "unit": "site-steps/s", "n_gpus": 1,
        "steps": steps, "warmup": args.warmup, "ms_per_step": 1e3 * el / steps,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "3D two-field 256^3 FP32: Model B phi coupled to Model A psi, c=-0.5 g=0.3 "
                               "D=0.005, dt=0.005, 2/3 radial de-aliasing, uniform[-0.1,0.1] initial fields",
                   "lattice": list(n), "parallelism": "single GPU", "geometry": lat.geometry(),
                   "autotuned_kernel_us_per_step": round(us_tuned, 1)},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None, "kernel": kname,
                     "bytes_per_launch": nb, "us_per_launch": round(ms * 1e3, 3)},
        "cpu_baseline": None,
    }


def model_h(args, pss, torch, cpu_steps=0):
    """2D Model H 1024^2 FP32 (pss.model_h: a=-1 b=1 k=1, M=1, eta=0.5,
    conserved noise 0.01 q^2 on phi, dt=0.01): three dynamic fields, two
    gradient intermediates, eight product channels over five factor slots."""
    n, dt = (1024, 1024), 0.01
    stream = torch.cuda.Stream()
    lat = pss.Lattice(n, dt=dt, seed=SEED)
    lat.stream(stream.cuda_stream)
    (phi, vx, vy), _ = pss.model_h(lat, a=A, b=B, k=K, M=1.0, eta=0.5, D=D)
    lat.init_uniform(phi, -0.4, 0.4)
    steps = min(args.steps, 500)
    warm = min(args.warmup, 50)
    lat.prepare(warm)
    lat.prepare(steps)
    lat.step(warm)
    lat.sync()
    times = timed_runs(torch, stream, lambda: lat.step(steps))
    el = statistics.median(times)
    sites = n[0] * n[1]
    names = ("update_kernel", "xrow_kernel")
    best = None
    for w in range(lat.kernels_per_step()):
        ms, _ = lat.time_kernel(w, max(10, args.kernel_reps // 10))
        nb = lat.kernel_bytes(w)
        log(f"bench: model h {names[w]} {ms * 1e3:.1f} us/launch, {nb / 1e6:.1f} MB -> "
            f"{nb / (ms * 1e-3) / 1e9:.0f} GB/s")
        if best is None or ms > best[0]:
            best = (ms, nb, names[w])
    ms, nb, kname = best
    achieved = nb / (ms * 1e-3) / 1e9
    log(f"bench: model h {1e6 * el / steps:.1f} us/step, {sites * steps / el:.4e} site-steps/s")
    cpu = None
    if cpu_steps > 0:
        from oracle import model as om
        from oracle.spectral import Lattice as OLattice
        m = om.model_h(OLattice(n[0], n[1], 1), dt, a=A, b=B, k=K, M=1.0, eta=0.5, D=D, seed=SEED)
        m.init_uniform(0, -0.4, 0.4)
        m.step(1)
        t0 = time.perf_counter()
        m.step(cpu_steps)
        cel = time.perf_counter() - t0
        cpu = {"value": sites * cpu_steps / cel, "unit": "site-steps/s", "cores": os.cpu_count(),
               "kind": "oracle", "sample": f"{cpu_steps} steps of the 1024x1024 Model H workload after 1 warm-up step"}
    return {
        "value": sites * steps / el, "unit": "site-steps/s", "steps": steps, "warmup": warm,
        "ms_per_step": 1e3 * el / steps, "geometry": lat.geometry(),
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None, "kernel": kname,
                     "bytes_per_launch": nb, "us_per_launch": round(ms * 1e3, 3)},
        "cpu_baseline": cpu,
    }


def mixed_radix(args, pss, torch):
    """2D Model B at 960x960 (960 = 2^6 3 5: the generic mixed-radix path,
    full spectra and one block per line) with the workload's coefficients;
    HBM bytes per step from pss_kernel_bytes of its two launches."""
    n = (960, 960)
    stream = torch.cuda.Stream()
    lat = pss.Lattice(n, dt=DT, seed=SEED)
    lat.stream(stream.cuda_stream)
    f, _ = pss.model_b(lat, a=A, b=B, k=K, D=D)
    lat.init_uniform(f, -0.1, 0.1)
    steps = min(args.steps, 200)
    warm = min(args.warmup, 20)
    lat.prepare(warm)
    lat.prepare(steps)
    lat.step(warm)
    lat.sync()
    times = timed_runs(torch, stream, lambda: lat.step(steps))
    el = statistics.median(times)
    sites = n[0] * n[1]
    step_bytes = lat.kernel_bytes(0) + lat.kernel_bytes(1)
    ms = 1e3 * el / steps
    log(f"bench: mixed-radix 960^2 {1e3 * ms:.1f} us/step, {sites * steps / el:.4e} site-steps/s, "
        f"{step_bytes / (ms * 1e-3) / 1e9:.0f} GB/s over the step")
    return {"value": sites * steps / el, "unit": "site-steps/s", "steps": steps, "ms_per_step": ms,
            "lattice": list(n), "step_bytes": step_bytes,
            "step_GBs": round(step_bytes / (ms * 1e-3) / 1e9, 1)}


def features(args, pss, torch):
    """Step rates of the other model forms at fixed sizes, each timed like the
    main workload (HIP events on the lattice stream, median of REPEATS runs):
    1D Model B lines of 4096 (radix 4) and 3000 (2^3 3 5^3, mixed radix)
    points, one block each; 2D Model B at 1024^2 with a boundary frame of 4
    columns held at 0.2 (each step also transforms the framed field to real
    space and back); 2D KPZ at 1024^2 (two gradient intermediates)."""
    out = {}

    def timed(name, lat, steps, warm):
        stream = torch.cuda.Stream()
        lat.stream(stream.cuda_stream)
        lat.prepare(warm)
        lat.prepare(steps)
        lat.step(warm)
        lat.sync()
        times = timed_runs(torch, stream, lambda: lat.step(steps))
        el = statistics.median(times)
        sites = 1
        for v in lat.n:
            sites *= v
        out[name] = {"lattice": list(lat.n), "steps": steps, "us_per_step": round(1e6 * el / steps, 3),
                     "site_steps_per_s": sites * steps / el}
        log(f"bench: {name} {1e6 * el / steps:.2f} us/step, {sites * steps / el:.4e} site-steps/s")

    for n in (4096, 3000):
        lat = pss.Lattice((n,), dt=DT, seed=SEED)
        f, _ = pss.model_b(lat, a=A, b=B, k=K, D=D)
        lat.init_uniform(f, -0.1, 0.1)
        timed(f"line_{n}", lat, 2000, 200)
    lat = pss.Lattice(N, dt=DT, seed=SEED)
    f, _ = pss.model_b(lat, a=A, b=B, k=K, D=D)
    lat.init_uniform(f, -0.1, 0.1)
    sites = [y * N[0] + x for y in range(N[1]) for x in range(4)]
    lat.frame(f, sites, [0.2] * len(sites))
    timed("frame_1024", lat, 500, 50)
    lat = pss.Lattice(N, dt=DT, seed=SEED)
    f, _ = pss.kpz(lat, sigma=1.0, lam=1.0, D=D)
    lat.init_uniform(f, -0.1, 0.1)
    timed("kpz_1024", lat, 500, 50)
    return out


def line(workload, value, steps, warmup, ms_per_step, extra):
    out = {"metric": "site-steps/s", "value": value, "unit": "site-steps/s", "n_gpus": 1,
           "steps": steps, "warmup": warmup, "ms_per_step": ms_per_step,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
           "data": "synthetic", "config": workload}
    out.update(extra)
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2000)
    ap.add_argument("--warmup", type=int, default=200)
    ap.add_argument("--kernel-reps", type=int, default=2000)
    ap.add_argument("--cpu-steps", type=int, default=40)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-extras", action="store_true",
                    help="default workload: leave out the ensemble and adjoint measurements")
    ap.add_argument("--workload", choices=("modelb1024", "ensemble", "adjoint", "3d", "modelh", "mixed", "features"),
                    default="modelb1024",
                    help="modelb1024: one 1024^2 lattice, with the ensemble and adjoint measurements "
                         "(default); ensemble: 256x128^2 + 64x256^2 + 16x512^2 independent lattices in one "
                         "batch, also timed one lattice per launch; adjoint: gradient of the structure-factor "
                         "loss through 2000 steps at 256^2; 3d: the two-field 256^3 system; modelh: 2D "
                         "Model H at 1024^2; mixed: 2D Model B at 960^2 (mixed-radix sizes); features: 1D lines, "
                         "a framed 1024^2 lattice and 2D KPZ")
    ap.add_argument("--autotune", dest="autotune", action="store_true",
                    help="ensemble: pss_autotune's launch geometry per size instead of the default one (a class "
                         "whose tuned geometry does not fit the fused launches then runs launches of its own)")
    ap.add_argument("--ens-steps", type=int, default=200,
                    help="ensemble: steps per timed run of either form")
    ap.add_argument("--copy-mib", type=int, default=0,
                    help="after the run, copy a buffer of this many MiB three times with a plain device "
                         "copy (a known-size reference for hardware byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); the lattice is not sharded.",
              file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2405_02410_amd as pss
    if not torch.cuda.is_available():
        log("no GPU visible")
        sys.exit(1)
    torch.cuda.set_device(0)
    ens_steps = args.ens_steps  # per timed run; both forms replay whole step graphs

    if args.workload == "ensemble":
        e = ensemble(args, pss, torch, ens_steps)
        cpu = None if args.no_cpu else ensemble_cpu_baseline(10)
        cfg = {"workload": "ensemble of 2D Model B lattices, 256x128^2 + 64x256^2 + 16x512^2 FP32, a=-1 b=1 "
                           "k=1, D=0.01 q^2, dt=0.01, 2/3 radial de-aliasing, independent seeds, one batch",
               "members": e["members"], "sites": e["sites"], "parallelism": "single GPU",
               "geometry": e["geometry"]}
        print(json.dumps(line(cfg, e["value"], ens_steps, ens_steps, e["ms_per_step"],
                              {"plain": e["plain"], "vs_plain": e["vs_plain"], "roofline": e["roofline"],
                               "cpu_baseline": cpu})), flush=True)
        return
    if args.workload == "adjoint":
        a = adjoint(args, pss, torch)
        cfg = {"workload": "adjoint of 2D Model B 256x256 FP32 through 2000 steps, checkpoints every 45 "
                           "steps, structure-factor loss, gradients in (a, b, k, D) and phi_0",
               "lattice": [256, 256], "parallelism": "single GPU"}
        print(json.dumps(line(cfg, a["value"], a["steps"], 0, a["ms"] / a["steps"],
                              {"plain": a["plain"], "vs_plain": a["vs_plain"], "cost_vs_plain": a["cost_vs_plain"],
                               "loss": a["loss"], "grad": a["grad"], "roofline": None,
                               "cpu_baseline": None})), flush=True)
        return
    if args.workload == "3d":
        print(json.dumps(three_d(args, pss, torch)), flush=True)
        return
    if args.workload == "modelh":
        h = model_h(args, pss, torch, cpu_steps=0 if args.no_cpu else 3)
        cfg = {"workload": "2D Model H 1024x1024 FP32: phi advected by an incompressible viscous flow driven by "
                           "its interfaces, a=-1 b=1 k=1 M=1 eta=0.5, conserved noise D=0.01 q^2 on phi, "
                           "dt=0.01, 2/3 radial de-aliasing, uniform[-0.4,0.4] initial phi",
               "lattice": [1024, 1024], "parallelism": "single GPU", "geometry": h["geometry"]}
        print(json.dumps(line(cfg, h["value"], h["steps"], h["warmup"], h["ms_per_step"],
                              {"roofline": h["roofline"], "cpu_baseline": h["cpu_baseline"]})), flush=True)
        return

    if args.workload == "features":
        x = features(args, pss, torch)
        cfg = {"workload": "1D Model B lines of 4096 and 3000 points; 2D Model B 1024^2 with a 4-column frame; "
                           "2D KPZ 1024^2 (sigma=1, lam=1, D=0.01); coefficients of the main workload",
               "parallelism": "single GPU"}
        first = x["line_4096"]
        print(json.dumps(line(cfg, first["site_steps_per_s"], first["steps"], 200, first["us_per_step"] * 1e-3,
                              {"features": x, "roofline": None, "cpu_baseline": None})), flush=True)
        return
    if args.workload == "mixed":
        x = mixed_radix(args, pss, torch)
        cfg = {"workload": "2D Model B 960x960 FP32 (960 = 2^6 3 5), a=-1 "
                           "b=1 k=1, conserved noise D=0.01 q^2, dt=0.01, 2/3 radial de-aliasing",
               "lattice": x["lattice"], "parallelism": "single GPU"}
        print(json.dumps(line(cfg, x["value"], x["steps"], min(args.warmup, 20), x["ms_per_step"],
                              {"step_bytes": x["step_bytes"], "step_GBs": x["step_GBs"], "roofline": None,
                               "cpu_baseline": None})), flush=True)
        return

    m = modelb1024(args, pss, torch)
    extras = {}
    if not args.no_extras:
        log(f"bench: ensemble workload, {ens_steps} steps per timed run")
        extras["ensemble"] = ensemble(args, pss, torch, ens_steps)
        log("bench: adjoint workload")
        extras["adjoint"] = adjoint(args, pss, torch)
        log("bench: model h workload")
        h = model_h(args, pss, torch)
        extras["model_h"] = {k: h[k] for k in ("value", "unit", "steps", "ms_per_step", "roofline")}
        log("bench: mixed-radix workload")
        extras["mixed_radix"] = mixed_radix(args, pss, torch)

    if args.copy_mib > 0:
        nbytes = args.copy_mib << 20
        src = torch.ones(nbytes, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        log(f"bench: copied {args.copy_mib} MiB three times")
        del src, dst

    cpu = None
    if not args.no_cpu:
        log(f"bench: timing the oracle on {args.cpu_steps} steps")
        cpu = cpu_baseline(args.cpu_steps)

    cfg = {"workload": "2D Model B 1024x1024 FP32, a=-1 b=1 k=1, conserved noise D=0.01 q^2, "
                       "dt=0.01, 2/3 radial de-aliasing, uniform[-0.1,0.1] initial field, seed 1",
           "lattice": list(N), "parallelism": "single GPU", "geometry": m["geometry"]}
    out = line(cfg, m["value"], args.steps, args.warmup, m["ms_per_step"],
               {"timing": f"median of {REPEATS} runs of {args.steps} steps, HIP events on the lattice stream",
                "runs_ms_per_step": m["runs_ms_per_step"], "roofline": m["roofline"], "cpu_baseline": cpu,
                "mass_after": m["mass_after"]})
    out.update(extras)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
