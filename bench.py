"""Benchmark of the D2Q25 RK-3 step on one MI355X.

Default workload (the metric's configuration): 2048 x 2048 periodic lattice,
FP64, superposed shear and longitudinal waves (wavelength 64 cells), vdW
a = 9/49, b = 2/21, T = 1, tau = 0.005, dt = 5e-4.  A step is one full RK-3
step (three fused stage-kernel launches).  Inputs are resident in HBM before
the timed region starts.

Prints one JSON line with MLUPS (cells x steps / s / 1e6), the roofline of
the stage kernel (its average launch time from HIP events on the library's
stream over the timed region) and the CPU oracle timed on a bounded sample of
the same workload.
"""
import argparse
import hashlib
import re
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X HBM3E, published
FP64_VEC_PEAK_TFLOPS = 78.6  # MI355X vector FP64, published (FMA = 2 flops)
FP32_VEC_PEAK_TFLOPS = 157.3
# VALU issue: a SIMD issues one VALU instruction per quad-cycle (4 cycles, one
# wave64 instruction), or two FP32 add / mul / FMA instructions without
# scalar-register operands in one quad-cycle (SQ_ACTIVE_INST_VALU2 counts
# those quad-cycles; the issue probes of olb_probes measure the forms);
# 256 CUs x 4 SIMDs at the 2.4 GHz peak clock
SIMDS = 256 * 4
PEAK_CLOCK_GHZ = 2.4
VALU_ISSUE_PEAK_GQUAD = SIMDS * PEAK_CLOCK_GHZ / 4
# a kernel whose VALU issue time covers this much of its launch is VALU-bound
VALU_BOUND_FRAC = 0.9

# Algorithmic HBM bytes per cell per RK-3 step: 25 populations x 8 accesses
# (stage 1: read f^n, write f1; stages 2, 3: read f_src and f^n, write).
ALG_VALUES_PER_CELL_STEP = 25 * 8
# FP64/FP32 flops per cell per stage of the stage kernel's formulation
# (counted from its arithmetic; an FMA counts 2): 40 WENO faces x 54, the
# rest (advection differences, force term, BGK, equilibrium, moments, 7x7
# stencils, RK combine) 1710.  See the design notes for the tally.
ALG_FLOPS_PER_CELL_STAGE = 3870


def _code_only(text):
    """Source text without comments and with whitespace collapsed: what the
    compiler sees, so that editing a comment does not orphan a measurement."""
    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    return " ".join(text.split())


def kernel_source_hash():
    h = hashlib.sha256()
    # the runtime file sets the launch configuration (tile order), which the
    # measured bytes depend on too
    for name in ("olb_kernels.hip", "olb_split.hpp", "olb_runtime.hip", "olb_consts.hpp", "olb_device.hpp",
                 "olb_feq.hpp"):
        with open(os.path.join(ROOT, "paper_1702_01690_amd", "csrc", name), encoding="utf-8") as fh:
            h.update(_code_only(fh.read()).encode())
    # and the compiler flags the library is built with
    from paper_1702_01690_amd import build as hip_build
    h.update(" ".join(hip_build.FLAGS[:-2]).encode())
    return h.hexdigest()[:16]


def load_counters(workload):
    """Counter figures per stage launch (HBM bytes, VALU instructions) from
    committed rocprofv3 runs, if they were taken on the current kernel source."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        t = json.load(fh)
    entry = t.get(workload)
    if not entry or entry.get("kernel_hash") != kernel_source_hash():
        return None
    return entry



WORKLOADS = {
    "wave2048": "2048x2048 periodic FP64, shear + longitudinal waves, vdW a=9/49 b=2/21, T=1, "
                "tau=0.005, dt=5e-4, ds=1/64",
    "spinodal4096": "4096x4096 periodic FP32-mixed spinodal decomposition at T=0.9 T_c, "
                    "n=3.5(1+-1% noise), tau=0.005, dt=2e-4, ds=1/320",
    "shard4096x512": "one GPU's share of the 4096x4096 FP32-mixed spinodal split into 8 y-strips: rows "
                     "0..511 of the same field, 4096x512, periodic in y in place of the 3-row halo exchange "
                     "with the neighbouring strips",
    "channels": "256 walled channels (nx 64..512, ny 128..1024, 43.6 M nodes), FP32-mixed, "
                "T_w in [0.7, 0.95] T_c, one launch per stage over all channels, graphs of 10 steps",
    "quench": "phase separation between suddenly cooled plates (Sec. 7): 320x640 FP64 (walls across y), "
              "a=9/8 b=1/3, fluid at T=1 with n = 1 +- 1%, walls at T_w=0.8, ds=1/320, dt=2e-4, tau=5e-3, "
              "sigma=1e-4, to t = 25",
    "planar": "planar interface (Sec. 5): 13 half channels of 1x160 nodes (specular centre plane, diffuse "
              "wall), a=9/8 b=1/3, T_w = 0.74..0.98, ds=1/320, dt=2e-4, tau=5e-3, sigma=1e-4, one batch "
              "in HIP graphs, relaxed to the steady state",
    "galilei": "shear waves seen from a moving frame (Sec. 6.1): ideal gas (n=1) and vdW vapour / liquid "
               "(a=9/8 b=1/3, coexistence densities at T0=0.8), N_x = 20..60 periodic, V = 0..2 step 0.1, "
               "u0=1e-3, tau=5e-4, dt=2e-4; 315 instances in one batch, 2e5 steps, amplitude every 1000 steps; "
               "then the moving bubble (Sec. 6.3, 320x160, V = 0..0.1, to t = 30)",
    "laplace": "Laplace pressure test (Sec. 6): gas bubbles of R0 = 0.15..0.35 in the corner of a 160x160 FP64 "
               "box (specular planes on three sides, diffuse wall at T_w = 0.8), a=9/8 b=1/3, ds=1/320, dt=2e-4, "
               "tau=5e-3, sigma = 5e-5 and 1e-4; 10 instances in one batch, 4e5 steps; planar columns for gamma_pl",
    "precision4096": "4096x4096 periodic spinodal decomposition at T=0.9 T_c (n=3.5(1+-1% noise), seed 3, "
                     "tau=0.005, dt=2e-4, ds=1/320), 5000 RK3 steps in FP32-mixed storage (departure base "
                     "at the state's T) and in FP64, side by side: density error of FP32 against FP64, "
                     "mass drift, structure-factor peak and liquid fraction over time",
    "closure": "learned closure: coarse 512x512 FP32-mixed (ds 1/80, dt 8e-4) corrected every 10 steps "
               "by the bf16 conv net, against fine 2048x2048 FP64 (ds 1/320, dt 2e-4); spinodal at "
               "T in [0.75, 0.95] T_c, n = 3.5(1 +- 1% noise), tau = 0.005; 200 coarse steps",
}
# bf16 dense matrix-core peak of one MI355X
MFMA_BF16_PEAK_TFLOPS = 2500.0
# network flops per node and forward pass: 2 x (36 x 32 + 288 x 32 + 288 x 4) MACs
CLOSURE_FLOPS_PER_NODE = 2 * (36 * 32 + 288 * 32 + 288 * 4)


def make_cases(workload):
    import olb_inputs as I
    if workload == "wave2048":
        c = I.wave2048()
        c.params["precision"] = 0
        return [c]
    if workload == "spinodal4096":
        c = I.spinodal(4096, 4096)
        c.params["precision"] = 1
        c.params["rho_ref"] = I.N_CRIT
        return [c]
    if workload == "shard4096x512":
        # the seeded field is drawn row by row, so these are the first 512
        # rows of the 4096^2 lattice's field
        c = I.spinodal(4096, 512)
        c.params["precision"] = 1
        c.params["rho_ref"] = I.N_CRIT
        return [c]
    if workload == "channels":
        return I.channels()
    raise SystemExit(f"unknown workload {workload}")


def shard_halo_bytes(nx, precision):
    """Bytes a y-strip shard would receive per RK stage: 3 rows of the 25
    populations and of the carried (n, Delta p) from each of its two
    neighbours."""
    rb = 8 if precision == 0 else 4
    return 2 * 3 * nx * (25 * rb + 16)


def cpu_baseline(workload, min_seconds):
    """The oracle, as it stands, on a bounded sample of the workload itself:
    whole instances at their full size (the 2048^2 lattice of the default
    workload; the first channels of the batch), one RK-3 step at a time
    until min_seconds of stepping have passed (at least one step), on all of
    the host's threads; then one thread on a 256^2 lattice of the same
    physics for about min_seconds."""
    import olb_inputs as I
    import oracle
    threads = oracle.get_threads()
    cells_steps, secs, used = 0, 0.0, []
    for case in make_cases(workload):
        o = oracle.Oracle(case.params)
        o.set_fields(*case.fields)
        cells = case.params["nx"] * case.params["ny"]
        steps = 0
        while secs < min_seconds:
            t0 = time.perf_counter()
            o.step(1)
            secs += time.perf_counter() - t0
            steps += 1
            cells_steps += cells
            if case.params.get("bc_y", 0) != 0:
                break                      # channels: one step each, then the next channel
        o.close()
        used.append(f"{case.params['nx']}x{case.params['ny']} x {steps}")
        if secs >= min_seconds:
            break
    full = {"value": cells_steps / secs / 1e6, "unit": "MLUPS", "cores": threads, "kind": "oracle",
            "sample": f"FP64 oracle on full-size instances of the workload ({', '.join(used)} RK3 steps), "
                      f"{secs:.1f} s of stepping on {threads} threads"}
    # one thread on a lattice that does not fit in the caches either
    if workload == "wave2048":
        small = I.tile(I.wave64(), 4, 4)
    elif workload in ("spinodal4096", "shard4096x512"):
        small = I.spinodal(256, 256)
    else:
        small = I.channel(256, 256, tw=0.8 * I.T_CRIT)
    oracle.set_threads(1)
    try:
        o = oracle.Oracle(small.params)
        o.set_fields(*small.fields)
        steps, t1 = 0, 0.0
        while t1 < min_seconds:
            t0 = time.perf_counter()
            o.step(1)
            t1 += time.perf_counter() - t0
            steps += 1
        o.close()
    finally:
        oracle.set_threads(threads)
    cells = small.params["nx"] * small.params["ny"]
    full["one_core"] = {"value": cells * steps / t1 / 1e6, "unit": "MLUPS", "cores": 1,
                        "sample": f"{small.params['nx']}x{small.params['ny']} lattice of the same physics, "
                                  f"{steps} RK3 steps, {t1:.1f} s on 1 thread"}
    return full


def copy_gbps(gib, reps=10):
    """Bandwidth of a plain device-to-device copy of gib GiB (bytes read plus
    bytes written per second), the best a streaming kernel does on this GPU."""
    import torch
    n = int(gib * (1 << 30)) // 8
    a = torch.ones(n, dtype=torch.float64, device="cuda:0")
    b = torch.empty_like(a)
    b.copy_(a)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        b.copy_(a)
    e1.record()
    torch.cuda.synchronize()
    secs = e0.elapsed_time(e1) / 1e3 / reps
    del a, b
    torch.cuda.empty_cache()
    return n * 8, 2 * n * 8 / secs / 1e9


def stream_ceilings():
    """Best copy, read-only and write-only bandwidth of `olb_probes stream`
    (16-byte accesses over 2 GiB buffers, run as a child process), or None
    when the program is not built or fails."""
    import subprocess
    exe = os.path.join(ROOT, "paper_1702_01690_amd", "olb_probes")
    if not os.path.exists(exe):
        return None
    try:
        r = subprocess.run([exe, "stream"], capture_output=True, text=True, timeout=120)
    except subprocess.TimeoutExpired:
        return None
    if r.returncode != 0:
        return None
    for line in reversed(r.stdout.splitlines()):
        d = json.loads(line)
        if "best" in d:
            return d["best"]
    return None


def copy_kernel(gib, reps=10):
    """Device-to-device copy of a known size: calibrates the HBM byte
    counters (FETCH_SIZE / WRITE_SIZE per dispatch) and measures the copy
    bandwidth this GPU sustains."""
    nbytes, gbps = copy_gbps(gib, reps)
    print(json.dumps({"copy_bytes_read": nbytes, "copy_bytes_written": nbytes,
                      "copy_GBps": round(gbps, 1), "reps": reps}))


def run_quench(args):
    """The cooled-plates quench to t = 25, timed, with the checks of the
    paper's description at t = 2.5, 5, 10, 12.5 and 25."""
    import torch
    import olb_inputs as I
    from paper_1702_01690_amd import olb, phase

    c = I.quench()
    tw, dt = c.params["tw_lo"], c.params["dt"]
    lat = olb.Lattice(c.params, device="cuda:0")
    lat.set_fields(*c.fields)
    m0 = float(c.n.sum())
    _, n_liq = phase.maxwell_coexistence(tw)
    snaps, done, secs = [], 0, 0.0
    for t in (2.5, 5.0, 10.0, 12.5, 25.0):
        k = int(round(t / dt)) - done
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ev0.record(lat.stream)
        lat.step(k)
        ev1.record(lat.stream)
        lat.sync()
        secs += ev0.elapsed_time(ev1) / 1e3
        done += k
        n, ux, uy, T = lat.moments()
        ny = n.shape[0]
        pn, pT = n.mean(axis=1), T.mean(axis=1)
        snaps.append({"t": t, "mass_drift": float((n.sum() - m0) / m0),
                      "wall_film_n": float(0.5 * (pn[:5].mean() + pn[-5:].mean())),
                      "centre_T": float(pT[ny // 2 - 5: ny // 2 + 5].mean()), "mean_T": float(T.mean()),
                      "hottest_row_from_wall": int(min(np.argmax(pT[: ny // 2]),
                                                       np.argmax(pT[ny // 2:][::-1]))),
                      "n_min": float(n.min()), "n_max": float(n.max()),
                      "max_speed": float(np.hypot(ux, uy).max())})
        print(f"[bench] {snaps[-1]}", file=sys.stderr, flush=True)
    cells = c.params["nx"] * c.params["ny"]
    mlups = cells * done / secs / 1e6
    achieved = ALG_VALUES_PER_CELL_STEP * 8 * cells * done / secs / 1e9
    out = {
        "metric": "MLUPS per full RK3 step (D2Q25)",
        "value": round(mlups, 2), "unit": "MLUPS", "n_gpus": 1, "steps": done, "warmup": 0,
        "ms_per_step": round(secs / done * 1e3, 5), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "quench", "description": WORKLOADS["quench"], "nodes": cells,
                   "maxwell_liquid_density": n_liq, "snapshots": snaps,
                   "timed": "stepping only (read-outs between snapshots excluded)"},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None},
        "cpu_baseline": None,
    }
    print(json.dumps(out))


def _moving_bubble(log):
    """Sec. 6.3: half bubbles (R0 = 0.25, sigma = 1e-4) carried with V = 0 ..
    0.1 along the specular plane and a moving diffuse wall, to t = 30; the
    Laplace-law surface tension against the bubble at rest and the lag of
    the centre behind V t."""
    import olb_inputs as I
    from paper_1702_01690_amd import galilei as G, olb, phase

    ng, nl = phase.maxwell_coexistence(0.8)
    speeds = [0.0, 0.01, 0.02, 0.05, 0.1]
    cases = [I.moving_bubble(V, ng, nl) for V in speeds]
    b = olb.Batch([c.params for c in cases], device="cuda:0")
    b.use_graph(10)
    for i, c in enumerate(cases):
        b.set_fields(i, *c.fields)
    eps = {V: [] for V in speeds[1:]}
    lag = {}
    for s in range(1, 16):                               # t = 2, 4, ..., 30
        b.step(10000)
        t = 2.0 * s
        track = []
        for i, (V, c) in enumerate(zip(speeds, cases)):
            n, _, _, T = b.moments(i)
            track.append(phase.track_bubble(n, T, c.extra["x"], c.extra["y"], V * t, c.extra["R0"],
                                            c.extra["xi"], 1.0))
        g0 = track[0][1] * track[0][3]
        for V, tr in zip(speeds[1:], track[1:]):
            if t >= 20.0:
                eps[V].append(abs(tr[1] * tr[3] / g0 - 1.0))
            lag[V] = tr[0] - V * t
    b.close()
    mean = {str(V): float(np.mean(eps[V])) for V in speeds[1:]}
    big = speeds[2:]                                     # V = 0.01 sits at the noise floor of the fit
    out = {"mean_eps_gamma_20_30": mean, "eps_gamma_max": float(max(max(e) for e in eps.values())),
           "exponent_b_from_V_0.02_0.1": G.order(big, [mean[str(V)] for V in big]),
           "lag_at_t30": {str(V): lag[V] for V in speeds[1:]},
           "lag_exponent": G.order(speeds[1:], [-lag[V] for V in speeds[1:]])}
    log(f"moving bubble: {out}")
    return out


def run_galilei(args):
    """The Galilean shear-wave sweep behind the paper's two exponent tables:
    every (medium, N_x, V) run as one instance of a batch; the exponents of
    dx and of V from the sampled amplitudes."""
    import olb_inputs as I
    from paper_1702_01690_amd import galilei as G, phase

    def log(msg):
        print(f"[bench] {msg}", file=sys.stderr, flush=True)

    T0, tau, dt, u0 = 0.8, 5e-4, 2e-4, 1e-3
    ng, nl = phase.maxwell_coexistence(T0)
    media = {"ideal": (1.0, 0.0, 0.0, 0.0), "vapour": (ng, 9 / 8, 1 / 3, 1e-4),
             "liquid": (nl, 9 / 8, 1 / 3, 1e-4)}
    sizes = (20, 30, 40, 50, 60)
    speeds = tuple(round(0.1 * i, 1) for i in range(21))
    keys = [(m, N, V) for m in media for N in sizes for V in speeds]
    cases = [I.shear_wave(N, V, *media[m], T0=T0, tau=tau, dt=dt, u0=u0) for m, N, V in keys]
    log(f"galilei: {len(cases)} instances")
    t0 = time.perf_counter()
    times, amps, secs = G.sweep(cases, samples=200, every=1000, graph=args.graph or 10, log=log)
    wall = time.perf_counter() - t0
    res = {k: (G.viscosity_ratio(a, times, u0, tau, T0), G.l2_norm(a, times, u0, tau, T0))
           for k, a in zip(keys, amps)}
    dx, vv = G.orders(res, tuple(media), sizes)
    bubble = _moving_bubble(log)
    steps = 200 * 1000
    cells = sum(N for _, N, _ in keys)
    mlups = cells * steps / secs / 1e6
    achieved = ALG_VALUES_PER_CELL_STEP * 8 * cells * steps / secs / 1e9
    out = {
        "metric": "MLUPS per full RK3 step (D2Q25)",
        "value": round(mlups, 3), "unit": "MLUPS", "n_gpus": 1, "steps": steps, "warmup": 0,
        "ms_per_step": round(secs / steps * 1e3, 5), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "galilei", "description": WORKLOADS["galilei"], "nodes": cells,
                   "instances": len(cases), "wall_s": round(wall, 2),
                   "timed": "stepping only (amplitude read-outs excluded)",
                   "dx_orders": {m: {str(V): [round(x, 6) for x in v] for V, v in dx[m].items()} for m in dx},
                   "v_orders": {m: {str(N): [round(x, 6) for x in v] for N, v in vv[m].items()} for m in vv},
                   "moving_bubble": bubble,
                   "note": "1 x N_x lattices, each held in one workgroup for whole steps: the step time is "
                           "the chain of one stage, not bandwidth"},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 3), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 7), "traffic": None},
        "cpu_baseline": None,
    }
    print(json.dumps(out))


def run_laplace(args):
    """The Laplace pressure test: bubbles of five radii for two surface-
    tension parameters in one batch; gamma_Lap from p_in - p_out against
    1 / R_f, gamma_pl from planar interfaces of the same parameters."""
    import torch
    import olb_inputs as I
    from paper_1702_01690_amd import olb, phase

    def log(msg):
        print(f"[bench] {msg}", file=sys.stderr, flush=True)

    tw, steps = 0.8, args.laplace_steps
    ng, nl = phase.maxwell_coexistence(tw)
    radii, sigmas = [0.15, 0.2, 0.25, 0.3, 0.35], [5e-5, 1e-4]
    cases = [I.laplace_bubble(R, ng, nl, sigma=s, tw=tw) for s in sigmas for R in radii]
    planar = [I.planar_interface(tw, ng, nl, sigma=s) for s in sigmas]
    b = olb.Batch([c.params for c in cases], device="cuda:0")
    b.use_graph(10)
    for i, c in enumerate(cases):
        b.set_fields(i, *c.fields)
    q = olb.Batch([c.params for c in planar], device="cuda:0")
    q.use_graph(10)
    for i, c in enumerate(planar):
        q.set_fields(i, *c.fields)
    m0 = [float(c.n.sum()) for c in cases]
    torch.cuda.synchronize()
    secs, done = 0.0, 0
    while done < steps:
        k = min(50000, steps - done)
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ev0.record(b.stream)
        b.step(k)
        ev1.record(b.stream)
        q.step(k)
        b.sync()
        q.sync()
        secs += ev0.elapsed_time(ev1) / 1e3
        done += k
        log(f"{done} steps")
    rows, table = [], {}
    ds = cases[0].params["ds"]
    for si, s in enumerate(sigmas):
        rf_list, dp_list = [], []
        for j, R0 in enumerate(radii):
            i = si * len(radii) + j
            n, ux, uy, T = b.moments(i)
            xiw = cases[i].extra["xi"]
            rf, xi, nin, nout = phase.bubble_profile(n, ds, R0, xiw)
            pin, pout = phase.bubble_pressures(n, T, ds, rf, xi)
            rf_list.append(rf)
            dp_list.append(pin - pout)
            rows.append({"sigma": s, "R0": R0, "R_f": rf, "xi_over_xi_w": xi / xiw, "n_in": nin, "n_out": nout,
                         "p_in_minus_p_out": pin - pout, "max_u": float(np.hypot(ux, uy).max()),
                         "mass_drift": float(n.sum() / m0[i] - 1.0)})
        gl = phase.laplace_tension(rf_list, dp_list)
        gp = phase.surface_tension(q.moments(si)[0], planar[si].params["ds"], s)
        table[str(s)] = {"gamma_lap": gl, "gamma_pl": gp, "gamma_lap_over_gamma_pl_minus_1": gl / gp - 1.0}
        log(f"sigma {s}: gamma_Lap {gl:.6e}, gamma_pl {gp:.6e}, ratio - 1 {gl / gp - 1.0:+.4f}")
    cells = sum(c.params["nx"] * c.params["ny"] for c in cases)
    mlups = cells * steps / secs / 1e6
    achieved = ALG_VALUES_PER_CELL_STEP * 8 * cells * steps / secs / 1e9
    b.close()
    q.close()
    out = {
        "metric": "MLUPS per full RK3 step (D2Q25)",
        "value": round(mlups, 2), "unit": "MLUPS", "n_gpus": 1, "steps": steps, "warmup": 0,
        "ms_per_step": round(secs / steps * 1e3, 5), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "laplace", "description": WORKLOADS["laplace"], "nodes": cells,
                   "instances": len(cases), "bubbles": rows, "surface_tension": table,
                   "timed": "bubble batch stepping only (planar columns and read-outs excluded)"},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 5), "traffic": None},
        "cpu_baseline": None,
    }
    print(json.dumps(out))


def run_planar(args):
    """Phase diagram of the solver: a batch of half channels, one per wall
    temperature, relaxed to the steady state; coexistence densities against
    the Maxwell construction, spurious velocity and heating."""
    import torch
    import olb_inputs as I
    from paper_1702_01690_amd import olb, phase

    def log(msg):
        print(f"[bench] {msg}", file=sys.stderr, flush=True)

    temps = [round(0.74 + 0.02 * i, 2) for i in range(13)]
    maxwell = [phase.maxwell_coexistence(t) for t in temps]
    cases = [I.planar_interface(t, ng, nl) for t, (ng, nl) in zip(temps, maxwell)]
    b = olb.Batch([c.params for c in cases], device="cuda:0")
    b.use_graph(10)
    for i, c in enumerate(cases):
        b.set_fields(i, *c.fields)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    ev0.record(b.stream)
    steps, change = phase.relax(b, chunk=20000, rtol=1e-7, max_steps=args.planar_steps, log=log)
    ev1.record(b.stream)
    b.sync()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    secs = ev0.elapsed_time(ev1) / 1e3
    cells = sum(c.params["nx"] * c.params["ny"] for c in cases)
    rows = []
    for i, t in enumerate(temps):
        m = b.moments(i)
        ng, nl = phase.coexistence(m[0])
        u, dT = phase.spurious(m, t)
        gam = phase.surface_tension(m[0], cases[i].params["ds"], cases[i].params["sigma"])
        xiw = np.sqrt(8.0 * cases[i].params["sigma"] / (9.0 * (1.0 - t)))
        xi, _ = phase.interface_width(m[0], cases[i].params["ds"], 0.25, xiw)
        rows.append({"T_w": t, "n_g": ng, "n_l": nl,
                     "n_g_vs_maxwell": (ng - maxwell[i][0]) / maxwell[i][0],
                     "n_l_vs_maxwell": (nl - maxwell[i][1]) / maxwell[i][1],
                     "max_u": u, "max_T_minus_Tw": dT, "gamma_pl": gam, "xi_over_xi_w": xi / xiw})
        log(f"T_w {t}: n_g {ng:.7f} ({rows[-1]['n_g_vs_maxwell']:+.2e}), n_l {nl:.7f} "
            f"({rows[-1]['n_l_vs_maxwell']:+.2e}), |u| {u:.2e}, dT {dT:.2e}, gamma_pl {gam:.7e}")
    mlups = cells * steps / secs / 1e6
    launch_s = secs / (3 * steps)
    achieved = ALG_VALUES_PER_CELL_STEP * 8 * cells / 3 / launch_s / 1e9
    out = {
        "metric": "MLUPS per full RK3 step (D2Q25)",
        "value": round(mlups, 3),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": steps,
        "warmup": 0,
        "ms_per_step": round(secs / steps * 1e3, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": "planar", "description": WORKLOADS["planar"], "nodes": cells,
                   "instances": len(cases), "final_relative_change_per_20000_steps": change,
                   "wall_s": round(wall, 2), "phase_diagram": rows,
                   "note": "1-D columns of 160 nodes, each held in one workgroup for whole steps: the step "
                           "time is the chain of one stage, not bandwidth"},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 3), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 7), "traffic": None},
        "cpu_baseline": None,
    }
    print(json.dumps(out))


def run_closure(args):
    """Learned-closure workload: trains the network on the GPU from solver
    pairs (fine 512^2 -> coarse 128^2; the network is local, so its weights
    carry over to any lattice size), then runs the 2048^2 / 512^2 pair."""
    import torch
    import olb_inputs as I
    from paper_1702_01690_amd import olb, closure as C

    def log(msg):
        print(f"[bench] {msg}", file=sys.stderr, flush=True)

    nf_train, nf, factor, window, horizon = 512, 2048, 4, 10, 200
    samples = []
    for seed in range(5000, 5000 + args.closure_samples):
        s = I.closure_sample(nf_train, seed=seed)
        samples.append((s.params, s.fields))
    small = olb.Closure(nf_train // factor, nf_train // factor)
    t0 = time.perf_counter()
    info = C.train_closure(samples, I.coarse_params, small, windows=args.closure_windows, window=window,
                           epochs=args.closure_epochs, rounds=args.closure_rounds,
                           round_epochs=max(1, args.closure_epochs // 2),
                           init_params=I.closure_params(seed=7), seed=1, log=log)
    t_train = time.perf_counter() - t0
    del samples
    log(f"trained on {info['pairs']} pairs in {t_train:.1f} s")

    seeds = [int(v) for v in args.closure_held_seeds.split(",")]
    net = olb.Closure(nf // factor, nf // factor)
    net.set_norm(*info["norm"])
    net.set_params(small.get_params())
    # per-window errors on every held-out sample; the free runs and the
    # timing on the first
    per_sample = []
    for k, seed in enumerate(seeds):
        held = I.closure_sample(nf, seed=seed)
        cp = I.coarse_params(held.params)
        refs_k = C.fine_references(held.params, held.fields, cp, horizon // window, window, factor)
        pw, fw = C.window_errors(refs_k, cp, net, window)
        per_sample.append((seed, pw, fw))
        log(f"held-out sample {seed}: per-window mean max plain {np.mean([m for m, _ in pw]):.3e}, "
            f"closure {np.mean([m for m, _ in fw]):.3e}")
        if k == 0:
            first, refs, plain_w, fixed_w = held, refs_k, pw, fw
        else:
            del refs_k
    held = first
    cp = I.coarse_params(held.params)
    roll_p, _ = C.rollout_errors(refs, cp, None, window)
    roll_f, skipped = C.rollout_errors(refs, cp, net, window)
    log("free run max/rms per window, plain:   " + " ".join(f"{a:.2e}/{b:.1e}" for a, b in roll_p))
    log("free run max/rms per window, closure: " + " ".join(f"{a:.2e}/{b:.1e}" for a, b in roll_f))

    t_fine, t_closure = C.timing(held.params, held.fields, cp, net, horizon, window, factor)
    _, t_plain = C.timing(held.params, held.fields, cp, None, horizon, window, factor)

    # the network's forward pass, timed with events on the closure's stream
    P = (nf // factor) ** 2
    X = refs[1].clone()
    delta = torch.empty_like(X)
    net.forward(X, delta)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    reps = 50
    ev0.record(net.stream)
    for _ in range(reps):
        net.forward(X, delta)
    ev1.record(net.stream)
    torch.cuda.synchronize()
    fwd_s = ev0.elapsed_time(ev1) / 1e3 / reps
    fwd_tflops = CLOSURE_FLOPS_PER_NODE * P / fwd_s / 1e12

    fine_updates = nf * nf * horizon * factor
    mean = lambda xs: float(np.mean(xs))
    out = {
        "metric": "MLUPS per full RK3 step (D2Q25)",
        "value": round(fine_updates / t_closure / 1e6, 2),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": horizon,
        "warmup": 2,
        "ms_per_step": round(t_closure / horizon * 1e3, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32+f64 solver, bf16 net",
        "data": "synthetic",
        "config": {"workload": "closure", "description": WORKLOADS["closure"],
                   "value_is": "fine-lattice-equivalent updates per second (2048^2 x 4 fine steps per coarse step)",
                   "fine_fp64_mlups": round(fine_updates / t_fine / 1e6, 2),
                   "speedup_vs_fine_fp64": round(t_fine / t_closure, 2),
                   "speedup_plain_coarse": round(t_fine / t_plain, 2),
                   "training": {"pairs": info["pairs"], "seconds": round(t_train, 1),
                                "loss_first_last": [info["history"][0][0], info["history"][-1][-1]]},
                   "density_error_vs_fine": {
                       "held_out_seeds": seeds,
                       "per_window_mean_max_by_sample": [[mean([m for m, _ in pw]), mean([m for m, _ in fw])]
                                                         for _, pw, fw in per_sample],
                       "per_window_mean_max_over_samples": [mean([mean([m for m, _ in pw]) for _, pw, _ in per_sample]),
                                                            mean([mean([m for m, _ in fw]) for _, _, fw in per_sample])],
                       "per_window_mean_max": [mean([m for m, _ in plain_w]), mean([m for m, _ in fixed_w])],
                       "per_window_mean_rms": [mean([r for _, r in plain_w]), mean([r for _, r in fixed_w])],
                       "free_run_first_window_max": [roll_p[0][0], roll_f[0][0]],
                       "free_run_end_max": [roll_p[-1][0], roll_f[-1][0]],
                       "free_run_end_rms": [roll_p[-1][1], roll_f[-1][1]],
                       "free_run_by_window": {"coarse_steps": [window * (j + 1) for j in range(len(roll_p))],
                                              "plain_max": [a for a, _ in roll_p],
                                              "closure_max": [a for a, _ in roll_f],
                                              "plain_rms": [b for _, b in roll_p],
                                              "closure_rms": [b for _, b in roll_f]},
                       "order": "[plain coarse, coarse + closure]", "skipped_nodes": skipped}},
        "roofline": {"bound": "mfma", "kernel": "network forward (fused: persistent workgroups over 16x16 "
                               "tiles, three bf16 implicit-GEMM convolutions in LDS, plus the projection)",
                     "achieved": round(fwd_tflops, 2), "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                     "frac": round(fwd_tflops / MFMA_BF16_PEAK_TFLOPS, 5), "traffic": None,
                     "forward_ms": round(fwd_s * 1e3, 4)},
        "cpu_baseline": None,
    }
    print(json.dumps(out))


def spinodal_stats(n):
    """Statistics of a phase-separating density field that stay meaningful
    when two runs decorrelate pointwise: the first moment of the radially
    binned structure factor S(k) = |FFT(n - <n>)|^2 / N (k in units of
    2 pi / L), the wavenumber of its largest bin, the liquid fraction (nodes
    above the critical density) and the density spread."""
    import olb_inputs as I
    ny, nx = n.shape
    d = n - n.mean()
    S = np.abs(np.fft.rfft2(d)) ** 2 / d.size
    ky = np.fft.fftfreq(ny, 1.0 / ny)[:, None]
    kx = np.arange(S.shape[1])[None, :]
    k = np.sqrt(kx * kx + ky * ky)
    w = np.full(S.shape[1], 2.0)          # rfft columns stand for +-kx
    w[0] = 1.0
    if nx % 2 == 0:
        w[-1] = 1.0
    Sw = S * w[None, :]
    mask = k > 0
    k1 = float((k * Sw)[mask].sum() / Sw[mask].sum())
    kb = np.rint(k).astype(np.int64)
    tot = np.bincount(kb.ravel(), Sw.ravel())
    cnt = np.bincount(kb.ravel(), np.broadcast_to(w[None, :], S.shape).ravel())
    prof = tot[1:] / np.maximum(cnt[1:], 1)
    return {"k1": k1, "k_peak": int(np.argmax(prof) + 1), "liquid_fraction": float((n > I.N_CRIT).mean()),
            "n_std": float(d.std()), "n_min": float(n.min()), "n_max": float(n.max())}


def run_precision(args):
    """The 4096^2 spinodal of the FP32-mixed workload advanced to its full
    horizon in FP32-mixed storage and in FP64 from the same input: the
    density error of FP32 against the FP64 run, both runs' mass drift, and
    statistics that survive the pointwise decorrelation of a chaotic
    coarsening (structure factor, liquid fraction), at checkpoints; then the
    speeds of the two forms on the same lattice.  A third run, FP64 from the
    inputs rounded to FP32, gives the error that rounding the state once
    produces by itself (the condition of the problem)."""
    import torch
    import olb_inputs as I
    from paper_1702_01690_amd import olb

    def log(msg):
        print(f"[bench] {msg}", file=sys.stderr, flush=True)

    c = I.spinodal(4096, 4096)
    p64 = dict(c.params, precision=0)
    p32 = dict(c.params, precision=1, rho_ref=I.N_CRIT)
    l64 = olb.Lattice(p64, device="cuda:0")
    l32 = olb.Lattice(p32, device="cuda:0")
    # the condition of the problem: FP64 from the inputs rounded to FP32
    lrd = olb.Lattice(p64, device="cuda:0")
    l32.set_base_temperature(float(np.mean(c.T)))
    l64.set_fields(*c.fields)
    l32.set_fields(*c.fields)
    r32 = lambda a: a.astype(np.float32).astype(np.float64)
    lrd.set_fields(*(r32(a) for a in c.fields))
    m0 = float(c.n.sum())
    checkpoints = [int(s) for s in args.precision_checkpoints.split(",")]
    rows, done, secs = [], 0, {"fp64": 0.0, "fp32": 0.0}

    def errors(a, ref):
        e = np.abs(a - ref) / np.abs(ref)
        return float(e.max()), float(np.sqrt(np.mean(e * e))), float(np.quantile(e, 0.999))

    for target in checkpoints:
        k = target - done
        for name, lat in (("fp64", l64), ("fp32", l32), ("rounded", lrd)):
            ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            ev0.record(lat.stream)
            lat.step(k)
            ev1.record(lat.stream)
            lat.sync()
            if name in secs:
                secs[name] += ev0.elapsed_time(ev1) / 1e3
        done = target
        n64 = l64.moments()[0]
        n32 = l32.moments()[0]
        nrd = lrd.moments()[0]
        emax, erms, e999 = errors(n32, n64)
        smax, srms, s999 = errors(nrd, n64)
        row = {"step": done, "t": done * c.params["dt"],
               "n_max_rel_err": emax, "n_rms_rel_err": erms, "n_q999_rel_err": e999,
               "fp64_from_fp32_inputs": {"n_max_rel_err": smax, "n_rms_rel_err": srms, "n_q999_rel_err": s999},
               "mass_drift_fp64": float((n64.sum() - m0) / m0), "mass_drift_fp32": float((n32.sum() - m0) / m0),
               "fp64": spinodal_stats(n64), "fp32": spinodal_stats(n32)}
        rows.append(row)
        log(json.dumps(row))
    cells = c.params["nx"] * c.params["ny"]
    ml = {name: cells * done / s / 1e6 for name, s in secs.items()}
    l64.close()
    l32.close()
    lrd.close()
    out = {
        "metric": "MLUPS per full RK3 step (D2Q25)",
        "value": round(ml["fp32"], 2), "unit": "MLUPS", "n_gpus": 1, "steps": done, "warmup": 0,
        "ms_per_step": round(secs["fp32"] / done * 1e3, 4), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32+f64", "data": "synthetic",
        "config": {"workload": "precision4096", "description": WORKLOADS["precision4096"], "nodes": cells,
                   "mlups": {k: round(v, 1) for k, v in ml.items()},
                   "speedup_fp32_over_fp64": round(ml["fp32"] / ml["fp64"], 3),
                   "timed": "stepping only, both forms over the whole horizon (read-outs excluded)",
                   "checkpoints": rows},
        "roofline": None,
        "cpu_baseline": None,
    }
    print(json.dumps(out))


class _Sequential:
    """Single-instance lattices stepped one after another (same stream)."""

    def __init__(self, lats):
        self.lats = lats
        self.stream = lats[0].stream

    def step(self, n):
        for one in self.lats:
            one.step(n)

    def sync(self):
        for one in self.lats:
            one.sync()

    def close(self):
        for one in self.lats:
            one.close()


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="wave2048", choices=sorted(WORKLOADS))
    ap.add_argument("--graph", type=int, default=10, help="RK3 steps per HIP graph (batches)")
    ap.add_argument("--autotune", action="store_true", help="pick the tile height by trial (batches)")
    ap.add_argument("--tile", type=int, default=None, choices=[8, 12, 16],
                    help="the stage kernel at this tile height (default: the kernel the library takes by itself)")
    ap.add_argument("--strip", type=int, default=None, help="tile order: strip width in tiles (0 = rows)")
    ap.add_argument("--cpu-seconds", type=float, default=10.0,
                    help="stepping time of each CPU-baseline leg (the oracle on all threads, then one)")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--precision", default="auto", choices=["auto", "fp64", "fp32"],
                    help="override the workload's storage precision (speedup comparisons)")
    ap.add_argument("--sequential", action="store_true",
                    help="batched workload: step the instances as separate lattices, one after another")
    ap.add_argument("--planar-steps", type=int, default=600000,
                    help="step limit of the planar-interface relaxation")
    ap.add_argument("--laplace-steps", type=int, default=400000,
                    help="steps of the Laplace bubbles (sigma = 1e-4 settles by ~3e5)")
    ap.add_argument("--closure-samples", type=int, default=64,
                    help="training trajectories of the closure workload (8 pairs each)")
    ap.add_argument("--closure-epochs", type=int, default=30)
    ap.add_argument("--closure-windows", type=int, default=8,
                    help="windows of 10 coarse steps per training trajectory")
    ap.add_argument("--closure-rounds", type=int, default=1,
                    help="data-aggregation rounds after the nudged pairs")
    ap.add_argument("--closure-held-seeds", default="6000,6001,6002,6003",
                    help="held-out 2048^2 samples the closure is evaluated on (the first also "
                         "gives the free runs and the timing)")
    ap.add_argument("--precision-checkpoints", default="20,100,250,500,1000,2000,3000,4000,5000",
                    help="steps at which the precision4096 workload compares FP32 with FP64")
    ap.add_argument("--copy-gib", type=float, default=0.0,
                    help="only run a device copy of this many GiB (counter calibration)")
    args = ap.parse_args()
    if args.copy_gib > 0:
        copy_kernel(args.copy_gib)
        return
    if args.gpus != 1:
        print("bench.py: the stage kernels run on one GPU; --gpus above 1 is not supported "
              "(the lattice would shard into y-strips with a 3-row halo exchange per stage)",
              file=sys.stderr)
        sys.exit(2)

    if args.workload == "closure":
        run_closure(args)
        return
    if args.workload == "planar":
        run_planar(args)
        return
    if args.workload == "quench":
        run_quench(args)
        return
    if args.workload == "galilei":
        run_galilei(args)
        return
    if args.workload == "laplace":
        run_laplace(args)
        return
    if args.workload == "precision4096":
        run_precision(args)
        return

    import torch
    from paper_1702_01690_amd import olb

    cases = make_cases(args.workload)
    if args.precision != "auto":
        import olb_inputs as I
        for c in cases:
            c.params["precision"] = 0 if args.precision == "fp64" else 1
            c.params["rho_ref"] = I.N_CRIT if args.workload != "wave2048" else 1.0
    precision = cases[0].params["precision"]
    batched = args.workload == "channels"
    if args.sequential and not batched:
        raise SystemExit("--sequential applies to the batched workload")
    cells = sum(c.params["nx"] * c.params["ny"] for c in cases)
    print(f"[bench] {args.workload} instances={len(cases)} nodes={cells} precision={precision} "
          f"warmup={args.warmup} steps={args.steps}", file=sys.stderr, flush=True)
    if batched and args.sequential:
        # the same instances as separate lattices stepped one after another on
        # one stream: the method without the batched launch
        lat = _Sequential([olb.Lattice(c.params, device="cuda:0") for c in cases])
        for one, c in zip(lat.lats, cases):
            if args.tile:
                one.set_tile(args.tile)
            one.set_base_temperature(float(np.mean(c.T)))   # FP32 departure base (no-op in FP64)
            one.set_fields(*c.fields)
        n_stage, n_walls = 3, 3
    elif batched:
        lat = olb.Batch([c.params for c in cases], device="cuda:0")
        if args.autotune:
            lat.autotune(trial_steps=2)
        elif args.tile:
            lat.set_tile(args.tile)
        if args.graph:
            lat.use_graph(args.graph)
        for i, c in enumerate(cases):
            lat.set_base_temperature(i, float(np.mean(c.T)))
            lat.set_fields(i, *c.fields)
        n_stage, n_walls = 3, 3
    else:
        lat = olb.Lattice(cases[0].params, device="cuda:0")
        if args.tile:
            lat.set_tile(args.tile)
        if args.strip is not None:
            lat.set_tile_order(args.strip)
        lat.set_base_temperature(float(np.mean(cases[0].T)))
        lat.set_fields(*cases[0].fields)
        n_stage, n_walls = lat.launch_counts()
    if args.tile:
        tile = f"63x{args.tile}"
    elif args.autotune and batched:
        tile = f"autotuned, {lat.tiles()[1]} rows"
    else:
        tile = "default"
    stream = lat.stream

    lat.step(args.warmup)
    lat.sync()
    torch.cuda.synchronize()
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    ev0.record(stream)
    lat.step(args.steps)
    ev1.record(stream)
    lat.sync()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms_events = ev0.elapsed_time(ev1)
    secs = ms_events / 1e3
    mlups = cells * args.steps / secs / 1e6
    launches = n_stage * args.steps
    # the region holds the stage launches (and, with walls, the small ghost launches)
    avg_launch_s = secs / launches
    rb = 8 if precision == 0 else 4
    bytes_per_launch = ALG_VALUES_PER_CELL_STEP * rb * cells / n_stage
    achieved_gbs = bytes_per_launch / avg_launch_s / 1e9
    flops_per_launch = ALG_FLOPS_PER_CELL_STAGE * cells
    achieved_tflops = flops_per_launch / avg_launch_s / 1e12
    vec_peak = FP64_VEC_PEAK_TFLOPS if precision == 0 else FP32_VEC_PEAK_TFLOPS
    hbm_frac = achieved_gbs / HBM_PEAK_GBS
    alu_frac = achieved_tflops / vec_peak
    counters = load_counters(args.workload) if args.precision == "auto" and not args.sequential else None
    traffic = counters.get("bytes_per_launch") if counters else None
    valu = None
    if counters and "valu" in counters:
        v = counters["valu"]
        # issue quad-cycles summed over the SIMDs: one per instruction, less
        # one per quad-cycle that carried two
        quads = v["insts_per_launch"] - v["dual_issue_quads_per_launch"]
        issue_gquad = quads / avg_launch_s / 1e9
        cycles_per_simd = 4.0 * quads / SIMDS
        valu = {"insts_per_launch": v["insts_per_launch"],
                "dual_issue_quads_per_launch": v["dual_issue_quads_per_launch"],
                "issue_gquad_s": round(issue_gquad, 1), "issue_peak_gquad_s": VALU_ISSUE_PEAK_GQUAD,
                # share of this launch the SIMDs would spend issuing VALU work at the peak clock
                "issue_frac": round(issue_gquad / VALU_ISSUE_PEAK_GQUAD, 4),
                # the clock the profiled launches ran at (GRBM_GUI_ACTIVE per XCD over the
                # dispatch time) and the issue share of their cycles at that clock
                "profiled_clock_ghz": v["clock_ghz"],
                "issue_frac_of_profiled_cycles": round(cycles_per_simd / v["gui_cycles_per_xcd"], 4),
                "f64_tflops": round(v["f64_flops_per_launch"] / avg_launch_s / 1e12, 3),
                "f32_tflops": round(v["f32_flops_per_launch"] / avg_launch_s / 1e12, 3),
                "source": v["source"]}
    if valu and valu["issue_frac"] >= VALU_BOUND_FRAC:
        # VALU-bound: the issue rate against its peak
        roof = {"bound": "alu", "achieved": valu["issue_gquad_s"], "peak": VALU_ISSUE_PEAK_GQUAD,
                "unit": "G issue quad-cycles/s (VALU, all SIMDs)", "frac": valu["issue_frac"], "traffic": traffic,
                "hbm": {"achieved": round(achieved_gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": round(hbm_frac, 4)},
                "flops": {"achieved": round(achieved_tflops, 3), "peak": vec_peak, "unit": "TFLOP/s",
                          "frac": round(alu_frac, 4)}}
    elif alu_frac >= hbm_frac:
        roof = {"bound": "alu", "achieved": round(achieved_tflops, 3), "peak": vec_peak,
                "unit": "TFLOP/s", "frac": round(alu_frac, 4), "traffic": traffic,
                "hbm": {"achieved": round(achieved_gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                        "frac": round(hbm_frac, 4)}}
    else:
        roof = {"bound": "hbm", "achieved": round(achieved_gbs, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(hbm_frac, 4), "traffic": traffic,
                "alu": {"achieved": round(achieved_tflops, 3), "peak": vec_peak, "unit": "TFLOP/s",
                        "frac": round(alu_frac, 4)}}
    lat.close()
    # the streaming ceilings of the same GPU, after the timed region: what a
    # kernel that only moves data reaches here, beside the 8 TB/s of the
    # specification
    ceil = stream_ceilings()
    if ceil:
        copy_bw = ceil["copy_GBps"]
        roof["copy"] = {"achieved": copy_bw, "read_only": ceil["read_GBps"], "write_only": ceil["write_GBps"],
                        "unit": "GB/s", "what": "olb_probes stream: best of copy / read / write streams, 16-byte "
                                                "accesses over 2 GiB buffers (copy counts read + write)"}
    else:
        _, copy_bw = copy_gbps(1.0, reps=5)
        roof["copy"] = {"achieved": round(copy_bw, 1), "unit": "GB/s",
                        "what": "1 GiB torch device-to-device copy, read + write (olb_probes not built)"}
    roof["frac_of_copy"] = round(achieved_gbs / copy_bw, 4)
    if traffic:
        roof["traffic_GBps"] = round(traffic / avg_launch_s / 1e9, 1)
        roof["traffic_frac_of_copy"] = round(traffic / avg_launch_s / 1e9 / copy_bw, 4)

    cpu = None
    if not args.no_cpu:
        print("[bench] cpu baseline (oracle)", file=sys.stderr, flush=True)
        cpu = cpu_baseline(args.workload, args.cpu_seconds)

    out = {
        "metric": "MLUPS per full RK3 step (D2Q25)",
        "value": round(mlups, 2),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_events / args.steps, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if precision == 0 else "f32+f64",
        "data": "synthetic",
        "config": {"workload": args.workload, "description": WORKLOADS[args.workload],
                   "nodes": cells, "instances": len(cases), "tile": tile,
                   "precision": "fp64" if precision == 0 else "fp32-mixed",
                   "launch": "sequential instances" if args.sequential else "one launch per stage",
                   "wall_s": round(wall, 3)},
        "roofline": roof,
        "cpu_baseline": cpu,
    }
    if valu:
        out["roofline"]["valu"] = valu
    if args.workload == "shard4096x512":
        out["config"]["halo_bytes_per_stage"] = shard_halo_bytes(cases[0].params["nx"], precision)
        out["config"]["stage_launch_ms"] = round(avg_launch_s * 1e3, 4)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
