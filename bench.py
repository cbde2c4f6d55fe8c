"""Benchmark of the lattice Boltzmann collide-and-stream path on one MI355X.

Headline workload: D2Q9 isothermal BGK, 2048 x 2048 periodic, float32, tau = 0.6, random-phase
k^-5/3 decaying turbulence (seed 0, rms Mach 0.05), synthetic input. One step = one time step of
the whole lattice (the library takes up to six per launch). Prints ONE JSON line.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-variants] [--no-cpu]
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# Vector instructions per second of the chip: 1024 SIMDs, four cycles each, 2.4 GHz (wavefronts of
# 64; float64 and float32 issue at the same rate).
VALU_PEAK = 1024 * 2.4e9 / 4
# Most time steps per launch of the kernels that take several.
STEPS_PER_LAUNCH = {"d2q9_bgk": 6, "d2q9_ddf": 2, "d3q27_bgk": 2}
PROFILE_COUNTERS = os.path.join(ROOT, "profiles", "counters_d2q9_bgk_fp32_2048.txt")
KERNEL_SOURCES = [os.path.join(ROOT, "paper_2609_28679_amd", "csrc", f)
                  for f in ("bgk_multi.hip", "bgk_common.h", "device_common.h")]


# The density reading of the non-equilibrium extrapolation walls that the bench runs (the
# library's default): the wall node continues the neighbour's pressure.
NEQ_DENSITY = "pressure-continued rho_B = rho_N T_N / T_W (default; wall_density 1 selects " \
              "the literal rho_B = rho_N)"


def log(msg):
    print("[bench] " + msg, file=sys.stderr, flush=True)


def source_digest(paths):
    import hashlib
    h = hashlib.sha256()
    for p in paths:
        with open(p, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def headline_counters(nodes):
    """The committed rocprofv3 counter summary of the headline kernel if it was taken on the
    current kernel source and this many nodes; None otherwise."""
    if not os.path.exists(PROFILE_COUNTERS):
        return None
    kv = {}
    for line in open(PROFILE_COUNTERS):
        if "=" in line and not line.startswith("#"):
            k, v = line.split("=", 1)
            kv[k.strip()] = v.strip()
    if kv.get("kernel_source_sha256_16") != source_digest(KERNEL_SOURCES):
        return None
    if int(kv.get("nodes", -1)) != nodes:
        return None
    return kv


def counter_traffic(nodes):
    """Bytes per launch of six steps from the committed counter summary, or None."""
    kv = headline_counters(nodes)
    return float(kv["hbm_bytes_per_launch"]) if kv else None


def time_lattice(lat, steps, warmup):
    """(wall seconds for exactly `steps` steps bracketed by synchronisation, event ms)."""
    import torch
    lat.step(warmup)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ms = lat.time_steps(steps)
    torch.cuda.synchronize()
    return time.perf_counter() - t0, ms


def variant(name, make, steps, warmup, bytes_per_node, extra=None, steps_per_launch=1):
    """bytes_per_node: a state read and written once, which is what a launch has to move; a launch
    that takes several steps moves it once for all of them."""
    import torch
    lat = make()
    wall, ms = time_lattice(lat, steps, warmup)
    nodes = lat.nodes
    lat.close()
    del lat
    torch.cuda.empty_cache()
    per_launch_s = ms / 1e3 / steps
    gbs = bytes_per_node / steps_per_launch * nodes / per_launch_s / 1e9
    out = {"mlups": round(nodes * steps / wall / 1e6, 1),
           "kernel_us": round(per_launch_s * 1e6, 2),
           "algorithmic_GBs": round(gbs, 1),
           "hbm_frac": round(gbs / HBM_PEAK_GBS, 4),
           "bytes_per_node": bytes_per_node, "steps_per_launch": steps_per_launch}
    if extra:
        out.update(extra)
    log("%s: %s" % (name, out))
    return out


def surrogate_variant(binding, inputs, steps, inference_only=False):
    """Surrogate recipe: 1M training pairs harvested from 2048^2 turbulence runs at three tau,
    BF16 training (48000 Adam steps of batch 4096, learning rate 2e-3, 6e-4, 2e-4 in three equal
    stages), inference timed at 2048^2 (seed 5, tau 0.6) with the per-node plain judge;
    velocity rel-L2 against the FP64 oracle measured on a 256^2 held-out run.
    inference_only: skip harvest and training and time the inference with the initial weights
    (for profiling: the inference kernel evaluates the network and the plain collision at every
    node whatever the weights, so its work does not depend on them)."""
    import torch
    from paper_2609_28679_amd import surrogate
    from oracle import bgk
    from oracle.equilibrium import moments
    if inference_only:
        rho, u = inputs.random_phase_turbulence_2d(2048, seed=5)
        lat = binding.Lattice(rho, u, tau=0.6, collision="mlp")
        lat.set_mlp(binding.pack_mlp(inputs.mlp_init(11)), 0.05)
        wall, ms = time_lattice(lat, steps, 10)
        nodes = lat.nodes
        lat.close()
        per = ms / 1e3 / steps
        out = {"mlups": round(nodes * steps / wall / 1e6, 1), "kernel_us": round(per * 1e6, 2),
               "weights": "initial (inference only)"}
        log("surrogate (inference only): %s" % out)
        return out
    t0 = time.perf_counter()
    fields = inputs.random_phase_turbulence_2d(2048, seed=0)
    X, Y = surrogate.harvest(fields, [0.51, 0.6, 1.0], 1_000_000, (100, 10000), 20, seed=1)
    X, Y = surrogate.shuffle(X, Y, 7)
    t1 = time.perf_counter()
    init = inputs.mlp_init(11)
    torch.cuda.synchronize()
    tt0 = time.perf_counter()
    schedule = [(16000, 2e-3), (16000, 6e-4), (16000, 2e-4)]
    tr, w = surrogate.train(X, Y, init, batch=4096, schedule=schedule)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - tt0
    loss = surrogate.loss(tr, X[:65536], Y[:65536])
    tr.close()
    del X, Y
    tol = 0.05
    rho, u = inputs.random_phase_turbulence_2d(2048, seed=5)
    lat = binding.Lattice(rho, u, tau=0.6, collision="mlp")
    lat.set_mlp(w, tol)
    wall, ms = time_lattice(lat, steps, 10)
    fb, up = lat.mlp_stats()
    nodes = lat.nodes
    lat.close()
    # parity on a held-out 256^2 field against the oracle
    r2, u2 = inputs.random_phase_turbulence_2d(256, seed=5)
    lat = binding.Lattice(r2, u2, tau=0.6, collision="mlp")
    lat.set_mlp(w, tol)
    lat.step(100)
    _, ug, _, _ = lat.moments()
    lat.close()
    _, uo = moments(bgk.run(bgk.init_equilibrium(r2, u2), 1 / 0.6, 100))
    rel = float(np.sqrt(((ug - uo) ** 2).sum() / (uo ** 2).sum()))
    per = ms / 1e3 / steps
    out = {"mlups": round(nodes * steps / wall / 1e6, 1), "kernel_us": round(per * 1e6, 2),
           "algorithmic_GBs": round(72 * nodes / per / 1e9, 1),
           "hbm_frac": round(72 * nodes / per / 1e9 / HBM_PEAK_GBS, 4),
           "fallback_rate": round(fb / max(up, 1), 4), "tol": tol,
           "velocity_rel_l2_vs_oracle_256_100steps": rel,
           "train": {"samples": 1_000_000, "harvest_s": round(t1 - t0, 2),
                     "steps": sum(n for n, _ in schedule), "lr_stages": schedule,
                     "batch": 4096, "train_s": round(t_train, 2), "final_loss": loss}}
    log("surrogate: %s" % out)
    return out


def copy_ceiling(binding, nbytes=1 << 30, reps=20):
    """Device-to-device copy of nbytes (read nbytes + write nbytes) with the library's
    streaming copy kernel and with the runtime's copy (torch copy_), timed with HIP events on
    torch's current stream, on which both run. At 1 GiB nothing stays in the 256 MB
    last-level cache (the HBM ceiling of a streaming kernel); at the size of one 2048^2
    reduced-storage state (two buffers of 100.7 MB) both buffers fit it."""
    import torch
    n = nbytes // 4
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    out = {"bytes_moved": 2 * n * 4}
    for name, fn in (("lbm_device_copy", lambda: binding.device_copy(src, dst)),
                     ("runtime_copy", lambda: dst.copy_(src))):
        for _ in range(3):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        e1.synchronize()
        us = e0.elapsed_time(e1) * 1e3 / reps
        out[name] = {"us": round(us, 2), "GBs": round(2 * n * 4 / us / 1e3, 1),
                     "frac_of_peak": round(2 * n * 4 / us / 1e3 / HBM_PEAK_GBS, 4)}
    del src, dst
    torch.cuda.empty_cache()
    return out


def cpu_baseline():
    """The FP64 NumPy oracle on a bounded sample of the headline workload."""
    from threadpoolctl import threadpool_limits

    from oracle import bgk
    from paper_2609_28679_amd import inputs
    n, steps = 2048, 40
    rho, u = inputs.random_phase_turbulence_2d(n, seed=0)
    f = bgk.init_equilibrium(rho, u)
    omega = bgk.omega_from_tau_lb(0.6)
    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        bgk.run(f, omega, steps)
        dt = time.perf_counter() - t0
    return {"value": round(n * n * steps / dt / 1e6, 3), "unit": "MLUPS", "cores": 1,
            "kind": "oracle",
            "sample": "D2Q9 FP64 NumPy oracle, 2048x2048 turbulence, tau 0.6, %d steps "
                      "(%.1f s, one thread; host has %d CPUs)" % (steps, dt, os.cpu_count())}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10000)
    ap.add_argument("--warmup", type=int, default=100)
    ap.add_argument("--no-variants", action="store_true")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--only", default="",
                    help="comma-separated variant names to run (default: all)")
    ap.add_argument("--surrogate-inference-only", action="store_true",
                    help="surrogate variant without harvest and training (profiling)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="also run a 1 GiB device copy (reference kernel for HBM counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU only: the lattice is not sharded across GPUs in this "
              "library; run with --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2609_28679_amd import binding, inputs

    torch.cuda.set_device(0)
    binding.load()
    if args.copy_probe:
        src = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        log("copy probe: 3 x %d bytes read + written" % (src.numel() * 4))
        del src, dst
    n, tau = 2048, 0.6
    log("headline: D2Q9 FP32 %dx%d tau %g, warmup %d, steps %d" % (n, n, tau, args.warmup, args.steps))
    rho, u = inputs.random_phase_turbulence_2d(n, seed=0)
    lat = binding.Lattice(rho, u, tau=tau)
    nodes = lat.nodes
    wall, ms = time_lattice(lat, args.steps, args.warmup)
    lat.close()
    del lat
    torch.cuda.empty_cache()
    mlups = nodes * args.steps / wall / 1e6
    per_launch_s = ms / 1e3 / args.steps
    # a state read and written once per launch of six steps
    bytes_per_node = 72 / STEPS_PER_LAUNCH["d2q9_bgk"]
    achieved = bytes_per_node * nodes / per_launch_s / 1e9
    counters = headline_counters(nodes)
    traffic = issue = None
    if counters:
        per_step = int(counters["steps_per_launch"])
        traffic = round(float(counters["hbm_bytes_per_launch"]) / per_step)
        issue = float(counters["sq_insts_valu"]) / per_step / per_launch_s
    log("headline: %.1f MLUPS, kernel %.2f us, %.1f GB/s" % (mlups, per_launch_s * 1e6, achieved))
    # At 2048^2 the states stay in the 256 MB last-level cache for the most part. At 4096^2 (604 MB
    # per buffer, two buffers) the same kernel runs from HBM; it is timed here too, next to a 1 GiB
    # device copy (the practical HBM ceiling).
    n4 = 4096
    log("HBM-resident reference: D2Q9 FP32 %dx%d tau %g" % (n4, n4, tau))
    r4, u4 = inputs.random_phase_turbulence_2d(n4, seed=0)
    lat = binding.Lattice(r4, u4, tau=tau)
    steps4 = max(50, min(args.steps // 10, 500))
    _, ms4 = time_lattice(lat, steps4, 10)
    nodes4 = lat.nodes
    lat.close()
    del lat, r4, u4
    torch.cuda.empty_cache()
    per4 = ms4 / 1e3 / steps4
    achieved4 = bytes_per_node * nodes4 / per4 / 1e9
    copy = copy_ceiling(binding)
    log("4096^2: kernel %.2f us, %.1f GB/s; 1 GiB copy: %s" % (per4 * 1e6, achieved4, copy))
    copy_llc = copy_ceiling(binding, 2048 * 2048 * 24, reps=200)
    log("copy of one 2048^2 reduced-storage state (100.7 MB): %s" % copy_llc)

    variants = {}
    if not args.no_variants:
        vs = max(200, min(args.steps, 2000))
        n4 = 4096
        fields = {}

        def get(key, make):
            """Inputs shared by several variants, generated once on first use."""
            if key not in fields:
                fields[key] = make()
            return fields[key]

        turb4 = lambda: get("turb4096", lambda: inputs.random_phase_turbulence_2d(n4, seed=0))
        tgv3 = lambda: get("tgv256", lambda: inputs.taylor_green_3d(256, 0.05))
        shear4 = lambda: get("shear4096", lambda: inputs.thermal_shear_layer(n4, seed=0))

        def ddf_lattice(storage, phi=1, **kw):
            rs, us, ts = shear4()
            return binding.Lattice(rs, us, ts, model="ddf", tau=0.6, wall_y=True, phi=phi,
                                   storage=storage, **kw)

        def vdw_lattice():
            # van der Waals fluid above its critical point (T_cr 1.2, P_cr 0.25 in lattice
            # units: a = 27 R^2 T_cr^2 / (64 P_cr), b = R T_cr / (8 P_cr)) at rho = 1, where
            # theta = P / rho stays near 0.31
            _, us, ts = inputs.thermal_shear_layer(4096, seed=0, T0=1.4, dT=0.03)
            return binding.Lattice(np.ones_like(ts), us, ts, model="ddf", tau=0.6, wall_y=True,
                                   phi=1, storage="fp32", vdw=(0.27, 0.2))

        def vdw_tgv3():
            # the 3D Taylor-Green velocity at rho = 1, T = 1.4 (theta = P / rho ~ 0.31)
            _, u3 = inputs.taylor_green_3d(256, 0.05)
            return np.ones(u3.shape[1:]), u3, np.full(u3.shape[1:], 1.4)

        red = "fp32 moments + %s f-f_eq (6 of 9 stored)"
        red_ddf = "fp32 moments + %s non-equilibrium (6 f + 8 g of 18 stored)"
        plan = [
            ("d2q9_bgk_fp32_2048_two_buffers", lambda n: variant(
                n, lambda: binding.Lattice(rho, u, tau=tau, streaming="two"), vs, 20, 72,
                {"streaming": "two buffers"}, steps_per_launch=STEPS_PER_LAUNCH["d2q9_bgk"])),
            ("d2q9_bgk_fp32_2048_forced", lambda n: variant(
                n, lambda: binding.Lattice(rho, u, tau=tau, force=(1e-6, 0.0)), vs, 20, 72,
                {"force": "uniform (1e-6, 0), shifted equilibrium",
                 "streaming": "one buffer, through the read-out area and back"},
                steps_per_launch=STEPS_PER_LAUNCH["d2q9_bgk"])),
            ("d2q9_bgk_fp32_4096", lambda n: variant(
                n, lambda: binding.Lattice(*turb4(), tau=tau), vs, 20, 72,
                {"streaming": "two buffers (automatic choice above 384 MiB)"},
                steps_per_launch=STEPS_PER_LAUNCH["d2q9_bgk"])),
            ("d3q27_bgk_fp32_256", lambda n: variant(
                n, lambda: binding.Lattice(*tgv3(), lattice="D3Q27", tau=0.55, diag_every=100),
                max(100, vs // 10), 10, 216, {"diag_every": 100},
                steps_per_launch=STEPS_PER_LAUNCH["d3q27_bgk"])),
            ("d3q27_bgk_fp32_256_forced", lambda n: variant(
                n, lambda: binding.Lattice(*tgv3(), lattice="D3Q27", tau=0.55,
                                           force=(1e-6, 0.0, 0.0)),
                max(100, vs // 10), 10, 216, {"force": "uniform (1e-6, 0, 0)"})),
            ("d2q9_ddf_fp32_4096", lambda n: variant(
                n, lambda: ddf_lattice("fp32"), max(100, vs // 4), 10, 144,
                {"walls": "y", "phi": "central"},
                steps_per_launch=STEPS_PER_LAUNCH["d2q9_ddf"])),
            ("d2q9_ddf_fp32_4096_sources", lambda n: variant(
                n, lambda: ddf_lattice("fp32", force=(1e-7, 0.0), heat_source=1e-8),
                max(100, vs // 4), 10, 144,
                {"walls": "y", "phi": "central",
                 "sources": "uniform force (1e-7, 0) and heat source 1e-8"},
                steps_per_launch=STEPS_PER_LAUNCH["d2q9_ddf"])),
            ("d2q9_ddf_fp32_4096_prandtl", lambda n: variant(
                n, lambda: ddf_lattice("fp32", prandtl=0.71, eta_over_mu=1.0),
                max(100, vs // 4), 10, 144,
                {"walls": "y", "phi": "central",
                 "transport": "Pr 0.71 (heat flux q^c), eta/mu 1 (alpha theta div u)"},
                steps_per_launch=STEPS_PER_LAUNCH["d2q9_ddf"])),
            ("d2q9_ddf_fp32_4096_neq_walls", lambda n: variant(
                n, lambda: ddf_lattice("fp32", neq_walls=dict(u=((-0.05, 0.0), (0.05, 0.0)),
                                                              T=(0.8, 1.0))),
                max(100, vs // 4), 10, 144,
                {"walls": "y, non-equilibrium extrapolation (u_W = -+0.05, T_W = 0.8 / 1.0)",
                 "wall_density": NEQ_DENSITY, "phi": "central"},
                steps_per_launch=STEPS_PER_LAUNCH["d2q9_ddf"])),
            ("d2q9_ddf_fp32_4096_neq_walls_upwind", lambda n: variant(
                n, lambda: ddf_lattice("fp32", phi=2,
                                       neq_walls=dict(u=((-0.05, 0.0), (0.05, 0.0)),
                                                      T=(0.8, 1.0))),
                max(100, vs // 4), 10, 144,
                {"walls": "y, non-equilibrium extrapolation (u_W = -+0.05, T_W = 0.8 / 1.0)",
                 "wall_density": NEQ_DENSITY,
                 "phi": "upwind (sides keyed on the wall velocity on the boundary rows)"})),
            ("d2q9_ddf_fp32_4096_vdw", lambda n: variant(
                n, lambda: vdw_lattice(), max(100, vs // 4), 10, 144,
                {"walls": "y", "phi": "central",
                 "eos": "van der Waals a = 0.27, b = 0.2 (T_cr 1.2, P_cr 0.25), rho 1, "
                        "T 1.4 +- 0.03 shear layer"},
                steps_per_launch=STEPS_PER_LAUNCH["d2q9_ddf"])),
            ("d3q27_ddf_fp32_256", lambda n: variant(
                n, lambda: binding.Lattice(*inputs.thermal_taylor_green_3d(256, 0.05),
                                           lattice="D3Q27", model="ddf", tau=0.6, phi=1),
                max(50, vs // 20), 5, 432,
                {"phi": "central", "launches": "1 per step (fluxes and collision, marching in z)"})),
            ("d3q27_ddf_fp32_256_sources", lambda n: variant(
                n, lambda: binding.Lattice(*inputs.thermal_taylor_green_3d(256, 0.05),
                                           lattice="D3Q27", model="ddf", tau=0.6, phi=1,
                                           force=(1e-7, 0.0, 0.0), heat_source=1e-8),
                max(50, vs // 20), 5, 432,
                {"phi": "central", "launches": "1 per step (fluxes and collision, marching in z)",
                 "sources": "uniform force (1e-7, 0, 0) and heat source 1e-8"})),
            ("d3q27_ddf_fp32_256_prandtl", lambda n: variant(
                n, lambda: binding.Lattice(*inputs.thermal_taylor_green_3d(256, 0.05),
                                           lattice="D3Q27", model="ddf", tau=0.6, phi=1,
                                           prandtl=0.71, eta_over_mu=1.0),
                max(50, vs // 20), 5, 432,
                {"phi": "central", "launches": "1 per step (fluxes and collision, marching in z)",
                 "transport": "Pr 0.71 (heat flux q^c), eta/mu 1 (alpha theta div u)"})),
            ("d3q27_ddf_fp32_256_vdw", lambda n: variant(
                n, lambda: binding.Lattice(*vdw_tgv3(), lattice="D3Q27", model="ddf", tau=0.6,
                                           phi=1, vdw=(0.27, 0.2)),
                max(50, vs // 20), 5, 432,
                {"phi": "central", "launches": "1 per step (fluxes and collision, marching in z)",
                 "eos": "van der Waals a = 0.27, b = 0.2, rho 1, T 1.4"})),
            ("d3q27_ddf_fp32_256_neq_walls", lambda n: variant(
                n, lambda: binding.Lattice(*inputs.thermal_taylor_green_3d(256, 0.05),
                                           lattice="D3Q27", model="ddf", tau=0.6, phi=1,
                                           neq_walls=dict(u=((-0.05, 0.0), (0.05, 0.0)),
                                                          T=(0.8, 1.0))),
                max(50, vs // 20), 5, 432,
                {"phi": "central", "launches": "2 per step (boundary planes; fluxes and collision, marching in z)",
                 "walls": "y, non-equilibrium extrapolation (u_W = -+0.05, T_W = 0.8 / 1.0)",
                 "wall_density": NEQ_DENSITY})),
            ("d3q27_ddf_fp32_256_upwind", lambda n: variant(
                n, lambda: binding.Lattice(*inputs.thermal_taylor_green_3d(256, 0.05),
                                           lattice="D3Q27", model="ddf", tau=0.6, phi=2),
                max(50, vs // 20), 5, 432,
                {"phi": "upwind", "launches": "2 per step (fluxes, collision)"})),
            ("d2q9_ddf_fp32_4096_upwind", lambda n: variant(
                n, lambda: ddf_lattice("fp32", phi=2), max(100, vs // 4), 10, 144,
                {"walls": "y", "phi": "upwind"})),
            ("d2q9_ddf_bf16_4096", lambda n: variant(
                n, lambda: ddf_lattice("bf16"), max(100, vs // 4), 10, 88,
                {"walls": "y", "phi": "central", "storage": red_ddf % "bf16"})),
            ("d2q9_ddf_fp16_4096", lambda n: variant(
                n, lambda: ddf_lattice("fp16"), max(100, vs // 4), 10, 88,
                {"walls": "y", "phi": "central", "storage": red_ddf % "fp16"})),
            ("d2q9_bgk_bf16_4096", lambda n: variant(
                n, lambda: binding.Lattice(*turb4(), tau=tau, storage="bf16"),
                max(200, vs // 4), 20, 48, {"storage": red % "bf16"})),
            ("d2q9_bgk_bf16_2048", lambda n: variant(
                n, lambda: binding.Lattice(rho, u, tau=tau, storage="bf16"), vs, 20, 48,
                {"storage": red % "bf16"})),
            ("d2q9_bgk_fp16_2048", lambda n: variant(
                n, lambda: binding.Lattice(rho, u, tau=tau, storage="fp16"), vs, 20, 48,
                {"storage": red % "fp16"})),
            ("d2q9_bgk_mlp_2048", lambda n: surrogate_variant(
                binding, inputs, max(100, vs // 4), args.surrogate_inference_only)),
            ("d2q9_bgk_fp64_2048", lambda n: variant(
                n, lambda: binding.Lattice(rho, u, tau=tau, storage="fp64"),
                max(200, vs // 4), 20, 144, steps_per_launch=STEPS_PER_LAUNCH["d2q9_bgk"])),
        ]
        only = set(args.only.split(",")) if args.only else None
        if only and not only <= {name for name, _ in plan}:
            log("unknown variant(s) in --only: %s" % sorted(only - {name for name, _ in plan}))
            sys.exit(2)
        for name, run in plan:
            if only is None or name in only:
                variants[name] = run(name)
        fields.clear()

    line = {
        "metric": "MLUPS + % HBM roofline, plain FP32 vs reduced-storage vs surrogate at stated rel-L2",
        "value": round(mlups, 1),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(wall * 1e3 / args.steps, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        # the kernels compute in float64 on float32 storage (the roofline counts the stored
        # float32 bytes)
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": "D2Q9 BGK 2048x2048 periodic FP32, tau 0.6, random-phase "
                               "k^-5/3 turbulence (seed 0, rms Mach 0.05)",
                   "lattice": "D2Q9", "nx": n, "ny": n, "tau": tau, "storage": "fp32",
                   "arithmetic": "fp64",
                   "streaming": "one buffer, up to six steps per launch through the read-out area "
                                "(151 MB state, automatic choice)",
                   "parity": "velocity rel-L2 <= 1e-5 vs FP64 oracle (tests/test_gpu_bgk.py)"},
        # Launches of six steps are bound by vector issue: achieved = the vector instructions of a
        # step (counters of the committed profile of this kernel source, null once the source has
        # changed) / mean step time (HIP events on the context stream). hbm: the bytes of a state read
        # and written once per six steps / mean step time, against the 8 TB/s HBM peak; hbm_resident is
        # the same kernel at 4096^2, whose buffers do not fit the last-level cache. traffic: counter
        # bytes that leave the L2 towards the memory fabric per step (last-level-cache hits included).
        # one_step_equivalent: 72 bytes per node and step, which a run of one step per launch would
        # have to move at this speed; not a share of any bandwidth.
        "roofline": {"bound": "vector issue",
                     "achieved": None if issue is None else round(issue / 1e9, 1),
                     "peak": VALU_PEAK / 1e9, "unit": "G wavefront instructions/s",
                     "frac": None if issue is None else round(issue / VALU_PEAK, 4),
                     "hbm": {"achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                             "frac": round(achieved / HBM_PEAK_GBS, 4)},
                     "one_step_equivalent": {"GBs": round(72 * nodes / per_launch_s / 1e9, 1)},
                     "traffic": traffic,
                     "traffic_kind": "L2-to-fabric bytes per step (FETCH_SIZE + WRITE_SIZE), "
                                     "last-level-cache hits included",
                     "hbm_resident": {"workload": "D2Q9 BGK 4096x4096 FP32, two buffers "
                                                  "(604 MB each), same recipe",
                                      "kernel_us": round(per4 * 1e6, 2),
                                      "achieved": round(achieved4, 1),
                                      "frac": round(achieved4 / HBM_PEAK_GBS, 4)},
                     "copy_ceiling": copy,
                     "copy_ceiling_cache_resident": copy_llc},
        "variants": variants,
    }
    if not args.no_cpu:
        log("cpu baseline (oracle) ...")
        line["cpu_baseline"] = cpu_baseline()
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
