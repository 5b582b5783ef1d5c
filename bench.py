"""Throughput of the PIC-MCC step on one MI355X.

Workload (default): the 128x128x512-cell, dx = 2 nm, 1 GV/m gap preloaded
with 10 M electrons (5 eV), 10 M Cu+ at the same positions and 5 M Cu
neutrals (3000 K), with Fowler-Nordheim emission over a 20 nm disk and
1e5 evaporated neutrals per step, dt = 2e-16 s, Lotz ionisation + elastic
collisions, Poisson solved to a 1e-10 relative residual every step.

Prints one JSON line: particle-steps/s over the timed steps (live particles
of all species, summed over steps, divided by wall time with inputs
resident in HBM), ms per step, the dominant kernel's roofline (algorithmic
bytes per launch over its HIP-event-timed duration), and the CPU oracle on a
bounded sample of the same workload.

The forms of the step run one after another on the same preload: plain
FP64 (the JSON line's value), mixed precision, mixed precision with the
learned warm start, and plain FP64 again with the previous potential as the
start instead of the extrapolated one; every solve to the same residual.
Grids of this size solve Poisson's equation directly, so a better start saves
nothing there; the _mg forms ask for a multigrid depth and run V-cycles from
the extrapolated or the learned start.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W]
                       [--variant all|fp64|mixed|learned_mixed|fp64_prev|
                        fp64_mg|mixed_mg|learned_mixed_mg|...]
                       [--no-cpu-baseline]
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0

# HBM bytes per launch measured with rocprofv3 FETCH_SIZE and WRITE_SIZE
# (one counter per run) on the c2 FP64 workload, each scaled by what the
# counter reads for a 1 GiB device copy (reads x 2.0, writes x 1.0); see
# profiles/c2_fp64_hbm_traffic.md.  Valid only for these kernels as built
# when measured; set to None when they change.
MEASURED_TRAFFIC = {
    ("c2", "fp64", "k_smooth2"): 241.2e6,
    ("c2", "fp64", "k_push_tile"): 2558.0e6,
    # profiles/c2_mixed_hbm_traffic.md; the smoother's figures are of steps
    # that ran V-cycles (unchanged since), the mixed one the mean
    # over the four finest-level passes of a refinement round (zero start,
    # two plain, FP64 accumulation).
    ("c2", "mixed", "k_smooth2"): (77.2e6 + 2 * 120.7e6 + 237.0e6) / 4,
    ("c2", "mixed", "k_push_tile"): 1623.8e6,
}


def progress(msg):
    """A progress line on stderr (the JSON result is the only stdout line)."""
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="c2")
    ap.add_argument("--variant", default="all",
                    choices=["all", "fp64", "mixed", "learned_mixed", "fp64_prev",
                             "fp64_mg", "mixed_mg", "learned_mixed_mg",
                             "fp64_np", "fp64_coulomb", "fp64_ionproc"],
                    help="fp64: plain FP64; mixed: FP32 particles; "
                         "learned_mixed: mixed with the U-Net warm start "
                         "(trained first on pairs from another run); _mg: the "
                         "same with V-cycles (mixed: FP32 smoothing with FP64 "
                         "refinement) instead of the direct solve; all: every "
                         "one, value = fp64")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--phases", action="store_true",
                    help="print per-phase times to stderr")
    return ap.parse_args()


def _oracle_sample(args):
    """Four oracle steps of the workload scaled to 1/8 of the grid and
    particles (one process, one thread): (particle-steps, seconds)."""
    p_full, seed = args
    import workloads as W
    from oracle import pic as O
    from oracle import poisson as P
    pl = p_full["preload"]
    nx, ny, nz = p_full["nx"] // 2, p_full["ny"] // 2, p_full["nz"] // 2
    p = W.scaled(p_full, nx, ny, nz, n_e=pl["n_e"] // 8,
                 n_ion=pl["n_ion"] // 8, n_n=pl["n_n"] // 8)
    if "disk" in p["sources"]:
        p["sources"]["disk"]["n_n"] = p_full["sources"]["disk"]["n_n"] // 8
    p["seed"] = seed
    g = P.Grid(p["nx"], p["ny"], p["nz"], p["dx"], p["bc_lo"], p["bc_hi"],
               p["v_lo"], p["v_hi"])
    st = O.State(g, seed=p["seed"], w_sp=p["w_sp"])
    n0 = 0
    for s, (pos, vel, ids) in W.preload(p, seed=1 + seed).items():
        st.load(s, pos, vel, ids)
        n0 += pos.shape[0]
    st.next_id = n0
    psteps = 0
    t0 = time.perf_counter()
    for _ in range(4):
        psteps += sum(st.count(s) for s in range(3))
        O.step(st, p, p["dt"])
    return psteps, time.perf_counter() - t0


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(p_full):
    """The oracle, as it stands, on a bounded sample of the workload: four
    steps of the workload scaled to 1/8 of the grid and particles, once on
    one core and then as independent seeds on every core of the host share
    (at most 16 processes, one thread each).  Runs before the GPU is
    touched, so the worker processes fork from a process without GPU
    state."""
    import multiprocessing as mp
    os.environ.setdefault("OMP_NUM_THREADS", "1")
    pl = p_full["preload"]
    ps1, el1 = _oracle_sample((p_full, 0))
    try:
        avail = len(os.sched_getaffinity(0))
    except AttributeError:
        avail = os.cpu_count() or 1
    n = max(1, min(16, avail))
    t0 = time.perf_counter()
    with mp.get_context("fork").Pool(n) as pool:
        res = pool.map(_oracle_sample, [(p_full, k) for k in range(n)])
    wall = time.perf_counter() - t0
    psn = sum(r[0] for r in res)
    nx, ny, nz = p_full["nx"] // 2, p_full["ny"] // 2, p_full["nz"] // 2
    return {"value": psn / wall, "unit": "particle-steps/s", "cores": n,
            "kind": "oracle",
            "sample": f"4 oracle steps of the workload scaled to "
                      f"{nx}x{ny}x{nz} cells with 1/8 of the preload "
                      f"({pl['n_e'] // 8} e, {pl['n_ion'] // 8} Cu+, "
                      f"{pl['n_n'] // 8} Cu), numpy float64; {n} independent "
                      f"seeds in {n} processes of one thread each, "
                      f"aggregate over the wall time",
            "seconds": round(wall, 3),
            "one_core": {"value": ps1 / el1, "cores": 1,
                         "seconds": round(el1, 3)},
            "host": {"nproc": os.cpu_count(), "cpu_model": _cpu_model(),
                     "processes": n}}


UNET_LAYERS = ((2, 16, 0), (16, 16, 0), (16, 32, 1), (32, 32, 1), (32, 64, 2),
               (64, 64, 2), (64, 128, 3), (128, 128, 3), (192, 64, 2),
               (64, 64, 2), (96, 32, 1), (32, 32, 1), (48, 16, 0), (16, 16, 0))


def unet_flops(D, H, W):
    """FLOP of one forward pass (2 per multiply-add; 3x3x3 convolutions and
    the 1x1x1 head)."""
    V0 = D * H * W
    f = sum(2 * 27 * ci * co * (V0 >> (3 * lv)) for ci, co, lv in UNET_LAYERS)
    return f + 2 * 16 * V0


def capacities(p, total_steps):
    pl = p["preload"]
    per_step_n = p["sources"].get("disk", {}).get("n_n", 0) + \
        p["sources"].get("sphere", {}).get("n", 0)
    # Margins for what the collisions add over the run (secondaries,
    # recombined atoms, Cu2+), generous beside the measured few thousand a
    # step.
    extra = 50_000 * max(total_steps, 40)
    return (pl["n_e"] + extra,
            pl["n_n"] + per_step_n * (total_steps + 2) + extra,
            pl["n_ion"] + extra, 1_000_000 + 10_000 * total_steps), per_step_n


def sources_label(p):
    src = p["sources"]
    parts = []
    if "fn" in src:
        parts.append("FN disk")
    d = src.get("disk", {})
    if d.get("n_e"):
        parts.append(f"{d['n_e']} e/step disk")
    if d.get("n_n"):
        parts.append(f"{d['n_n']} Cu/step disk")
    if src.get("sphere", {}).get("n"):
        sp = src["sphere"]
        parts.append(f"{sp['n']} Cu/step {sp['radius'] * 1e9:g} nm sphere")
    return " + ".join(parts)


def event_capacity(p, total_steps):
    """Per-step event-list length for a run of total_steps: the evaporated
    atoms pile up above the disk and the ionisation matching lists every
    atom of a cell with an event, about 1e5 entries per step of the run.
    A sphere source's atoms (2e5 a step at 3500 K move about 1e-4 nm a
    step) stay in the cells around the sphere, tens of thousands to a cell
    within a few steps, so there a cell with an event lists millions."""
    if p["sources"].get("sphere", {}).get("n"):
        return 1 << (24 if total_steps <= 60 else 26)
    if total_steps <= 60:
        return 1 << 17
    return 1 << (22 if total_steps <= 300 else 26)


def new_context(G, p, precision, pre, n0, cap, total_steps=60):
    q = dict(p)
    q["precision"] = precision
    flags = G.FLAG_CELL_GROUPS if (q.get("coulomb") or q.get("ion_processes")) else 0
    gpu = G.Pic(q, capacity=cap, max_events=event_capacity(p, total_steps),
                queue_capacity=1 << 10, flags=flags)
    for s, (pos, vel, ids) in pre.items():
        gpu.load(s, pos, vel, ids)
    gpu.set_clock(0, n0)
    return gpu


def train_warm_start(G, W, WS, p, cap, steps=32, epochs=12):
    """The learned start's network, trained on pairs recorded by a mixed
    run from another preload (seed 2) than the timed runs (seed 1)."""
    import torch
    pre = W.preload(p, seed=2)
    n0 = sum(v[0].shape[0] for v in pre.values())
    # Room for the recording run's own steps (its sources keep adding).
    cap = tuple(max(a, b) for a, b in zip(cap, capacities(p, steps + 4)[0]))
    gpu = new_context(G, p, "mixed", pre, n0, cap)
    del pre
    for _ in range(2):
        gpu.step(p["dt"])
    pairs, _ = WS.collect_pairs(gpu, p["dt"], steps)
    del gpu
    torch.cuda.empty_cache()
    net = G.UNet(p["nz"], p["ny"], p["nx"], params=W.unet_init(0))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    losses = WS.train(net, pairs, epochs=epochs, lr_max=1e-3, lr_min=1e-5,
                      loss="residual", k0=1 if p["bc_lo"] == 0 else 0)
    torch.cuda.synchronize()
    info = {"pairs": len(pairs), "epochs": epochs,
            "train_s": round(time.perf_counter() - t0, 3),
            "epoch_loss": [round(v, 5) for v in losses],
            "source": "mixed run, preload seed 2", "loss": "residual"}
    del pairs
    torch.cuda.empty_cache()
    return net, info


WARM_LABEL = {"prev": "previous phi", "extrap": "extrapolated phi",
              "unet": "unet"}


def run_variant(G, p, precision, pre, n0, cap, steps, warmup, net=None,
                warm="extrap", diagnostics=False):
    import numpy as np
    import torch
    gpu = new_context(G, p, precision, pre, n0, cap, warmup + 2 * steps)
    if net is not None:
        warm = "unet"
        gpu.set_warm_start("unet", net)
    else:
        gpu.set_warm_start(warm)
    dt = p["dt"]
    for _ in range(warmup):
        gpu.step(dt)
    counts = [gpu.count(s) for s in range(3)]
    nps = []
    couls = []
    ips = []

    def timed(k):
        nonlocal counts
        psteps = 0
        solves, electrons, ions = [], [], []
        nps.clear()
        couls.clear()
        ips.clear()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(k):
            psteps += sum(counts)
            electrons.append(counts[0])
            ions.append(counts[2])
            _, d = gpu.step(dt)
            counts = d["counts"]
            solves.append(d["solve"])
            nps.append((d["np_absorbed"], d["np_heat"]))
            couls.append((d["coulomb_like"], d["coulomb_ei"]))
            ips.append((d["recombinations"], d["ionisations2"],
                        d["charge_exchanges"]))
        torch.cuda.synchronize()
        return time.perf_counter() - t0, psteps, solves, electrons, ions

    # Throughput without instrumentation, then the same number of steps
    # with HIP events around every phase and finest-level smoothing launch
    # for the per-kernel figures.
    el, psteps, solves, electrons, ions = timed(steps)
    gpu.enable_timing(True)
    el_i, _, solves_i, electrons_i, ions_i = timed(steps)
    ph = gpu.phase_times()
    nu = gpu.p.get("nu_pre", 2) + gpu.p.get("nu_post", 2)
    diag = None
    if diagnostics:
        # The Debye-length check on the state the run left, per cell and per
        # tile-sized block, timed with HIP events like the step's phases.
        diag = {}
        n_charged = gpu.count(0) + gpu.count(2)
        for block in (1, 8):
            # (Once before: a kernel's first launch loads it.)
            gpu.debye_check(block, 0.5, with_lambda=False)
            gpu.enable_timing(True)
            for _ in range(5):
                info, _ = gpu.debye_check(block, 0.5, with_lambda=False)
            ms, calls = gpu.phase_times()["debye"]
            nb = info["blocks"]
            # Per charged particle its position and velocity read (48 B), for
            # blocks of a whole tile the velocity (24 B).
            alg = (24 if block == 8 else 48) * n_charged
            t = ms / max(calls, 1) * 1e-3
            diag[f"debye_block{block}"] = {
                "ms": round(t * 1e3, 4), "blocks": nb,
                "checked": info["checked"], "unresolved": info["unresolved"],
                "lambda_min_m": info["lambda_min"],
                "ratio_max": round(info["ratio_max"], 4),
                "roofline": {"bound": "hbm", "achieved": round(alg / t / 1e9, 1),
                             "peak": HBM_PEAK_GBS, "unit": "GB/s",
                             "frac": round(alg / t / 1e9 / HBM_PEAK_GBS, 4),
                             "bytes_per_call": int(alg)}}
    del gpu
    torch.cuda.empty_cache()
    out = {"precision": precision,
           "warm_start": WARM_LABEL[warm],
           "value": psteps / el, "ms_per_step": el / steps * 1e3,
           "ms_per_step_instrumented": el_i / steps * 1e3,
           "particles_avg": psteps / steps,
           "electrons_avg": float(np.mean(electrons)),
           "ions_avg": float(np.mean(ions)),
           "vcycles_avg": float(np.mean([d["vcycles"] for d in solves])),
           "start_rel_residual_avg": float(np.mean([d["rel_residual0"] for d in solves])),
           "final_rel_residual_max": float(max(d["rel_residual"] for d in solves)),
           "phase_ms": {k: round(v[0] / max(v[1], 1), 4) for k, v in ph.items()
                        if k != "smooth_l0"}}
    if net is not None:
        out["warm_ratio_avg"] = float(np.mean([d["warm_ratio"] for d in solves]))
        out["fallback_rate"] = float(np.mean([d["warm_rejected"] for d in solves]))
    if diag is not None:
        out["debye_check"] = diag
    if any(sum(t) for t in ips):
        out["recombinations_avg"] = float(np.mean([t[0] for t in ips]))
        out["ionisations2_avg"] = float(np.mean([t[1] for t in ips]))
        out["charge_exchanges_avg"] = float(np.mean([t[2] for t in ips]))
    if any(a + b for a, b in couls):
        out["coulomb_like_avg"] = float(np.mean([a for a, _ in couls]))
        out["coulomb_ei_avg"] = float(np.mean([b for _, b in couls]))
    if any(h for h, _ in nps):
        out["np_absorbed_avg"] = float(np.mean([h for h, _ in nps]))
        out["np_heat_J_avg"] = float(np.mean([e for _, e in nps]))
    out["_phases"] = ph
    out["_vcycles_total"] = sum(d["vcycles"] for d in solves_i)
    out["_electrons_i"] = float(np.mean(electrons_i))
    out["_ions_i"] = float(np.mean(ions_i))
    out["_nu"] = nu
    return out


def variant_rooflines(p, r, workload):
    """Algorithmic-bytes rooflines of one variant's dominant kernels, from
    its HIP-event-timed phases.

    push (k_push_tile, both layouts): per electron x, y, z, vx, vy, vz
    read and written (96 B FP64; 56 B mixed as cell + FP32 offsets and
    velocities), id read (8 B), cell key written (4 B); per ion the same
    without the id; per node the three E components read once (24 B FP64,
    12 B mixed) and the int64 charge of the pushed state read and written
    once (16 B); per cell the neutral count read once (4 B).

    smooth (finest level): with two sweeps before and after the coarse
    correction on a grid at least one owned column wide (16 x 16 nodes) it is
    k_smooth2, one launch per two red-black
    sweeps, whose algorithmic bytes are u and f read and u written once: 24 B
    per unknown in FP64; in the mixed form's correction solve 13 B, the mean
    of a refinement round's four passes (8 B from a zero start, 12, 12, and
    20 B adding the correction to the FP64 potential).  Otherwise it is k_rbgs, one launch per colour: u
    read once, f of the colour's half read and u of that half written, 16 B
    (8 B) per unknown.  Launches that only find the solve converged are
    timed but not counted as work."""
    mixed = r["precision"] == "mixed"
    prec = r["precision"]
    ph = r["_phases"]
    nodes = p["nx"] * p["ny"] * (p["nz"] + 1)
    cells = p["nx"] * p["ny"] * p["nz"]
    unknowns = p["nx"] * p["ny"] * (p["nz"] - 1)
    ms_push, n_push = ph["push_electron"]
    per_e = (56 + 8 + 4) if mixed else (96 + 8 + 4)
    per_i = (56 + 4) if mixed else (96 + 4)
    per_node = (12 if mixed else 24) + 16
    alg = (r["_electrons_i"] * per_e + r["_ions_i"] * per_i
           + nodes * per_node + cells * 4)
    t_push = ms_push / max(n_push, 1) * 1e-3
    ach = alg / t_push / 1e9 if t_push > 0 else 0.0
    kname = "k_push_tile<PartsM>" if mixed else "k_push_tile"
    push = {"bound": "hbm", "kernel": kname,
            "achieved": round(ach, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": round(ach / HBM_PEAK_GBS, 4),
            "traffic": MEASURED_TRAFFIC.get((workload, prec, "k_push_tile")),
            "bytes_per_launch": int(alg),
            "avg_launch_ms": round(t_push * 1e3, 5)}
    ms_sm, n_sm = ph["smooth_l0"]
    if n_sm == 0:  # the steps solved directly: no smoothing to report
        return {"push": push}
    # The fused pass needs a level at least one owned column wide (16 x 16
    # nodes).
    fused = p["nx"] >= 16 and p["ny"] >= 16 and r["_nu"] == 4
    if fused:
        n_eff = 2 * r["_vcycles_total"]
        # Mixed: a refinement round's four finest-level passes move 8 (zero
        # start), 12, 12 and 20 (FP64 accumulation) bytes per unknown.
        per_u = 13 if mixed else 24
        sname = "k_smooth2<%s> (finest level, two red-black sweeps per launch)" % (
            "float" if mixed else "double")
    else:
        n_eff = 2 * r["_nu"] * r["_vcycles_total"]
        per_u = 8 if mixed else 16
        sname = "k_rbgs (finest level, one colour)"
    sm_bytes = unknowns * per_u
    ach_s = sm_bytes * n_eff / (ms_sm * 1e-3) / 1e9 if ms_sm > 0 else 0.0
    smooth = {"bound": "hbm", "kernel": sname,
              "achieved": round(ach_s, 1), "peak": HBM_PEAK_GBS,
              "unit": "GB/s", "frac": round(ach_s / HBM_PEAK_GBS, 4),
              "traffic": (MEASURED_TRAFFIC.get((workload, prec, "k_smooth2"))
                          if fused else None),
              "bytes_per_launch": int(sm_bytes),
              "launches_timed": int(n_sm), "launches_with_work": int(n_eff),
              "avg_launch_ms": round(ms_sm / max(n_eff, 1), 5)}
    return {"push": push, "smooth": smooth}


def main():
    a = parse()
    if a.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {a.gpus}); the "
              "multi-GPU sharding of this path is a design, not a build.",
              file=sys.stderr)
        sys.exit(2)
    import torch

    import workloads as W
    from paper_2606_05893_amd import pic as G
    from paper_2606_05893_amd import warmstart as WS

    p = W.config(a.workload)
    pl = p["preload"]
    # The oracle's CPU leg first, before anything touches the GPU.
    cpu = None if a.no_cpu_baseline else cpu_baseline(p)
    if cpu is not None:
        progress(f"cpu baseline: {cpu['value']:.3e} particle-steps/s on "
                 f"{cpu['cores']} cores")
    variants = (["fp64", "mixed", "learned_mixed", "fp64_prev", "fp64_mg",
                 "mixed_mg", "learned_mixed_mg", "fp64_np", "fp64_coulomb",
                 "fp64_ionproc"]
                if a.variant == "all" else [a.variant])
    cap, per_step_n = capacities(p, a.warmup + 2 * a.steps)
    torch.cuda.set_device(0)
    net, train_info = None, None
    if any(v.startswith("learned") for v in variants):
        tp, tcap = p, cap
        if p["nx"] * p["ny"] * p["nz"] > 128 * 128 * 512:
            # A larger grid takes the network trained on the 128x128x512
            # workload (same cell size and field): the network is fully
            # convolutional, and its training runs at that size.
            tp = W.config("c2")
            tcap = capacities(tp, 40)[0]
        net, train_info = train_warm_start(G, W, WS, tp, tcap)
        if tp is not p:
            net = G.UNet(p["nz"], p["ny"], p["nx"], params=net.get_params())
            train_info["grid"] = f"{tp['nx']}x{tp['ny']}x{tp['nz']}"
        progress(f"warm-start network trained: {train_info['pairs']} pairs, "
                 f"{train_info['train_s']} s")
    pre = W.preload(p, seed=1)
    n0 = sum(v[0].shape[0] for v in pre.values())
    res = {}
    for v in variants:
        prec = "fp64" if v.startswith("fp64") else "mixed"
        pv = p
        if v.endswith("_mg"):
            pv = dict(p, mg_levels=16)  # (as deep as the grid allows)
        if v == "fp64_np":
            # A nanoparticle of 5 nm radius at z = 200 nm over the disk
            # centre absorbing electrons (alpha_EH = 0.5); no extra source.
            pv = dict(p)
            pv["sources"] = dict(p["sources"])
            pv["sources"]["sphere"] = dict(
                cx=p["nx"] * p["dx"] / 2, cy=p["ny"] * p["dx"] / 2,
                cz=200e-9, radius=5e-9, n=0, T_K=3500.0, absorb=True,
                alpha_eh=0.5)
        if v == "fp64_coulomb":
            # Coulomb binary collisions of all charged particles each step.
            pv = dict(p)
            pv["coulomb"] = dict(enabled=True, ln_lambda=10.0)
        if v == "fp64_ionproc":
            # Recombination (1e-24 m^2 at 1 eV), Cu+ ionisation (Lotz,
            # 20.29 eV) and charge exchange (5e-19 m^2) each step.
            pv = dict(p)
            pv["ion_processes"] = dict(enabled=True, sigma_rec_1eV=1e-24,
                                       lotz_a2=4.5e-18, I2_eV=20.29,
                                       cx_a=7.0710678118654755e-10, cx_b=0.0)
        res[v] = run_variant(G, pv, prec, pre, n0, cap, a.steps, a.warmup,
                             net if v.startswith("learned") else None,
                             warm="prev" if v == "fp64_prev" else "extrap",
                             diagnostics=(v == "fp64"))
        progress(f"{v}: {res[v]['ms_per_step']:.3f} ms/step")
    del pre
    head = res[variants[0]]
    mixed = head["precision"] == "mixed"
    rooflines = {}
    for v, r in res.items():
        if v in ("fp64", "mixed", "fp64_mg", "mixed_mg"):
            rooflines[v] = variant_rooflines(p, r, a.workload)
    if variants[0] in rooflines:
        hr = rooflines[variants[0]]
    else:
        hr = variant_rooflines(p, head, a.workload)
    roofline = hr["push"]
    out = {
        "metric": "particle-steps/s + ms/PIC step at 10M particles; "
                  "learned+mixed vs plain MG",
        "value": head["value"], "unit": "particle-steps/s", "n_gpus": 1,
        "steps": a.steps, "warmup": a.warmup,
        "ms_per_step": head["ms_per_step"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None,
        "dtype": "f32+f64" if mixed else "f64",
        "data": "synthetic",
        "config": {"workload": f"{a.workload}: {p['nx']}x{p['ny']}x{p['nz']} "
                               f"cells dx=2nm 1GV/m, preload "
                               f"{pl['n_e']} e + {pl['n_ion']} Cu+ + "
                               f"{pl['n_n']} Cu, {sources_label(p)}, "
                               f"Poisson to 1e-10",
                   "variant": variants[0]},
        "roofline": roofline,
        "rooflines": rooflines,
        "variants": {k: {kk: vv for kk, vv in v.items() if not kk.startswith("_")}
                     for k, v in res.items()},
    }
    if "learned_mixed" in res:
        lm = res["learned_mixed"]
        ms_w, n_w = lm["_phases"]["warm"]
        fl = unet_flops(p["nz"], p["ny"], p["nx"])
        t_w = ms_w / max(n_w, 1) * 1e-3
        out["roofline_unet"] = {
            "bound": "mfma", "kernel": "U-Net forward (BF16 MFMA) within the "
                                      "warm-start stage",
            "achieved": round(fl / t_w / 1e12, 2), "peak": 2500.0,
            "unit": "TFLOP/s", "frac": round(fl / t_w / 1e12 / 2500.0, 4),
            "flop_per_inference": fl, "stage_ms": round(t_w * 1e3, 4)}
        out["warm_start_training"] = train_info
        if "fp64" in res:
            out["learned_mixed_vs_fp64_step_time"] = round(
                lm["ms_per_step"] / res["fp64"]["ms_per_step"], 4)
        if "mixed" in res:
            out["learned_mixed_vs_mixed_step_time"] = round(
                lm["ms_per_step"] / res["mixed"]["ms_per_step"], 4)
    if "learned_mixed_mg" in res:
        for v in ("fp64_mg", "mixed_mg"):
            if v in res:
                out[f"learned_mixed_mg_vs_{v}_step_time"] = round(
                    res["learned_mixed_mg"]["ms_per_step"] / res[v]["ms_per_step"], 4)
                out[f"learned_mixed_mg_vs_{v}_vcycles"] = [
                    res["learned_mixed_mg"]["vcycles_avg"], res[v]["vcycles_avg"]]
    if cpu is not None:
        out["cpu_baseline"] = cpu
    if a.phases:
        print(json.dumps(out["variants"], indent=1), file=sys.stderr)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
