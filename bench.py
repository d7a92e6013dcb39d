#!/usr/bin/env python3
"""Benchmark of the SP-MPS hot path on one MI355X.

A step is one full projected one-site sweep (right-moving 1..L-1, then
left-moving L..2, i.e. 2(L-1) site steps: local Davidson solve with
H_eff x / N_eff x over all quadrature points, gauge move, environment update)
of a synthetic open Hubbard chain L=32, t=1, U=8, N=32, M=0, S=0, D=256,
G=9, random seed-initialised MPS.  The headline value is projected site
steps per second; the JSON line also carries H_eff x throughput, the
roofline of the dominant kernel and the oracle timed on the host.

    python bench.py [--gpus 1] [--steps 3] [--warmup 1]

Other modes: --abinitio-full (the 30-orbital workload at K=30, D=500,
G=11: FP64 sweeps, then split-BF16 sweeps to the same energy; its own JSON
line) and --heff-only N (N products at a centre site for hardware-counter
runs, --heff-workload picking the state; log lines only).
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP64_TFLOPS = 78.6
PEAK_HBM_GBS = 8000.0


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def fused_kernel_sha256():
    """sha256 of the product kernel's source and the header of its lists,
    which key the committed hardware-counter summaries."""
    import hashlib
    hs = hashlib.sha256()
    for f in ("chain.hip", "kernels.h"):
        hs.update(open(os.path.join(ROOT, "paper_1703_04789_amd", "csrc", f), "rb").read())
    return hs.hexdigest()


def measured_traffic():
    """HBM bytes per launch of the chained product from the committed rocprofv3
    summary (FETCH_SIZE and WRITE_SIZE, calibrated on a 64 MiB copy), or None
    when the kernel source has changed since those counters were taken."""
    import hashlib
    import re
    path = os.path.join(ROOT, "profiles", "heff_hubbard_L32_D256_G9_fused_fp64_hbm_traffic.md")
    try:
        txt = open(path).read()
        now = fused_kernel_sha256()
    except OSError:
        return None
    m_b = re.search(r"traffic_bytes_per_launch: (\d+)", txt)
    m_h = re.search(r"chain.hip\+kernels.h sha256: ([0-9a-f]+)", txt)
    if not m_b or not m_h or m_h.group(1) != now:
        return None
    return float(m_b.group(1))


def host_cpu():
    """Cores this process may use and the CPU model (Linux)."""
    try:
        cores = len(os.sched_getaffinity(0))
    except AttributeError:
        cores = os.cpu_count() or 1
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return cores, model


def cpu_baseline(wl, mv_per_step):
    """The oracle on a bounded sample of the same workload, timed on the host
    cores: its set-up (right canonical form and right environments) and left
    environments to the centre, one untimed H_eff x + N_eff x, then the
    median of 5 H_eff x + N_eff x with NumPy's BLAS on every core and of 3 on
    one thread, and one environment update at the centre.  Site steps per
    second are extrapolated from these: 1 / (mean matvecs per site step of
    the GPU run x t_matvec + t_env)."""
    import numpy as np
    from threadpoolctl import threadpool_info, threadpool_limits

    from oracle import mpo as ompo, mps as omps
    nproc, model = host_cpu()
    # BLAS threads as configured for this process (OMP_NUM_THREADS and the
    # like); the many-thread leg runs with them
    cores = max([i.get("num_threads", 1) for i in threadpool_info()] + [1])
    tab = wl.table()
    t0 = time.perf_counter()
    orc = omps.SPMPSOracle(tab, wl.blocks(), ompo.hubbard_mpo(wl.L, wl.t, wl.U), wl.twoS, wl.G)
    kc = wl.L // 2
    for j in range(1, kc):
        orc.update_left(j)
    t_setup = time.perf_counter() - t0
    x = orc.mps.A[kc - 1]
    legs = {}
    with threadpool_limits(limits=cores):
        orc.heff(kc, x)  # warm-up
        for leg, reps, lim in (("blas_threads", 5, cores), ("one_thread", 3, 1)):
            with threadpool_limits(limits=lim):
                ts = []
                for _ in range(reps):
                    a = time.perf_counter()
                    orc.heff(kc, x)
                    ts.append(time.perf_counter() - a)
            legs[leg] = {"threads": lim, "heff_s_median": float(np.median(ts)), "heff_s_all": ts}
        a = time.perf_counter()
        orc.update_left(kc)
        t_env = time.perf_counter() - a
    t_mv = legs["blas_threads"]["heff_s_median"]
    rate = 1.0 / (mv_per_step * t_mv + t_env)
    log(f"[cpu] {cores} BLAS threads of {nproc} usable cores ({model}): oracle set-up {t_setup:.1f}s, H_eff x median {t_mv:.3f}s "
        f"(one thread {legs['one_thread']['heff_s_median']:.3f}s), env update {t_env:.2f}s")
    return {"value": rate, "unit": "site steps/s", "cores": cores, "kind": "oracle", "cpu_model": model,
            "nproc": nproc,
            "extrapolated": True, "heff_s_median": t_mv, "env_update_s": t_env, "setup_s": t_setup,
            "legs": legs,
            "sample": (f"{wl.name}: oracle set-up + left environments to site {kc} ({t_setup:.1f}s); after one "
                       f"warm-up, median of 5 H_eff x/N_eff x at site {kc} with {cores} BLAS threads ({t_mv:.3f}s; median "
                       f"of 3 on one thread {legs['one_thread']['heff_s_median']:.3f}s) and one environment "
                       f"update ({t_env:.2f}s); rate extrapolated as 1/({mv_per_step:.1f} matvecs per site step "
                       f"x t_matvec + t_env)")}


def small_sweep_runs(sp, W, torch):
    """The L=8, D=16, G=5 workload (4 sweeps, default solver settings) timed
    whole on the GPU and in the oracle on the host: the one size where full
    sweeps compare directly.  Local solves stop at max_iter on both sides,
    so the trajectories separate at the 1e-7 level."""
    from oracle import mpo as ompo, mps as omps
    wl = W.hubbard_small()
    tab, blocks = wl.table(), wl.blocks()
    from threadpoolctl import threadpool_info
    cores = max([i.get("num_threads", 1) for i in threadpool_info()] + [1])
    g = sp.SPMPS(tab, blocks, sp.mpo_hubbard(wl.L, wl.t, wl.U), wl.twoS, wl.G)
    g.sweep(1)  # warm-up on a throw-away copy of the state
    g.close()
    g = sp.SPMPS(tab, blocks, sp.mpo_hubbard(wl.L, wl.t, wl.U), wl.twoS, wl.G)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rc, gs = g.sweep(wl.sweeps)
    torch.cuda.synchronize()
    tg = time.perf_counter() - t0
    g.close()
    t0 = time.perf_counter()
    orc = omps.SPMPSOracle(tab, blocks, ompo.hubbard_mpo(wl.L, wl.t, wl.U), wl.twoS, wl.G)
    os_ = omps.sweep(orc, wl.sweeps)
    to = time.perf_counter() - t0
    log(f"[bench] {wl.name}: GPU {len(gs) / tg:.1f} site steps/s, oracle {len(os_) / to:.1f} site steps/s "
        f"({cores} BLAS threads); E {gs[-1]['theta']:.10f} vs {os_[-1]['theta']:.10f}")
    return {"workload": wl.name, "sweeps": wl.sweeps, "site_steps": len(gs), "unit": "site steps/s",
            "gpu": len(gs) / tg, "oracle": len(os_) / to, "oracle_blas_threads": cores,
            "gpu_energy": gs[-1]["theta"], "oracle_energy": os_[-1]["theta"],
            "dE_final": gs[-1]["theta"] - os_[-1]["theta"], "ed_energy": -4.235806999129714,
            "note": "whole sweeps timed on both sides (oracle: set-up included); capped local solves"}


def product_ms(prof):
    """Milliseconds of one H_eff x from sp_heff_profile's phases, without the
    once-per-local-problem pre-mixing of the left environment."""
    return sum(p["ms"] for name, p in prof.items() if name != "premix_once")


def abinitio_runs(sp, W, torch, sweeps=6):
    """Synthetic ab-initio-shaped Hamiltonian (seeded integrals, K=12, N=12,
    S=0, D=128, G=11) with the default per-site plans (no timing-based plan
    choice, so every precision runs the same kernels at every site):
      - FP64 tiled path: `sweeps` sweeps, energy after each;
      - FP32 products: the same number of sweeps, energy difference to the
        FP64 run after each sweep; its speed-up counts only when the final
        difference is at most 1e-6;
      - split-BF16 products: sweeps until the energy reaches the FP64 run's
        final energy + 1e-6 (at most 2 x `sweeps`): time to that energy
        against the FP64 time (energies are FP64 Rayleigh quotients, i.e.
        variational), plus its difference at equal sweep counts;
      - plain FP64 path: one sweep, against the first FP64 sweep step by
        step;
    and one H_eff x at the centre for each."""
    wl = W.abinitio_reduced(12, 128, 11)
    h, eri = wl.integrals()
    mpo = sp.mpo_abinitio(h, eri)
    tab, blocks = wl.table(), wl.blocks()
    kc = wl.K // 2

    def centre_heff(st):
        for j in range(1, kc):
            st.env_update(j, +1)
        x = torch.tensor(st.get_site(kc), dtype=torch.float64, device="cuda")
        y, ny = torch.empty_like(x), torch.empty_like(x)
        prof = st.heff_profile(kc, x, y, ny, reps=10)
        ms = product_ms(prof)
        fl = st.heff_flops(kc)
        return ms, fl, prof.get("premix_once", {}).get("ms", 0.0)

    def run(path, prec, tol, n_max, target=None):
        log(f"[bench] {wl.name} path={path} {prec}: init")
        st = sp.SPMPS(tab, blocks, mpo, wl.twoS, wl.G, path=path, precision=prec)
        plans = [st.heff_plan(k)[0] for k in range(1, wl.K + 1)]
        energies, times, steps, t = [], [], [], 0.0
        for _ in range(n_max):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            rc, s1 = st.sweep(1, tol=tol)
            torch.cuda.synchronize()
            t += time.perf_counter() - t0
            energies.append(s1[-1]["theta"])
            times.append(t)
            steps += s1
            if target is not None and energies[-1] <= target:
                break
        ms, fl, pm = centre_heff(st)
        st.close()
        r = {"sweeps": len(energies), "seconds": t, "value": len(steps) / t, "energies": energies,
             "seconds_after_sweep": times, "solver_tol": tol,
             "matvecs_per_site_step": float(sum(x["matvecs"] for x in steps) / len(steps)),
             "heff_ms_centre": ms, "heff_flops_centre": fl, "heff_tflops_centre": fl / (ms * 1e-3) / 1e12,
             "premix_ms_centre_once_per_local_solve": pm, "fused_sites": sum(1 for p in plans if p > 0)}
        log(f"[bench] {wl.name} {path} {prec}: {r['value']:.2f} site steps/s over {len(energies)} sweeps, "
            f"E {energies[-1]:.10f}, H_eff x at site {kc} {ms:.3f} ms")
        return r, steps

    t64, s64 = run("tiled", "fp64", 1e-9, sweeps)
    plain, sp1 = run("plain", "fp64", 1e-9, 1)
    dE_plain = max(abs(a["theta"] - b["theta"]) for a, b in zip(sp1, s64[:len(sp1)]))
    f32, _ = run("tiled", "fp32", 1e-6, sweeps)
    f32["dE_vs_fp64_per_sweep"] = [a - b for a, b in zip(f32["energies"], t64["energies"])]
    f32["matched"] = abs(f32["dE_vs_fp64_per_sweep"][-1]) <= 1e-6
    f32["speedup_site_steps_vs_fp64_tiled"] = f32["value"] / t64["value"] if f32["matched"] else None
    f32["note"] = "products FP32 at sites with a fused plan, FP64 at the others; FP64 Rayleigh quotient per step"
    target = t64["energies"][-1] + 1e-6
    b16, _ = run("tiled", "bf16x3", 1e-5, 2 * sweeps, target=target)
    n_eq = min(len(b16["energies"]), len(t64["energies"]))
    b16["dE_vs_fp64_per_sweep"] = [a - b for a, b in zip(b16["energies"][:n_eq], t64["energies"][:n_eq])]
    b16["reached_fp64_energy"] = b16["energies"][-1] <= target
    b16["time_to_fp64_energy_speedup"] = (t64["seconds"] / b16["seconds"]) if b16["reached_fp64_energy"] else None
    b16["note"] = ("block products in split BF16 (hi+lo, three matrix-core products, FP32 accumulation), products "
                   "FP32 at sites with a fused plan, FP64 Rayleigh quotient per step; its looser local solves and metric threshold "
                   "follow another trajectory, so it is compared by the time to reach the FP64 run's energy "
                   f"after {sweeps} sweeps (within 1e-6), not at equal sweep counts")
    log(f"[bench] {wl.name}: FP32 dE {f32['dE_vs_fp64_per_sweep'][-1]:.2e} (matched {f32['matched']}); split BF16 "
        f"reached the FP64 energy in {b16['sweeps']} sweeps, {b16['seconds']:.2f} s against {t64['seconds']:.2f} s")
    return {"workload": wl.name, "K": wl.K, "N": wl.N, "twoS": wl.twoS, "D": wl.D, "G": wl.G, "seed": wl.seed,
            "mpo_max_bond": int(max(mpo[0])), "unit": "site steps/s", "dtype": "f64", "plans": "default per site",
            "tiled": t64, "plain_fp64": plain, "fp32": f32, "bf16x3": b16,
            "speedup_site_steps": t64["value"] / plain["value"],
            "max_step_dE_tiled_vs_plain_first_sweep": dE_plain,
            "note": "integrals from the seeded recipe of the 30-orbital workload at 12 orbitals; one-site sweeps "
                    "with a fixed block table descend slowly here (about 1e-3 per sweep after ten sweeps)"}


def abinitio_full_runs(sp, W, torch, sweeps=3):
    """The 30-orbital workload at its stated size (K=30, N=30, S=0, D=500,
    G=11, seed 4) from the seeded random start: `sweeps` FP64 sweeps, then
    split-BF16 sweeps from the same start until the energy reaches the FP64
    run's final energy + 1e-6 (at most 2 x `sweeps`), each with the site
    steps per second, energy after every sweep and the centre H_eff x after
    the sweeps.  The library prints one line per site step."""
    wl = W.abinitio_full()
    h, eri = wl.integrals()
    t0 = time.perf_counter()
    mpo = sp.mpo_abinitio(h, eri)
    t_mpo = time.perf_counter() - t0
    log(f"[bench] {wl.name}: MPO {t_mpo:.1f} s, max bond {int(max(mpo[0]))}")
    tab, blocks = wl.table(), wl.blocks()
    kc = wl.K // 2

    def run(prec, tol, n_max, target=None):
        log(f"[bench] {wl.name} {prec}: init")
        t0 = time.perf_counter()
        st = sp.SPMPS(tab, blocks, mpo, wl.twoS, wl.G, precision=prec)
        torch.cuda.synchronize()
        t_init = time.perf_counter() - t0
        free, total = torch.cuda.mem_get_info()
        energies, times, steps, t = [], [], [], 0.0
        for n in range(n_max):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            rc, s1 = st.sweep(1, tol=tol, verbose=True)
            torch.cuda.synchronize()
            t += time.perf_counter() - t0
            energies.append(s1[-1]["theta"])
            times.append(t)
            steps += s1
            log(f"[bench] {wl.name} {prec} sweep {n}: E {energies[-1]:.10f}, {len(steps) / t:.3f} site steps/s")
            if target is not None and energies[-1] <= target:
                break
        for j in range(1, kc):
            st.env_update(j, +1)
        x = torch.tensor(st.get_site(kc), dtype=torch.float64, device="cuda")
        y, ny = torch.empty_like(x), torch.empty_like(x)
        prof = st.heff_profile(kc, x, y, ny, reps=3)
        ms = product_ms(prof)
        pm = prof.get("premix_once", {}).get("ms", 0.0)
        fl = st.heff_flops(kc)
        st.close()
        del st
        torch.cuda.empty_cache()
        return {"setup_s": t_init, "device_gb_in_use_after_setup": (total - free) / 1e9, "solver_tol": tol,
                "sweeps": len(energies), "seconds": t, "value": len(steps) / t, "energies": energies,
                "seconds_after_sweep": times,
                "matvecs_per_site_step": float(sum(x["matvecs"] for x in steps) / len(steps)),
                "converged_steps": int(sum(1 for x in steps if x["converged"])), "site_steps": len(steps),
                "heff_ms_centre": ms, "heff_flops_centre": fl, "heff_tflops_centre": fl / (ms * 1e-3) / 1e12,
                "premix_ms_centre_once_per_local_solve": pm}

    t64 = run("fp64", 1e-9, sweeps)
    target = t64["energies"][-1] + 1e-6
    b16 = run("bf16x3", 1e-5, 2 * sweeps, target=target)
    n_eq = min(len(b16["energies"]), len(t64["energies"]))
    b16["dE_vs_fp64_per_sweep"] = [a - b for a, b in zip(b16["energies"][:n_eq], t64["energies"][:n_eq])]
    b16["reached_fp64_energy"] = b16["energies"][-1] <= target
    b16["time_to_fp64_energy_speedup"] = (t64["seconds"] / b16["seconds"]) if b16["reached_fp64_energy"] else None
    log(f"[bench] {wl.name}: FP64 {t64['value']:.3f} site steps/s, E {t64['energies'][-1]:.10f} after {sweeps} "
        f"sweeps in {t64['seconds']:.1f} s; split BF16 {b16['value']:.3f} site steps/s, "
        f"E {b16['energies'][-1]:.10f} after {b16['sweeps']} sweeps in {b16['seconds']:.1f} s "
        f"(reached the FP64 energy: {b16['reached_fp64_energy']})")
    return {"workload": wl.name, "K": wl.K, "N": wl.N, "twoS": wl.twoS, "D": wl.D, "G": wl.G, "seed": wl.seed,
            "mpo_max_bond": int(max(mpo[0])), "mpo_build_s": t_mpo, "unit": "site steps/s", "fp64": t64,
            "bf16x3": b16}


def batch_runs(sp, W, torch, n=64):
    """The broken-symmetry guesses of the batched workload (n = 64 Hubbard
    states, L in 12..32, U in {4, 8}, D in {64, 128, 256, 512}, G=9): one
    sweep of all of them through sp_sweep_batch against the same sweep of
    each state one after another (fresh states each way, no warm-up: a sweep
    of every state is the unit of work), and one batched fused H_eff launch
    over every state at its centre site against the same products launched
    state by state."""
    ws = W.hubbard_batch(n)

    def make():
        return [sp.SPMPS(w.table(), w.blocks(), sp.mpo_hubbard(w.L, w.t, w.U), w.twoS, w.G) for w in ws]
    log(f"[bench] batch of {n}: batched")
    hs = make()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rc, st = sp.sweep_batch(hs, 1)
    torch.cuda.synchronize()
    tb = time.perf_counter() - t0
    nsteps = sum(len(x) for x in st)
    eb = [x[-1]["theta"] for x in st]
    # one batched fused H_eff launch over every state at its centre site,
    # against the same products launched state by state
    sites = [w.L // 2 for w in ws]
    single_us = 0.0
    for h, k in zip(hs, sites):
        for j in range(1, k):
            h.env_update(j, +1)
        x = torch.tensor(h.get_site(k), dtype=torch.float64, device="cuda")
        y, ny = torch.empty_like(x), torch.empty_like(x)
        single_us += 1e3 * h.heff_profile(k, x, y, ny, reps=10)["fused_heff"]["ms"]
    bp = sp.heff_batch_profile(hs, sites, reps=10)
    log(f"[bench] batched H_eff launch: {bp['usec']:.1f} us for {len(hs)} states ({bp['flops'] / bp['usec'] / 1e6:.2f} "
        f"TFLOP/s), {single_us:.1f} us one state at a time; as a HIP graph {bp['graph_usec']:.1f} us "
        f"(replays exact to {bp['graph_max_diff']:.1e})")
    for h in hs:
        h.close()
    log(f"[bench] batch of {n}: batched, host-driven subspace solves")
    hs = make()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rc, sth = sp.sweep_batch(hs, 1, solver="host")
    torch.cuda.synchronize()
    th = time.perf_counter() - t0
    for h in hs:
        h.close()
    log(f"[bench] batch of {n}: one after another")
    hs = make()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    es = [h.sweep(1)[1][-1]["theta"] for h in hs]
    torch.cuda.synchronize()
    ts = time.perf_counter() - t0
    for h in hs:
        h.close()
    log(f"[bench] batch of {n}: {nsteps / tb:.1f} vs {nsteps / ts:.1f} site steps/s")
    return {"workload": f"hubbard_batch n={n} L 12..32 D 64..512 G=9", "states": [w.name for w in ws],
            "site_steps": nsteps, "unit": "site steps/s", "batched": nsteps / tb,
            "batched_host_driven": sum(len(x) for x in sth) / th, "one_after_another": nsteps / ts,
            "batched_driver": "device-resident Davidson iteration (one HIP graph per round for all states)",
            "speedup": ts / tb, "max_energy_diff": max(abs(a - b) for a, b in zip(eb, es)),
            "batched_heff": {"sites": sites, "usec": bp["usec"], "flops": bp["flops"], "bytes": bp["bytes"],
                             "workgroups": bp["workgroups"],
                             "tflops": bp["flops"] / (bp["usec"] * 1e-6) / 1e12,
                             "frac_fp64_peak": bp["flops"] / (bp["usec"] * 1e-6) / 1e12 / PEAK_FP64_TFLOPS,
                             "gbs": bp["bytes"] / (bp["usec"] * 1e-6) / 1e9,
                             "frac_hbm_peak": bp["bytes"] / (bp["usec"] * 1e-6) / 1e9 / PEAK_HBM_GBS,
                             "usec_one_state_at_a_time": single_us,
                             "graph_usec": bp["graph_usec"], "graph_replay_max_diff": bp["graph_max_diff"]}}


def precond_runs(sp, W, torch):
    """Learned Davidson preconditioner, for each scope (the whole site vector,
    one N-block): record the solver's training pairs on the L=8, D=16
    workload, the L=32, D=256 workload and six broken-symmetry guesses
    (D <= 128; one sweep each, search space 64, 128 iterations), train the
    256-wide model for 20 epochs (batches of 16384 rows, Adam, lr 1e-3);
    then two sweeps of Hubbard L=48, U=6, D=512, G=9 at S=0 and S=2 with the
    diagonal rule and with each model (search space 32, 64 iterations,
    tolerance 1e-9).  G=9 is below the exact point count of
    L=48, so the projector there is approximate."""
    srcs = [W.hubbard_small(), W.hubbard_bench(0)] + W.hubbard_batch(16, D_choices=(64, 128))[:6]
    models, training = {}, {}
    for scope in ("vector", "nblock"):
        log(f"[bench] learned preconditioner ({scope}): recording")
        model = sp.MLP(W.mlp_init(256, 0), capacity=20_000_000, scope=scope)
        t0 = time.perf_counter()
        for w in srcs:
            st = sp.SPMPS(w.table(), w.blocks(), sp.mpo_hubbard(w.L, w.t, w.U), w.twoS, w.G)
            st.set_precond(record=model)
            st.sweep(1, max_sub=64, max_iter=128)
            st.close()
        torch.cuda.synchronize()
        t_rec = time.perf_counter() - t0
        rows = model.rows()
        t0 = time.perf_counter()
        loss = model.train(20, 16384, 1e-3)
        torch.cuda.synchronize()
        t_train = time.perf_counter() - t0
        log(f"[bench] learned preconditioner ({scope}): {rows} pairs, loss {loss[0]:.4f} -> {loss[-1]:.4f}")
        models[scope] = model
        training[scope] = {"training_pairs": rows, "record_seconds": t_rec, "train_seconds": t_train,
                           "loss_first_epoch": float(loss[0]), "loss_last_epoch": float(loss[-1])}
    evals = []
    for twoS, seed in ((0, 5), (4, 6)):
        wl = W.HubbardWorkload(f"hubbard_L48_U6_D512_G9_S{twoS // 2}", L=48, t=1.0, U=6.0, N=48, twoS=twoS,
                               twoM=0, D=512, G=9, sweeps=2, seed=seed)
        row = {"workload": wl.name}
        for name, use in (("diagonal", None), ("learned", models["vector"]), ("learned_nblock", models["nblock"])):
            st = sp.SPMPS(wl.table(), wl.blocks(), sp.mpo_hubbard(wl.L, wl.t, wl.U), wl.twoS, wl.G)
            if use is not None:
                st.set_precond(use=use)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            rc, steps = st.sweep(2, max_sub=32, max_iter=64)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            st.close()
            row[name] = {"davidson_iterations": int(sum(s["iters"] for s in steps)),
                         "converged_steps": int(sum(s["converged"] for s in steps)), "site_steps": len(steps),
                         "seconds": dt, "energy": steps[-1]["theta"]}
        log(f"[bench] {wl.name}: iterations diagonal {row['diagonal']['davidson_iterations']} learned "
            f"{row['learned']['davidson_iterations']} learned per N-block "
            f"{row['learned_nblock']['davidson_iterations']}")
        evals.append(row)
    for m in models.values():
        m.close()
    return {"model": "2-layer MLP, hidden 256, 5 features per element, FP32 weights, FP64 arithmetic; "
                     "'learned': rms over the site vector, 'learned_nblock': the residual restricted to one "
                     "N-block (rms over the block, block weight from the diagonal rule)",
            "training": training, "eval": evals,
            "note": "0.5 is the loss of a zero prediction"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--twoS", type=int, default=0)
    ap.add_argument("--max-iter", type=int, default=64)
    ap.add_argument("--max-sub", type=int, default=32)
    ap.add_argument("--keep", type=int, default=8)
    ap.add_argument("--tol", type=float, default=1e-9)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-autotune", action="store_true",
                    help="keep the default H_eff plans instead of timing them per site (sp_autotune)")
    ap.add_argument("--path", default="tiled", choices=["tiled", "plain"])
    ap.add_argument("--precision", default="fp64", choices=["fp64", "fp32", "bf16x3"],
                    help="precision of the H_eff products inside the local solves (SP_FP64 / SP_FP32 / SP_BF16X3)")
    ap.add_argument("--no-plain", action="store_true", help="skip the plain FP64 comparison run")
    ap.add_argument("--no-fp32", action="store_true", help="skip the reduced-precision (SP_FP32) run")
    ap.add_argument("--no-device", action="store_true",
                    help="skip the run with the device-resident Davidson iteration")
    ap.add_argument("--fp32-tol", type=float, default=1e-6,
                    help="local-solver residual tolerance of the SP_FP32 run (its products floor near 1e-6)")
    ap.add_argument("--no-abinitio", action="store_true",
                    help="skip the ab-initio-shaped Hamiltonian runs (K=12 orbitals, D=128, G=11)")
    ap.add_argument("--no-batch", action="store_true",
                    help="skip the batched-states run (64 broken-symmetry Hubbard guesses, D up to 512)")
    ap.add_argument("--no-precond", action="store_true",
                    help="skip the learned-preconditioner training and evaluation")
    ap.add_argument("--heff-workload", default="hubbard", choices=["hubbard", "abinitio", "abinitio16", "abinitio30"],
                    help="state of the --heff-only run: the benchmark Hubbard chain, the ab-initio workload "
                         "(K=12, D=128), a larger ab-initio state (K=16, D=256) or the 30-orbital one at its "
                         "stated size (K=30, D=500)")
    ap.add_argument("--abinitio-full", action="store_true",
                    help="only the 30-orbital ab-initio workload at K=30, D=500, G=11: FP64 sweeps, then split "
                         "BF16 until it reaches the FP64 energy (about 6 minutes); one JSON line")
    ap.add_argument("--abinitio-sweeps", type=int, default=3, help="FP64 sweeps of --abinitio-full")
    ap.add_argument("--heff-only", type=int, default=0,
                    help="only run this many H_eff x applications at the centre site, after a 64 MiB "
                         "device copy of known size (for hardware-counter runs), and exit")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py runs on exactly one GPU: the SP-MPS path here is single-GPU "
              "(sharding over quadrature points is a design, not built)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_1703_04789_amd as sp
    import workloads as W

    torch.cuda.set_device(0)
    wl = W.hubbard_bench(args.twoS)
    tab = wl.table()
    kw = dict(tol=args.tol, max_iter=args.max_iter, max_sub=args.max_sub, keep=args.keep)
    kc = wl.L // 2

    if args.abinitio_full:
        r = abinitio_full_runs(sp, W, torch, sweeps=args.abinitio_sweeps)
        print(json.dumps({"metric": "projected-sweep site steps per second", "value": r["fp64"]["value"],
                          "unit": "site steps/s", "n_gpus": 1, "steps": r["fp64"]["sweeps"], "warmup": 0,
                          "ms_per_step": r["fp64"]["seconds"] / r["fp64"]["sweeps"] * 1e3,
                          "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
                          "data": "synthetic", "config": {"workload": r["workload"], "K": r["K"], "D": r["D"],
                                                          "G": r["G"], "twoS": r["twoS"]},
                          "abinitio_full": r}), flush=True)
        return

    if args.heff_only:
        # calibration: a plain copy of exactly 64 MiB (read 64 MiB, write 64 MiB)
        src = torch.ones(8 << 20, dtype=torch.float64, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        if args.heff_workload in ("abinitio", "abinitio16", "abinitio30"):
            aw = {"abinitio": lambda: W.abinitio_reduced(12, 128, 11),
                  "abinitio16": lambda: W.abinitio_reduced(16, 256, 11),
                  "abinitio30": W.abinitio_full}[args.heff_workload]()
            gpu = sp.SPMPS(aw.table(), aw.blocks(), sp.mpo_abinitio(*aw.integrals()), aw.twoS, aw.G, path=args.path,
                           precision=args.precision)
            kc = aw.K // 2
        else:
            gpu = sp.SPMPS(tab, wl.blocks(), sp.mpo_hubbard(wl.L, wl.t, wl.U), wl.twoS, wl.G, path=args.path,
                           precision=args.precision)
        log(f"[bench] --heff-only: state of {args.heff_workload} set up")
        if args.path == "tiled" and not args.no_autotune:
            gpu.autotune(reps=5)
        for j in range(1, kc):
            gpu.env_update(j, +1)
        torch.cuda.synchronize()
        log(f"[bench] --heff-only: left environments up to site {kc} built")
        x = torch.tensor(gpu.get_site(kc), dtype=torch.float64, device="cuda")
        y, ny = torch.empty_like(x), torch.empty_like(x)
        for _ in range(args.heff_only):
            gpu.heff_apply(kc, x, y, ny)
        torch.cuda.synchronize()
        log(f"[bench] {args.heff_only} H_eff x applications at site {kc} ({args.path}); "
            f"site size {x.numel()}, algorithmic flops {gpu.heff_flops(kc):.4e}, plan {gpu.heff_plan(kc)}")
        if args.heff_workload != "hubbard":
            prof = gpu.heff_profile(kc, x, y, ny, reps=5)
            ms = product_ms(prof)
            log(f"[bench] {args.heff_workload} H_eff x at site {kc}: {ms:.3f} ms, "
                f"{gpu.heff_flops(kc) / (ms * 1e-3) / 1e12:.3f} TFLOP/s algorithmic")
        gpu.close()
        return

    def run(path, precision="fp64", tol=args.tol, solver="auto", n_steps=args.steps, warmup=args.warmup):
        log(f"[bench] {wl.name} path={path} {precision} solver={solver}: init")
        gpu = sp.SPMPS(tab, wl.blocks(), sp.mpo_hubbard(wl.L, wl.t, wl.U), wl.twoS, wl.G, path=path,
                       precision=precision)
        tuned = None
        if path == "tiled" and not args.no_autotune:
            # the H_eff plan of every site (in FP64 all plans run the same products)
            tuned = gpu.autotune(reps=5)
        kw = dict(tol=tol, max_iter=args.max_iter, max_sub=args.max_sub, keep=args.keep)
        if path == "tiled":
            kw["solver"] = solver
        for i in range(warmup):
            rc, st = gpu.sweep(1, **kw)
            log(f"[bench] {path} warmup sweep {i}: E={st[-1]['theta']:.10f}")
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        steps = []
        for i in range(n_steps):
            rc, st = gpu.sweep(1, **kw)
            steps += st
            log(f"[bench] {path} timed sweep {i}: E={st[-1]['theta']:.10f}")
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        # H_eff x throughput and per-phase timing at the centre site
        for j in range(1, kc):
            gpu.env_update(j, +1)
        x = torch.tensor(gpu.get_site(kc), dtype=torch.float64, device="cuda")
        y, ny = torch.empty_like(x), torch.empty_like(x)
        prof = gpu.heff_profile(kc, x, y, ny, reps=50)
        heff_ms = product_ms(prof)
        heff_flops = gpu.heff_flops(kc)
        plan = gpu.heff_plan(kc) if path == "tiled" else (0, 0)
        gpu.close()
        log(f"[bench] {path}: {len(steps) / (t1 - t0):.2f} site steps/s; H_eff x at site {kc}: {heff_ms:.3f} ms; "
            + ", ".join(f"{k} {v['ms']:.3f} ms" for k, v in prof.items()))
        return dict(steps=steps, elapsed=t1 - t0, prof=prof, heff_ms=heff_ms, heff_flops=heff_flops,
                    heff_tflops=heff_flops / (heff_ms * 1e-3) / 1e12, plan=plan, tuned=tuned)

    main_run = run(args.path)
    steps, elapsed, prof = main_run["steps"], main_run["elapsed"], main_run["prof"]
    n_site_steps = len(steps)
    value = n_site_steps / elapsed
    mv = float(np.mean([s["matvecs"] for s in steps]))
    energy = steps[-1]["theta"]
    heff_ms, heff_flops, heff_tflops = main_run["heff_ms"], main_run["heff_flops"], main_run["heff_tflops"]
    plain = None
    if args.path != "plain" and not args.no_plain:
        pr = run("plain")
        pv = len(pr["steps"]) / pr["elapsed"]
        plain = {"value": pv, "unit": "site steps/s", "heff_tflops": pr["heff_tflops"], "heff_ms": pr["heff_ms"],
                 "energy_after_timed_sweeps": pr["steps"][-1]["theta"],
                 "speedup_site_steps": value / pv, "speedup_heff": pr["heff_ms"] / heff_ms,
                 "dE_final_vs_this_path": pr["steps"][-1]["theta"] - energy,
                 "max_step_dE_vs_this_path": max(abs(a["theta"] - b["theta"]) for a, b in zip(steps, pr["steps"])),
                 "note": "step energies of the two paths differ while local solves stop at max_iter (rounding "
                         "steers the truncated Davidson runs apart); the energies reached agree"}
    device_resident = None
    if args.path == "tiled" and not args.no_device:
        dr = run("tiled", solver="device", n_steps=min(args.steps, 3), warmup=1)
        iters = sum(s["iters"] for s in dr["steps"])
        device_resident = {"value": len(dr["steps"]) / dr["elapsed"], "unit": "site steps/s",
                           "sweeps": min(args.steps, 3),
                           "usec_per_iteration": 1e6 * dr["elapsed"] / iters,
                           "usec_per_iteration_host_driven": 1e6 * elapsed / sum(s["iters"] for s in steps),
                           "energy_after_timed_sweeps": dr["steps"][-1]["theta"],
                           "note": "the same sweeps with the device-resident Davidson iteration (FP64 subspace "
                                   "solve in one GPU work-group, each iteration replayed from a HIP graph, no "
                                   "host decision within a local solve) instead of the host-core subspace solve"}
    fp32 = None
    if args.path == "tiled" and not args.no_fp32:
        fr = run("tiled", "fp32", args.fp32_tol)
        fv = len(fr["steps"]) / fr["elapsed"]
        e32 = fr["steps"][-1]["theta"]
        fp32 = {"value": fv, "unit": "site steps/s", "solver_tol": args.fp32_tol,
                "matvecs_per_site_step": float(np.mean([s["matvecs"] for s in fr["steps"]])),
                "heff_ms": fr["heff_ms"], "heff_tflops": fr["heff_tflops"],
                "energy_after_timed_sweeps": e32, "dE_vs_fp64_path": e32 - energy,
                "speedup_site_steps_vs_plain_fp64": (fv / plain["value"]) if plain else None,
                "note": "H_eff products in FP32 (FP32 environments, FP32 accumulation); Davidson, subspace "
                        "solve and the per-step Rayleigh quotient in FP64"}
    abinitio = None if args.no_abinitio else abinitio_runs(sp, W, torch)
    batch = None if args.no_batch else batch_runs(sp, W, torch)
    precond = None if args.no_precond else precond_runs(sp, W, torch)
    dom_name, dom = max(prof.items(), key=lambda kv: kv[1]["ms"])
    intensity = dom["flops"] / dom["bytes"]
    ridge = PEAK_FP64_TFLOPS * 1e12 / (PEAK_HBM_GBS * 1e9)
    if intensity >= ridge:
        achieved = dom["flops"] / (dom["ms"] * 1e-3) / 1e12
        roof = {"bound": "mfma", "achieved": achieved, "peak": PEAK_FP64_TFLOPS, "unit": "TFLOP/s",
                "frac": achieved / PEAK_FP64_TFLOPS, "traffic": None}
    else:
        achieved = dom["bytes"] / (dom["ms"] * 1e-3) / 1e9
        roof = {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                "frac": achieved / PEAK_HBM_GBS, "traffic": None}
    roof["kernel"] = f"{'k_bgemm' if args.path == 'plain' else 'k_chain'} ({dom_name}) at site {kc}"
    roof["plan"] = {"rows_per_task": main_run["plan"][0], "lds_doubles": main_run["plan"][1]}
    if args.path == "tiled" and dom_name == "fused_heff":
        roof["traffic"] = measured_traffic()
        roof["traffic_unit"] = "B per launch (HBM, rocprofv3 FETCH_SIZE + WRITE_SIZE, calibrated)"
    roof["per_launch"] = {k: {"ms": v["ms"], "flops": v["flops"], "bytes": v["bytes"]} for k, v in prof.items()}

    out = {
        "metric": "projected sweep sites/sec + H_eff·x TFLOP/s vs plain FP64 GPU at |dE|<=1e-6 Eh",
        "value": value,
        "unit": "site steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": elapsed / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": wl.name, "L": wl.L, "t": wl.t, "U": wl.U, "N": wl.N, "twoS": wl.twoS,
                   "twoM": wl.twoM, "D": wl.D, "G": wl.G, "seed": wl.seed, "path": f"{args.path} FP64",
                   "davidson": {"tol": args.tol, "max_iter": args.max_iter, "max_sub": args.max_sub,
                                "keep": args.keep},
                   "fused_plans": "autotuned per site (sp_autotune, 5 repetitions each)"
                   if main_run["tuned"] is not None else "default LDS budget"},
        "site_steps": n_site_steps,
        "matvecs_per_site_step": mv,
        "energy_after_timed_sweeps": energy,
        "heff_tflops": heff_tflops,
        "heff_ms": heff_ms,
        "heff_flops": heff_flops,
        "roofline": roof,
        "plain_fp64": plain,
        "device_resident": device_resident,
        "fp32": fp32,
        "abinitio": abinitio,
        "batch": batch,
        "learned_precond": precond,
    }
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(wl, mv)
        out["small_sweeps"] = small_sweep_runs(sp, W, torch)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
