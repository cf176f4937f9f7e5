"""Benchmark: CV-ADAPT-VQE steps per second on the Kitaev-Kerr chain
(L=8, d=8, open, J=1, Delta=0.5, K=0.2; 16.7M complex64 amplitudes), one GPU.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline]

A step is one full ADAPT iteration on the device path: pool scoring (H psi and
all 28 pool gradients), selection, append, and BFGS re-optimisation of all
angles with energy + adjoint-gradient evaluations (gate build, forward gates,
H psi, fused reverse sweep).  The vacuum is even and every pool generator keeps
the total parity, so the driver keeps its states in the parity-halved layout
(the top mode's level follows from the other modes' parity: 8,388,608 stored
amplitudes).  Every gate the run selects is HR or PR and the vacuum is real,
so its evaluations run their gates and reverse steps on real float32
amplitudes (scoring on a complex64 copy), and runs of consecutive gates inside
three consecutive modes take one LDS-staged pass.  --full-layout,
--complex-states and --no-real-fusion switch these off; "variants" also
reports the default run gate by gate, with the full layout, with complex
states and with both.  W warm-up steps run on a separate ADAPT instance;
the K timed steps are steps 1..K of a fresh run from the vacuum.  Per-kernel
durations come from HIP events recorded on the launch stream inside the timed
region, around one launch in --prof-sample (default 4) of each kernel family:
two event records per timed launch lengthen the gap to the next kernel, and
timing every launch costs about 9% of the step rate.  The roofline entry is
the kernel with the largest total time.  A fused run's algorithmic bytes are
one pass over its states whatever its gate count; the fused kernels' entries
add the mean gates per launch and the bandwidth counted per gate.  BFGS
starts every step from the previous step's inverse Hessian, padded with the
identity for the new angle (Appendix D); --no-hessian-recycling starts from
the scaled identity.  After the timed region, "variants" reports the same
workload with central-difference BFGS gradients (the plain method), adjoint
gradients without and with Hessian recycling, and adjoint gradients through
the batched engine (persistent kernels, graph-replayed BFGS rounds), and
"warm_start": the learned warm start trained on 8 nearby points run by the
batched sweep, proposing angles after each step's selection (see
warm_start_leg; --no-warm-start skips it).  Then,
on the host, the FP64 oracle re-evaluates the GPU's ansatz after steps 5, 10,
15 and 20 ("replay_checked_steps", |dE| <= 1e-5 |E|) and is timed on steps
1..3 of the same trajectory at all BLAS threads and at one ("cpu_baseline");
--no-cpu-baseline skips both.  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
METRIC = "ADAPT steps/s, Kitaev-Kerr L=8 d=8, |ΔE|<1e-5 vs ED; apply-H GB/s vs peak"
KERNEL_NAMES = {0: "apply_h", 1: "pool_grads", 2: "gate2", 3: "gate2_adjoint", 4: "diag_gate", 9: "score",
                10: "gate2_real", 11: "gate2_adjoint_real", 12: "real_convert", 13: "apply_h_real",
                14: "gate2_real_fused", 15: "gate2_adjoint_real_fused", 16: "small_eval", 17: "gate2_fused",
                18: "gate2_adjoint_fused"}


def traffic_for(kid: int):
    """HBM bytes per launch from the committed rocprofv3 counter summary, or
    None when absent or when the kernel source changed since it was taken."""
    from paper_2606_05297_amd.rocprof_summary import source_sha

    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    try:
        t = json.load(open(path)).get("families", {}).get(KERNEL_NAMES[kid])
    except (ValueError, OSError):
        return None
    if not t or t.get("source_sha") != source_sha(KERNEL_NAMES[kid]):
        return None
    return t.get("hbm_bytes_per_launch")


def _blas_threads():
    try:
        from threadpoolctl import threadpool_info
        return max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        return 1


def cpu_leg(cfg, psi0, snaps, reps):
    """The oracle on the host, after the timed region.

    (1) Replay: the oracle (FP64) re-evaluates the GPU's own ansatz and angles
    after steps 5, 10, 15, 20 (those run) and compares energies to the GPU's,
    |dE| <= 1e-5 |E|.
    (2) Timing sample, steps 1..3 of the same trajectory: the oracle's pool
    scoring on the step-3 state (H psi and the 28 pool gradients) and one
    energy + adjoint evaluation of the step-3 ansatz (3 gates), each timed
    once with all BLAS threads and once with one; a step is scoring + the GPU
    run's mean evaluation count over steps 1..3 times one evaluation."""
    import numpy as np
    from threadpoolctl import threadpool_limits

    import oracle as O
    h = O.Ham(cfg["L"], cfg["d"], cfg["periodic"], cfg["J"], cfg["U"], cfg["mu"], cfg["Delta"], cfg["K"])
    L, d = cfg["L"], cfg["d"]
    replay = []
    for s in sorted(snaps):
        ops, th = snaps[s]
        t = time.perf_counter()
        psi = O.ansatz_state(psi0, ops, th, L, d)
        E = float(np.vdot(psi, O.apply_H_slices(h, psi)).real / np.vdot(psi, psi).real)
        Eg = reps[s - 1]["E"]
        replay.append({"step": s, "n_gates": len(ops), "E_gpu": Eg, "E_oracle": E, "rel_err": abs(Eg - E) / abs(E),
                       "ok": abs(Eg - E) <= 1e-5 * abs(E), "oracle_s": time.perf_counter() - t})
        print(f"[bench] replay step {s}: E_gpu={Eg:.8f} E_oracle={E:.8f}", file=sys.stderr, flush=True)
    ops3, th3 = snaps[3]
    evals = float(np.mean([r["bfgs_evals"] for r in reps[:3]]))

    def sample():
        t0 = time.perf_counter()
        psi3 = O.ansatz_state(psi0, ops3, th3, L, d)
        O.pool_gradients(h, psi3, cfg["pool"], apply_h=O.apply_H_slices)
        t1 = time.perf_counter()
        O.energy_and_grad_adjoint(h, psi0, ops3, th3, apply_h=O.apply_H_slices)
        t2 = time.perf_counter()
        return t1 - t0, t2 - t1

    threads = _blas_threads()
    ts_all, te_all = sample()
    with threadpool_limits(limits=1):
        ts_one, te_one = sample()
    step_all = ts_all + evals * te_all
    step_one = ts_one + evals * te_one
    base = {"value": 1.0 / step_all, "unit": "ADAPT steps/s", "cores": threads, "kind": "oracle",
            "value_1thread": 1.0 / step_one,
            "sample": (f"steps 1-3 of the same L=8 d=8 trajectory: oracle (NumPy/SciPy FP64) pool scoring on the "
                       f"GPU's step-3 state ({ts_all:.1f} s) and one energy + adjoint evaluation of its step-3 "
                       f"ansatz ({te_all:.1f} s), each timed once with {threads} BLAS threads "
                       f"(1 thread: {ts_one:.1f} s, {te_one:.1f} s); a step = scoring + the GPU run's "
                       f"{evals:.1f} evaluations per step over steps 1-3"),
            "seconds_per_step": step_all, "seconds_per_step_1thread": step_one}
    return base, replay


def warm_start_leg(cfg, hl, psi0, k, plain):
    """Batched + adjoint + learned warm start against the plain GPU method.

    Training data: plain ADAPT (adjoint gradients) for k steps on 8 points
    around the benchmark point, (Delta, K) scaled by U[0.9, 1.1] (seed 5), all
    run together by the batched sweep; their steps on the majority operator
    sequence become samples (J, Delta, K, n / 64) -> angles after step n, and
    the 4-128-128-64 network is trained on the GPU (bf16 MFMA kernels, Adam).
    Then steps 1..k of the benchmark point with Hessian recycling, as the
    headline, where every step selects first and, when the chosen circuit
    still follows the training sequence, proposes the network's angles
    (previous angles + predicted shift, predicted new angle); the library
    keeps a proposal only if its energy is not above the plain start.  The
    timed part is the k steps including network forwards and proposals;
    training is reported separately."""
    import numpy as np

    from paper_2606_05297_amd import warmstart as WS

    rng = np.random.default_rng(5)
    pts = [dict(cfg, Delta=cfg["Delta"] * f1, K=cfg["K"] * f2) for f1, f2 in rng.uniform(0.9, 1.1, (8, 2))]
    t0 = time.perf_counter()
    recs, ang = WS.run_sweep(pts, k)
    t_data = time.perf_counter() - t0
    seq, agree = WS.consensus(recs)
    X, T, nv = WS.dataset_agreeing(pts, ang, agree)
    t0 = time.perf_counter()
    net, hist = WS.train(X, T, nv, epochs=300, batch=256)
    t_train = time.perf_counter() - t0
    rs, proposed, kept, dt = WS.adapt_with_network(cfg, hl, psi0, k, net, seq, recycle_hessian=True)
    net.close()
    done = [r for r in rs if r["k_sel"] >= 0]
    return {"steps": len(done), "steps_per_s": len(done) / dt, "E_final": rs[-1]["E"],
            "bfgs_evals_per_step": float(np.mean([r["bfgs_evals"] for r in done])),
            "bfgs_iters_per_step": float(np.mean([r["bfgs_iters"] for r in done])),
            "proposals": proposed, "accepted": kept,
            "speedup_vs_plain_adjoint_recycling": (len(done) / dt) / plain["steps_per_s"],
            "training": {"points": len(pts), "samples": int(len(X)), "sequence_steps": len(seq),
                         "points_on_sequence_per_step": [int(sum(1 for a in agree if a > s)) for s in range(len(seq))],
                         "sweep_s": t_data, "train_s": t_train, "loss_first_last": [hist[0][1], hist[-1][1]]}}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--grad-mode", choices=["adjoint", "fd"], default="adjoint")
    ap.add_argument("--no-hessian-recycling", action="store_true",
                    help="start every BFGS from the scaled identity instead of the previous inverse Hessian")
    ap.add_argument("--no-variants", action="store_true", help="skip the FD-gradient and Hessian-recycling lines")
    ap.add_argument("--no-warm-start", action="store_true", help="skip the learned warm-start leg")
    ap.add_argument("--full-layout", action="store_true",
                    help="keep the ADAPT states in the full d^L layout (parity-halved layout off)")
    ap.add_argument("--complex-states", action="store_true",
                    help="evaluate every circuit on complex64 states (real states off)")
    ap.add_argument("--no-real-fusion", action="store_true",
                    help="run real-state gates and reverse steps gate by gate (fused runs off)")
    ap.add_argument("--prof-sample", type=int, default=4,
                    help="time one launch in this many per kernel family with HIP events (1: every launch)")
    ap.add_argument("--gate-fusion", type=int, choices=[0, 1, 2, 3], default=None,
                    help="0 per-gate passes, 1 fused forward circuit, 2 fused forward and adjoint, 3 passes planned "
                         "by the library (its default)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); the multi-GPU design is "
              "documented but not built", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import workload as W
    from paper_2606_05297_amd import lib

    torch.cuda.set_device(0)
    if args.gate_fusion is not None:
        lib.set_gate_fusion(args.gate_fusion)
    if args.full_layout:
        lib.set_sector_layout(lib.SECTOR_OFF)
    if args.complex_states:
        lib.set_real_states(lib.REAL_OFF)
    if args.no_real_fusion:
        lib.set_real_fusion(lib.RFUSE_OFF)
    cfg = W.config("kk_l8_d8")
    hl = lib.ham_from(cfg)
    n = cfg["d"] ** cfg["L"]
    psi0 = torch.zeros(n, dtype=torch.complex64, device="cuda")
    psi0[0] = 1.0  # vacuum
    gm = 0 if args.grad_mode == "adjoint" else 1
    rh = not args.no_hessian_recycling
    print(f"[bench] warmup {args.warmup} steps", file=sys.stderr, flush=True)
    if args.warmup > 0:
        ad = lib.Adapt(hl, cfg["pool"], psi0, max_iters=cfg["max_iters"], grad_mode=gm, recycle_hessian=rh)
        for _ in range(args.warmup):
            ad.step()
        ad.close()
    ad = lib.Adapt(hl, cfg["pool"], psi0, max_iters=cfg["max_iters"], grad_mode=gm, recycle_hessian=rh)
    layout = ad.layout()
    layout_desc = {lib.LAYOUT_FULL: "full d^L tensor (16,777,216 amplitudes)",
                   lib.LAYOUT_EVEN: "parity-halved, even sector (8,388,608 stored amplitudes)",
                   lib.LAYOUT_ODD: "parity-halved, odd sector (8,388,608 stored amplitudes)"}[layout]
    if ad.real():
        layout_desc += "; real float32 amplitudes for evaluations whose gates are all HR or PR"
        if lib.get_real_fusion() == lib.RFUSE_ON:
            layout_desc += ", runs of gates inside three consecutive modes fused into one pass"
    lib.prof_set_sample(args.prof_sample)
    lib.prof_reset()
    lib.prof_enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    reps = []
    snaps = {}
    for k in range(args.steps):
        reps.append(ad.step())
        if (k + 1) % 5 == 0 or k + 1 == 3:  # host copy of the angles for the oracle replay (after the timed region)
            snaps[k + 1] = ad.ansatz()
        print(f"[bench] step {k + 1}: E={reps[-1]['E']:.8f} evals={reps[-1]['bfgs_evals']}", file=sys.stderr,
              flush=True)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    lib.prof_enable(False)
    prof = {kid: lib.prof_query(kid) for kid in KERNEL_NAMES}
    ops_final = ad.ansatz()[0]
    real_run = ad.real()
    ad.close()
    dt = t1 - t0
    value = args.steps / dt

    def kernel_entry(kid):
        p = prof[kid]
        if p["launches"] == 0:
            return None
        per_launch_bytes = p["bytes"] / p["launches"]
        avg_ms = p["ms"] / p["launches"]
        gbs = per_launch_bytes / (avg_ms * 1e-3) / 1e9
        return {"bound": "hbm", "achieved": gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": gbs / HBM_PEAK_GBS,
                "traffic": traffic_for(kid), "kernel": KERNEL_NAMES[kid], "launches": p["launches"],
                "event_sample": args.prof_sample,
                "avg_us": avg_ms * 1e3, "algorithmic_bytes_per_launch": per_launch_bytes,
                "total_ms": p["ms"]}

    # Fused runs carry several gates per launch; their algorithmic bytes are
    # one pass.  Gates per fused launch, from the run planner applied to each
    # step's ansatz, weighted by the step's evaluations (forward runs also
    # prepare the step's scoring); "gate_equivalent_GBs" counts every gate's pass.
    fused_gpl = {}
    if real_run and lib.get_real_fusion() == lib.RFUSE_ON:
        hf = lib.ham_from(cfg, layout=layout | lib.LAYOUT_REAL)
        for kid, extra in ((14, 1), (15, 0)):
            g_sum = l_sum = 0
            for r in reps:
                n_s = r["n_params"]
                order = lib.real_fusion_order(hf, ops_final[:n_s])  # as the evaluations run them
                runs = lib.real_fusion_plan(hf, [ops_final[k] for k in order])
                ends = [k0 for k0, _ in runs[1:]] + [n_s]
                for (k0, a), k1 in zip(runs, ends):
                    if a >= 0:
                        w = r["bfgs_evals"] + extra
                        g_sum += w * (k1 - k0)
                        l_sum += w
            if l_sum:
                fused_gpl[kid] = g_sum / l_sum

    def with_gates(kid, e):
        if e is not None and kid in fused_gpl:
            e["gates_per_launch"] = fused_gpl[kid]
            e["gate_equivalent_GBs"] = e["achieved"] * fused_gpl[kid]
            e["gate_equivalent_frac"] = e["gate_equivalent_GBs"] / HBM_PEAK_GBS
        return e

    dom = max((k for k in KERNEL_NAMES if prof[k]["launches"]), key=lambda k: prof[k]["ms"])
    roof = with_gates(dom, kernel_entry(dom))
    ed = None
    edp = os.path.join(ROOT, "tests", "golden", "ed_reference.json")
    if os.path.exists(edp):
        ed = json.load(open(edp)).get("kk_l8_d8", {}).get("E0")
    evals = float(np.mean([r["bfgs_evals"] for r in reps]))
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "ADAPT steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * dt / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64",
        "data": "synthetic",
        "config": {"workload": (f"Kitaev-Kerr open chain L=8 d=8 (16,777,216 amplitudes), J=1 Delta=0.5 K=0.2, "
                                f"vacuum start, 28-op nearest-neighbour pool, ADAPT steps 1..{args.steps} with "
                                f"{args.grad_mode} BFGS gradients"
                                f"{', inverse Hessian recycled across steps' if rh else ''}; states kept "
                                f"{layout_desc}"),
                   "L": 8, "d": 8, "pool": len(cfg["pool"]), "grad_mode": args.grad_mode, "hessian_recycling": rh,
                   "gate_fusion": lib.get_gate_fusion(), "real_fusion": lib.get_real_fusion() == lib.RFUSE_ON,
                   "state_layout": layout_desc},
        "roofline": roof,
        # H psi of the timed evaluations: on real states when the run uses them
        "apply_h": kernel_entry(13) if prof[13]["launches"] else kernel_entry(0),
        "kernels": {KERNEL_NAMES[k]: with_gates(k, kernel_entry(k)) for k in KERNEL_NAMES if prof[k]["launches"]},
        "adapt": {"E_final": reps[-1]["E"], "E0_ed": ed, "dE_vs_ed": (reps[-1]["E"] - ed) if ed is not None else None,
                  "tolerance_reached": (abs(reps[-1]["E"] - ed) <= 1e-5 * abs(ed)) if ed is not None else None,
                  "note": ("the timed steps are the first steps of the run, far from the ground state; the ED gap "
                           "is reported, and per-step parity is the oracle replay below"),
                  "bfgs_evals_per_step": evals, "n_params": reps[-1]["n_params"],
                  "selected": [r["k_sel"] for r in reps]},
    }
    # the same workload by other gradient / optimiser settings (steps 1..k of a fresh run each)
    def variant(k, **kw):
        a = lib.Adapt(hl, cfg["pool"], psi0, max_iters=cfg["max_iters"], **kw)
        torch.cuda.synchronize()
        t = time.perf_counter()
        rs = [a.step() for _ in range(k)]
        torch.cuda.synchronize()
        dt_v = time.perf_counter() - t
        a.close()
        return {"steps": k, "steps_per_s": k / dt_v, "E_final": rs[-1]["E"],
                "bfgs_evals_per_step": float(np.mean([r["bfgs_evals"] for r in rs])),
                "bfgs_iters_per_step": float(np.mean([r["bfgs_iters"] for r in rs]))}

    def variant_graph(k):
        """The same point through the batched engine: persistent kernels and one
        captured graph replayed per BFGS round (fresh Hessian)."""
        sw = lib.Sweep([dict(ham=hl, pool=cfg["pool"], psi0=psi0, warm_ops=[], warm_theta0=np.zeros(0))],
                       max_iters=cfg["max_iters"])
        sw.autotune(None)
        torch.cuda.synchronize()
        t = time.perf_counter()
        rs = [sw.step()[0][0] for _ in range(k)]
        torch.cuda.synchronize()
        dt_v = time.perf_counter() - t
        sw.close()
        return {"steps": k, "steps_per_s": k / dt_v, "E_final": rs[-1]["E"],
                "bfgs_evals_per_step": float(np.mean([r["bfgs_evals"] for r in rs])),
                "bfgs_iters_per_step": float(np.mean([r["bfgs_iters"] for r in rs]))}

    if not args.no_variants and args.grad_mode == "adjoint":
        print("[bench] variants: central-difference gradients, Hessian recycling", file=sys.stderr, flush=True)
        main = {"steps": args.steps, "steps_per_s": value, "E_final": reps[-1]["E"], "bfgs_evals_per_step": evals,
                "bfgs_iters_per_step": float(np.mean([r["bfgs_iters"] for r in reps]))}
        out["variants"] = {
            "plain_fd_gradients": variant(args.steps, grad_mode=1),
            "adjoint": main if not rh else variant(args.steps),
            "adjoint_hessian_recycling": main if rh else variant(args.steps, recycle_hessian=True),
            "adjoint_graph_replay": variant_graph(args.steps),
        }
        # the headline's state representations switched off one at a time, then both
        for name, sector, real, fuse in (("unfused", lib.SECTOR_AUTO, lib.REAL_AUTO, lib.RFUSE_OFF),
                                         ("full_layout", lib.SECTOR_OFF, lib.REAL_AUTO, lib.RFUSE_ON),
                                         ("complex_states", lib.SECTOR_AUTO, lib.REAL_OFF, lib.RFUSE_ON),
                                         ("full_layout_complex_states", lib.SECTOR_OFF, lib.REAL_OFF, lib.RFUSE_ON)):
            lib.set_sector_layout(sector)
            lib.set_real_states(real)
            lib.set_real_fusion(fuse)
            try:
                out["variants"]["adjoint_hessian_recycling_" + name] = variant(args.steps, recycle_hessian=rh)
            finally:
                lib.set_sector_layout(lib.SECTOR_AUTO)
                lib.set_real_states(lib.REAL_AUTO)
                lib.set_real_fusion(lib.RFUSE_ON)
    if not args.no_variants and args.grad_mode == "adjoint" and not args.no_warm_start:
        print("[bench] warm-start leg: training data from 8 nearby points, network, proposals after selection",
              file=sys.stderr, flush=True)
        out["warm_start"] = warm_start_leg(cfg, hl, psi0, args.steps, out["variants"]["adjoint_hessian_recycling"])
    if not args.no_cpu_baseline and 3 in snaps:
        print("[bench] oracle on the host: replay of steps 5/10/15/20 and the steps 1-3 timing sample", file=sys.stderr,
              flush=True)
        p0 = np.zeros(n, dtype=np.complex128)
        p0[0] = 1.0
        out["cpu_baseline"], out["replay_checked_steps"] = cpu_leg(cfg, p0, snaps, reps)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
