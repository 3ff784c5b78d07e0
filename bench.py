#!/usr/bin/env python3
"""HAP benchmark on one MI355X: N^2*L message updates per second.

Workload: 8192 points in 2-D from 64 Gaussian blobs (centres U[-100,100]^2,
sigma U[0.5,2], multinomial sizes), FP32 similarity, L = 3 levels, damping 0.9,
median preference, up to 500 iterations or 50 iterations with unchanged labels.
Synthetic data from paper_1403_7394_amd.synth (seed 1002).

One step is one pass of the whole hot path with the points already on the GPU:
similarity build, median preference and initial state, the sweeps until the
stop rule, exemplars of every level and the FP64 net similarity.  `value` is
N^2*L*(sweeps performed) / (wall time of the timed steps).  The row pass runs in
points mode (s_ij recomputed from the 2-D points, bit-identical to reading S;
--read-s reads S instead).

The roofline entry is for the dominant kernel, the fused row pass: its
algorithmic traffic (read R, A and write R, A: 4 N^2 words per level per sweep,
3 N^2 in the first sweep, which has no alpha to finish; 5 N^2 and 4 N^2 when S is
read) divided by its average launch duration, measured with HIP events recorded
on its own stream around the launches of every 8th sweep of the timed steps.
The L = 3 run does not meet the stop rule under the literal Eq. 2.6, so the line
also times, once each, the same workload at L = 1 and with the optional Eq. 2.7
update (kappa = 0.5), which do, from the points on the GPU to the labels
(`converging_variants`).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "HAP N²·L message updates/s and time-to-converge vs plain, same GPU"
HBM_PEAK_GBS = 8000.0
TRAFFIC_FILES = {True: os.path.join(ROOT, "profiles", "row_pass_traffic_plain8192_points.json"),
                 False: os.path.join(ROOT, "profiles", "row_pass_traffic_plain8192.json")}
SWEEP_SRC = os.path.join(ROOT, "paper_1403_7394_amd", "csrc", "sweep.hip")
ROWPASS_SRC = os.path.join(ROOT, "paper_1403_7394_amd", "csrc", "rowpass.h")
FLOWPASS_SRC = os.path.join(ROOT, "paper_1403_7394_amd", "csrc", "flowpass.h")
PROF_EVERY = 8


def _hash16(path: str) -> str:
    with open(path, "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()[:16]


def measured_traffic(points: bool, first_launches: int, steady_launches: int):
    """HBM bytes per row-pass launch from the committed counter summary (FETCH_SIZE and
    WRITE_SIZE scaled by a 1 GiB device copy), weighted over this run's first-sweep and
    later launches; None unless the counters were taken on the current kernel source."""
    try:
        with open(TRAFFIC_FILES[points]) as f:
            t = json.load(f)
    except (OSError, ValueError):
        return None
    if (t.get("sweep_source_sha256_16") != _hash16(SWEEP_SRC)
            or t.get("rowpass_source_sha256_16") != _hash16(ROWPASS_SRC)
            or t.get("flowpass_source_sha256_16") != _hash16(FLOWPASS_SRC)):
        return None
    total = first_launches + steady_launches
    if total == 0:
        return None
    return (first_launches * t["hbm_bytes_per_launch_first"]
            + steady_launches * t["hbm_bytes_per_launch_steady"]) / total


def cpu_baseline(X, rp, sweeps: int = 2):
    """The FP64 NumPy oracle on the same workload: `sweeps` full sweeps (all levels), timed."""
    import numpy as np

    from oracle import hap_ref
    from oracle import similarity as sim

    S32 = sim.similarity(X).astype(np.float32)
    p = float(sim.median_offdiag(S32, np.float32))
    S64 = S32.astype(np.float64)
    n = X.shape[0]
    w0, c0 = time.perf_counter(), time.process_time()
    hap_ref.hap(S64, p, rp.levels, rp.damping, sweeps)
    wall, cpu = time.perf_counter() - w0, time.process_time() - c0
    return {
        "value": n * n * rp.levels * sweeps / wall,
        "unit": "updates/s",
        "cores": max(1, round(cpu / wall)),
        "kind": "oracle",
        "sample": f"first {sweeps} of up to {rp.max_iters} sweeps (all {rp.levels} levels) of the same "
                  f"{n}-point workload, FP64 NumPy oracle; similarity build and median not timed",
        "seconds": wall,
        "host": _host_info(),
    }


def _host_info() -> dict:
    """CPU count, usable cores and CPU model of the machine the oracle ran on."""
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"cpu_count": os.cpu_count(), "affinity": len(os.sched_getaffinity(0)), "model": model}


def run_precision_form(args, torch, hap, synth) -> dict:
    """Precision form: the similarity of the 32768-point, 64-dimensional workload built four
    ways (FP64-accumulated direct build = plain; FP32 GEMM, BF16 and BF16x3 on the matrix
    cores), each followed by the same HAP run (L=4, damping 0.9, 300 iterations).  Every label
    that differs from the direct build's run is reported with its decision margin in that run:
    (alpha + rho)(i, e_direct) - (alpha + rho)(i, e_mode), in units of |p|."""
    import numpy as np
    dev = torch.device("cuda:0")
    blobs, rp = synth.workload_precision()
    n, d = blobs.X.shape
    L = rp.levels
    iters = args.form_iters if args.form_iters else rp.max_iters
    X = torch.from_numpy(blobs.X).to(dev)
    S = torch.empty((n, n), dtype=torch.float32, device=dev)
    S_direct = torch.empty((n, n), dtype=torch.float32, device=dev)
    ws = torch.empty(hap.workspace_size(n, L, hap.HAP_F32), dtype=torch.uint8, device=dev)
    ws_direct = torch.empty_like(ws)
    rng = np.random.default_rng(7)
    pi = rng.integers(0, n, size=1_000_000)
    pj = rng.integers(0, n, size=1_000_000)
    keep = pi != pj
    pi, pj = pi[keep], pj[keep]
    X64 = blobs.X.astype(np.float64)
    ref = -np.sum((X64[pi] - X64[pj]) ** 2, axis=1)
    same = blobs.truth[pi] == blobs.truth[pj]
    pit, pjt = torch.from_numpy(pi).to(dev), torch.from_numpy(pj).to(dev)
    modes = [("direct", hap.BUILD_DIRECT), ("gemm_f32", hap.BUILD_GEMM), ("bf16", hap.BUILD_BF16),
             ("bf16x3", hap.BUILD_BF16X3)]
    results = {}
    base_labels = None
    h_direct = None
    prefs = None
    scores = {}

    def direct_scores(l):
        # (alpha + rho) of the direct build's run at level l (n x n, on the device)
        if l not in scores:
            m = h_direct.messages(l)
            scores.clear()
            scores[l] = m["alpha"].add_(m["rho"])
            del m
        return scores[l]

    for name, mode in modes:
        Sm = S_direct if mode == hap.BUILD_DIRECT else S
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        hap.build_similarity(X, Sm, mode=mode)
        e1.record()
        torch.cuda.synchronize()
        build_ms = e0.elapsed_time(e1)
        got = Sm[pit, pjt].double().cpu().numpy()
        err = np.abs(got - ref)
        t0 = time.perf_counter()
        hap.build_similarity(X, Sm, mode=mode)
        h = hap.Hap(Sm, L, rp.damping, workspace=ws_direct if mode == hap.BUILD_DIRECT else ws)
        torch.cuda.synchronize()
        ts0 = time.perf_counter()
        h.iterate(iters, 0)
        torch.cuda.synchronize()
        sweep_s = time.perf_counter() - ts0
        labels = h.labels()
        counts = [h.exemplars(l)[1] for l in range(L)]
        ns = [h.net_similarity(l, X=X) for l in range(L)]
        torch.cuda.synchronize()
        ttc = time.perf_counter() - t0
        margins = None
        if base_labels is None:
            base_labels, base_ns, h_direct = labels, ns, h
            prefs = h.preference()
        else:
            h.close()
            margins = []
            for l in range(L):
                diff = torch.nonzero(labels[l] != base_labels[l]).flatten()
                if diff.numel() == 0:
                    margins.append({"count": 0})
                    continue
                v = direct_scores(l)[diff]
                mg = (v.gather(1, base_labels[l][diff].long()[:, None]) - v.gather(1, labels[l][diff].long()[:, None]))
                mg = (mg.flatten().double() / abs(prefs[l])).cpu().numpy()
                del v
                margins.append({"count": int(diff.numel()), "min": float(mg.min()), "median": float(np.median(mg)),
                                "max": float(mg.max()),
                                "below_1e-6": int(np.sum(mg < 1e-6)), "below_1e-3": int(np.sum(mg < 1e-3))})
        agree = [(labels[l] == base_labels[l]).float().mean().item() for l in range(L)]
        flops = 2.0 * n * n * d * (3 if mode == hap.BUILD_BF16X3 else 1)
        results[name] = {
            "build_ms": build_ms,
            "build_write_GBs": n * n * 4 / (build_ms * 1e-3) / 1e9,
            "build_TFLOPs": flops / (build_ms * 1e-3) / 1e12 if mode != hap.BUILD_DIRECT else None,
            "S_max_abs_err": float(err.max()),
            "S_max_rel_err": float((err / np.abs(ref)).max()),
            "S_within_blob_max_rel_err": float((err[same] / np.abs(ref[same])).max()) if same.any() else None,
            "time_to_converge_s": ttc,
            "sweeps_s": sweep_s,
            "build_share_of_wall": build_ms * 1e-3 / ttc,
            "label_agreement_vs_direct": agree,
            "net_similarity_rel_diff_vs_direct": [abs(a - b) / abs(b) for a, b in zip(ns, base_ns)],
            "disagreement_margins_vs_direct": margins,
            "exemplars_per_level": counts,
        }
        print(json.dumps({"form": "precision", "mode": name, **results[name]}), file=sys.stderr, flush=True)
    scores.clear()
    h_direct.close()
    return {"form": "precision", "workload": "32768 points, d=64, 256 blobs, FP32, L=4, damping 0.9, "
            f"{iters} iterations", "n": n, "d": d,
            "note": "the wall time is bound by the sweeps (iterations x L row passes over 32768^2), not "
                    "by the build, so a faster build cannot shorten it appreciably",
            "margin_units": "|p| of the level; margin = (alpha+rho)(i, e_direct) - (alpha+rho)(i, e_mode) "
                            "in the direct build's run",
            "results": results}


def run_batched_form(args, torch, hap, synth) -> dict:
    """Batched form: 512 independent problems (N ~ U{64..2048}, d=16, L=3, damping 0.8,
    200 iterations) in one persistent launch, against the plain single-problem path run
    problem by problem on the same GPU (with the column sums in the batch's order: row order
    for a problem one workgroup runs, member order of row blocks for a problem a gang shares,
    so the two compute the same trajectory).  The autotuner picks the launch shape and the
    split of the large problems over gangs of workgroups."""
    import numpy as np

    from paper_1403_7394_amd import autotune
    dev = torch.device("cuda:0")
    problems, rp = synth.workload_batched()
    iters = args.form_iters if args.form_iters else rp.max_iters
    sizes = [b.X.shape[0] for b in problems]
    X = torch.from_numpy(np.concatenate([b.X for b in problems])).to(dev)
    L = rp.levels
    bt = hap.HapBatch(sizes, 16, L)
    if args.batch_split:
        shape = tuple(int(v) for v in args.batch_launch.split(","))
        bt.set_launch(*shape)
        bt.set_split(*(int(v) for v in args.batch_split.split(",")))
        shape = shape + bt.get_split()
    else:
        shape = autotune.tune_batch(bt, X, rp.damping)
    members, rows = bt.members()
    print(json.dumps({"form": "batched", "step": "tuned", "launch": shape}), file=sys.stderr, flush=True)
    out = bt.outputs(dev)
    bt.run(X, rp.damping, iters, out=out)          # warm-up
    torch.cuda.synchronize()
    reps = max(1, args.steps)
    t0 = time.perf_counter()
    for _ in range(reps):
        bt.run(X, rp.damping, iters, out=out)
    torch.cuda.synchronize()
    t_batch = (time.perf_counter() - t0) / reps
    labels_b, ns_b, iters_b = out
    print(json.dumps({"form": "batched", "step": "batch timed", "s": t_batch}), file=sys.stderr, flush=True)
    # the plain path, one problem after another, with one reused workspace and S buffer: timed at its
    # default launch (the speed baseline), and on a sample of problems run with the batch's
    # column-sum order (row order for a problem one workgroup runs, member order of row blocks for
    # a problem a gang shares), where the two must give identical labels
    nmax = max(sizes)
    S = torch.empty((nmax, nmax), dtype=torch.float32, device=dev)
    ws = torch.empty(hap.workspace_size(nmax, L, hap.HAP_F32), dtype=torch.uint8, device=dev)

    def plain(bidx, rows_per_block=0):
        n = sizes[bidx]
        o = bt.offsets[bidx]
        Sv = S[:n, :n]
        hap.build_similarity(X[o:o + n], Sv)
        h = hap.Hap(Sv, L, rp.damping, workspace=ws)
        if rows_per_block:
            # a gang member owns a contiguous block of rows: the plain path's HAP_LAUNCH_BLOCKS order
            h.set_launch(rows_per_block=rows_per_block, blocks=True)
        h.iterate(iters, 0)
        lab = h.labels()
        ns = h.net_similarity(-1)
        h.close()
        return lab, ns

    agree_default = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for bidx in range(len(problems)):
        lab, _ = plain(bidx)
        agree_default.append(float((lab == bt.labels_of(labels_b, bidx)).float().mean().item()))
        if bidx % 128 == 127:
            print(json.dumps({"form": "batched", "step": f"plain path {bidx + 1}/{len(problems)}",
                              "s": time.perf_counter() - t0}), file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    t_plain = time.perf_counter() - t0
    split_ids = [b for b in range(len(sizes)) if members[b] > 1]
    whole_ids = [b for b in range(len(sizes)) if members[b] == 1]
    rng = np.random.default_rng(5)
    check = sorted(rng.choice(whole_ids, size=min(48, len(whole_ids)), replace=False).tolist() +
                   (rng.choice(split_ids, size=min(6, len(split_ids)), replace=False).tolist() if split_ids else []))
    identical, ns_rel = 0, []
    for bidx in check:
        lab, ns = plain(bidx, rows[bidx] if members[bidx] > 1 else 1)
        identical += int(torch.equal(lab, bt.labels_of(labels_b, bidx)))
        ns_rel.append(abs(ns - ns_b[bidx, L].item()) / abs(ns))
    print(json.dumps({"form": "batched", "step": "parity sample", "identical": identical, "checked": len(check)}),
          file=sys.stderr, flush=True)
    upd = float(sum(n * n for n in sizes)) * L * iters
    # algorithmic traffic of the sweeps: per element, level and iteration read S, R, A and write
    # R, A (12 + 8 bytes)
    alg_bytes = upd * 20.0
    bt.close()
    # a batch of fewer, large problems (the 16 largest of the workload): one workgroup per problem
    # leaves most of the device idle, gangs spread each problem over several workgroups
    few = sorted(range(len(sizes)), key=lambda b: -sizes[b])[:16]
    Xf = torch.cat([X[bt.offsets[b]:bt.offsets[b] + sizes[b]] for b in few])
    few_sizes = [sizes[b] for b in few]
    bf = hap.HapBatch(few_sizes, 16, L)
    bf.set_launch(shape[0], shape[1], shape[2])
    few_out = {}
    for split in ((0, 1), (256, 16)):
        bf.set_split(*split)
        of = bf.outputs(dev)
        bf.run(Xf, rp.damping, iters, out=of)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        bf.run(Xf, rp.damping, iters, out=of)
        torch.cuda.synchronize()
        few_out["split_%d_%d" % split] = {"s": time.perf_counter() - t0, "workgroups_busy": int(sum(bf.members()[0])),
                                          "iters_min": int(of[2].min().item())}
    bf.close()
    print(json.dumps({"form": "batched", "step": "few large problems", **few_out}), file=sys.stderr, flush=True)
    return {"form": "batched", "workload": f"{len(sizes)} problems, N ~ U{{64..2048}}, d=16, L={L}, "
            f"damping {rp.damping}, {iters} iterations", "sum_n2": int(sum(n * n for n in sizes)),
            "launch": {"threads": shape[0], "workgroups": shape[1], "row_groups": shape[2],
                       "split_n": shape[3], "max_members": shape[4]},
            "problems_split": int(sum(k > 1 for k in members)), "gang_members_total": int(sum(members)),
            "batched_s": t_batch, "plain_default_launch_s": t_plain, "speedup_vs_plain": t_plain / t_batch,
            "batched_updates_per_s": upd / t_batch, "plain_updates_per_s": upd / t_plain,
            "roofline": {"bound": "hbm", "achieved": alg_bytes / t_batch / 1e9, "peak": HBM_PEAK_GBS,
                         "unit": "GB/s", "frac": alg_bytes / t_batch / 1e9 / HBM_PEAK_GBS,
                         "alg_bytes": alg_bytes, "kernel": "batch_kernel (whole run, wall time of the launch)"},
            "iters_min": int(iters_b.min().item()),
            "few_large_problems": {"problems": 16, "sizes": f"{min(few_sizes)}..{max(few_sizes)}", **few_out},
            "label_agreement_vs_plain_default_min": min(agree_default),
            "label_agreement_vs_plain_default_mean": float(np.mean(agree_default)),
            "parity_sample": {"problems_checked": len(check), "split_problems_checked": sum(members[b] > 1 for b in check),
                              "identical_labels": identical, "net_similarity_rel_diff_max": max(ns_rel)},
            "problems": len(sizes)}


def run_warm_form(args, torch, hap, synth) -> dict:
    from paper_1403_7394_amd import metrics
    """Warm-start form: a perceptron trained on HAP runs of 2-D blob problems (8192 points,
    k in {3, 8, 16, 32, 64}, 5 seeds each) predicts the warm initial availabilities of the
    65536-point, 32-dimensional, 1024-blob workload; the warm run (with the cold start as
    fallback) is compared with the cold run on the same GPU, at L = 3 (the workload's levels)
    and at L = 1."""
    import numpy as np
    dev = torch.device("cuda:0")
    blobs, rp = synth.workload_warm_eval()
    n_eval = blobs.X.shape[0]
    iters = args.form_iters if args.form_iters else rp.max_iters
    K = rp.stable_iters
    kappa = args.kappa
    out = {"form": "warm", "workload": f"{n_eval} points, d=32, 1024 blobs, FP32, damping {rp.damping}, "
           f"up to {iters} iterations or {K} stable; network trained on 25 runs of 8192 2-D points",
           "kappa": kappa, "levels": {}}
    n_tr = 8192
    S_tr = torch.empty((n_tr, n_tr), dtype=torch.float32, device=dev)
    for L in [int(v) for v in args.warm_levels.split(",")]:
        t0 = time.perf_counter()
        ws = torch.empty(hap.workspace_size(n_tr, L, hap.HAP_F32), dtype=torch.uint8, device=dev)
        Fs, Ts, conv_tr = [], [], 0
        for k in (3, 8, 16, 32, 64):
            for rep in range(5):
                b = synth.workload_warm_train(k, rep, n=n_tr)
                hap.build_similarity(torch.from_numpy(b.X).to(dev), S_tr)
                h = hap.Hap(S_tr, L, rp.damping, workspace=ws, kappa=kappa if L > 1 else 0.0)
                res = h.iterate(iters, K)
                conv_tr += int(res.converged)
                Fs.append(h.warm_features())
                Ts.append(h.warm_targets())
                h.close()
        del ws
        F = torch.cat(Fs)
        T = torch.cat(Ts)
        torch.cuda.synchronize()
        t_data = time.perf_counter() - t0
        batch, steps = 4096, 3000
        m = hap.Mlp(torch.from_numpy(synth.mlp_init(3000 + L, hap.WARM_FEATURES, 128, L)).to(dev),
                    hap.WARM_FEATURES, 128, L, precision=hap.HAP_BF16)
        idx = torch.from_numpy(synth.minibatch_order(4000 + L, F.shape[0], batch, steps)).to(dev)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        hist = m.train(F, T, idx, batch, steps, 1e-3)
        torch.cuda.synchronize()
        t_train = time.perf_counter() - t0
        hist = hist.cpu().numpy()
        del F, T, idx
        print(json.dumps({"form": "warm", "levels": L, "train_runs_converged": conv_tr, "data_s": t_data,
                          "train_s": t_train, "loss_first": float(hist[:50].mean()),
                          "loss_last": float(hist[-50:].mean())}), file=sys.stderr, flush=True)

        X = torch.from_numpy(blobs.X).to(dev)
        S = torch.empty((n_eval, n_eval), dtype=torch.float32, device=dev)
        hap.build_similarity(X, S)
        ws = torch.empty(hap.workspace_size(n_eval, L, hap.HAP_F32), dtype=torch.uint8, device=dev)

        def run(mode: str):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            h = hap.Hap(S, L, rp.damping, workspace=ws, kappa=kappa if L > 1 else 0.0)
            fell, t_pred, extra = False, 0.0, {}
            if mode != "cold":
                Y = m.forward(h.warm_features())
                torch.cuda.synchronize()
                t_pred = time.perf_counter() - t0
            if mode == "warm":
                res, fell = h.iterate_warm(Y, iters, K)
            elif mode == "judged":
                res, fell, ns_w, ns_c = h.iterate_warm_judged(Y, iters, K, X=X)
                extra = {"judge_ns_warm_fp64": ns_w, "judge_ns_cold_fp64": ns_c}
            else:
                res = h.iterate(iters, K)
            labels = h.labels().cpu().numpy()
            counts = [h.exemplars(l)[1] for l in range(L)]
            ns = [h.net_similarity(l) for l in range(L)]
            torch.cuda.synchronize()
            wall = time.perf_counter() - t0
            h.close()
            return dict(iters=res.iters, converged=res.converged, fell_back=fell, wall_s=wall,
                        predict_s=t_pred, exemplars_per_level=counts, net_similarity=ns, **extra), labels

        cold, lab_c = run("cold")
        print(json.dumps({"form": "warm", "levels": L, "cold": cold}), file=sys.stderr, flush=True)
        warm_r, lab_w = run("warm")
        print(json.dumps({"form": "warm", "levels": L, "warm": warm_r}), file=sys.stderr, flush=True)
        judged, lab_j = run("judged")
        print(json.dumps({"form": "warm", "levels": L, "judged": judged}), file=sys.stderr, flush=True)
        # sweeps performed: a converged run stops one sweep after its stop iteration
        sw = lambda r: (r["iters"] + 1) if (r["converged"] and r["iters"] < iters) else r["iters"]
        warm_sweeps = sw(warm_r) + (iters if warm_r["fell_back"] else 0)
        out["levels"][str(L)] = {
            "train": {"runs": 25, "runs_converged": conv_tr, "samples": 25 * n_tr, "batch": batch,
                      "steps": steps, "lr": 1e-3, "precision": "bf16", "data_s": t_data, "train_s": t_train,
                      "loss_first50": float(hist[:50].mean()), "loss_last50": float(hist[-50:].mean())},
            "cold": cold, "warm": warm_r,
            # the judged form (opt-in) runs both starts and keeps the larger FP64 net similarity
            "judged": judged, "judged_equals_cold": bool(np.array_equal(lab_j, lab_c)),
            "sweeps_cold": sw(cold), "sweeps_warm_total": warm_sweeps,
            "wall_ratio_warm_over_cold": warm_r["wall_s"] / cold["wall_s"],
            "exemplar_agreement": [float(np.mean(lab_c[l] == lab_w[l])) for l in range(L)],
            "purity_cold": [metrics.purity(lab_c[l], blobs.truth) for l in range(L)],
            "purity_warm": [metrics.purity(lab_w[l], blobs.truth) for l in range(L)],
            "adjusted_rand_index": [metrics.adjusted_rand_index(lab_c[l], lab_w[l]) for l in range(L)],
            "net_similarity_rel_diff": [(a - b) / abs(b) for a, b in zip(warm_r["net_similarity"],
                                                                       cold["net_similarity"])],
        }
        del S, ws, X
        # held-out problems from the training distribution (2-D, 8192 points, new k and seeds)
        held = []
        ws_h = torch.empty(hap.workspace_size(n_tr, L, hap.HAP_F32), dtype=torch.uint8, device=dev)
        for k in (5, 12, 24, 48, 96):
            b = synth.gaussian_blobs(9001 + k, n_tr, 2, k, centre="uniform", centre_scale=10.0, sigma_lo=1.0,
                                     sigma_hi=1.0, sizes="multinomial", dtype=np.float32)
            hap.build_similarity(torch.from_numpy(b.X).to(dev), S_tr)
            rows = {}
            for warm in (False, True, "judged"):
                h = hap.Hap(S_tr, L, rp.damping, workspace=ws_h, kappa=kappa if L > 1 else 0.0)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                if warm == "judged":
                    res, fell, _, _ = h.iterate_warm_judged(m.forward(h.warm_features()), iters, K)
                elif warm:
                    res, fell = h.iterate_warm(m.forward(h.warm_features()), iters, K)
                else:
                    res, fell = h.iterate(iters, K), False
                lab = h.labels().cpu().numpy()
                torch.cuda.synchronize()
                rows[warm] = (res, fell, time.perf_counter() - t0, lab, h.net_similarity(-1))
                h.close()
            (rc_, _, tc, lc, nc), (rw_, fw, tw, lw, nw) = rows[False], rows[True]
            rj_, fj, tj, lj, nj = rows["judged"]
            held.append({"k": k, "cold_iters": rc_.iters, "cold_converged": rc_.converged, "warm_iters": rw_.iters,
                         "warm_converged": rw_.converged, "fell_back": fw, "cold_s": tc, "warm_s": tw,
                         "exemplar_agreement": float(np.mean(lc == lw)),
                         "purity_cold": [metrics.purity(lc[l], b.truth) for l in range(L)],
                         "purity_warm": [metrics.purity(lw[l], b.truth) for l in range(L)],
                         "adjusted_rand_index": [metrics.adjusted_rand_index(lc[l], lw[l]) for l in range(L)],
                         "net_similarity_rel_diff": (nw - nc) / abs(nc),
                         "judged_kept": "cold" if fj else "warm", "judged_s": tj,
                         "judged_net_similarity_rel_diff": (nj - nc) / abs(nc)})
        out["levels"][str(L)]["held_out_2d_8192"] = held
        print(json.dumps({"form": "warm", "levels": L, "held_out": held}), file=sys.stderr, flush=True)
        del ws_h, m
        torch.cuda.empty_cache()
    return out


def run_profile_form(args, torch, hap, synth) -> int:
    """Short runs of one part of the hot path for hardware-counter profiling (rocprofv3); a
    line is printed after each step, every kernel runs on torch's current stream.

    sweeps: the FP32 similarity of the 2-D 64-blob workload (--n points, default 8192), then
      --sweeps full sweeps (L = 3, damping 0.9, no stop rule; points mode unless --read-s;
      --rows R updates rows [0, R) only, one device's block of a run split by rows; --rb B sets
      the rows per workgroup, --sweep-launch the whole row-pass shape; --schedule mrhap runs
      the MapReduce schedule, whose levels share one row-pass launch unless --unfused), after
      one device copy of --copy-gib GiB whose counter readings calibrate the HBM byte counters.
    builds: the similarity of the 32768-point, 64-dimensional workload built once in each mode
      (direct, FP32 GEMM, BF16, BF16x3).
    batch-once: the batched workload run once for --form-iters iterations (default 200) in the
      launch shape --batch-launch, after the calibration copy."""
    import numpy as np
    dev = torch.device("cuda:0")
    if args.form == "builds":
        blobs, _ = synth.workload_precision()
        n = blobs.X.shape[0]
        X = torch.from_numpy(blobs.X).to(dev)
        S = torch.empty((n, n), dtype=torch.float32, device=dev)
        for name, mode in (("direct", hap.BUILD_DIRECT), ("gemm_f32", hap.BUILD_GEMM), ("bf16", hap.BUILD_BF16),
                           ("bf16x3", hap.BUILD_BF16X3)):
            hap.build_similarity(X, S, mode=mode)
            torch.cuda.synchronize()
            print(f"build {name}: {n} x {n} from d = {blobs.X.shape[1]}", flush=True)
        return 0
    if args.copy_gib > 0:
        words = int(args.copy_gib * (1 << 30)) // 4
        src = torch.ones(words, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        print(f"copy: {words * 4} bytes read, {words * 4} bytes written", flush=True)
        del src, dst
    if args.form == "batch-once":
        problems, rp = synth.workload_batched()
        iters = args.form_iters if args.form_iters else rp.max_iters
        sizes = [b.X.shape[0] for b in problems]
        X = torch.from_numpy(np.concatenate([b.X for b in problems])).to(dev)
        bt = hap.HapBatch(sizes, problems[0].X.shape[1], rp.levels)
        shape = tuple(int(v) for v in args.batch_launch.split(","))
        bt.set_launch(*shape)
        if args.batch_split:
            bt.set_split(*(int(v) for v in args.batch_split.split(",")))
        out = bt.outputs(dev)
        torch.cuda.synchronize()
        print(f"batch ready: {len(sizes)} problems, sum n^2 = {sum(k * k for k in sizes)}, launch {shape}", flush=True)
        bt.run(X, rp.damping, iters, out=out)
        torch.cuda.synchronize()
        print(f"batch done: {iters} iterations", flush=True)
        bt.close()
        return 0
    blobs, rp = synth.workload_plain_f32(n=args.n)
    n = blobs.X.shape[0]
    X = torch.from_numpy(blobs.X).to(dev)
    S = torch.empty((n, n), dtype=torch.float32, device=dev)
    hap.build_similarity(X, S)
    h = hap.Hap(S, rp.levels, rp.damping,
                schedule=hap.SCHEDULE_MRHAP if args.schedule == "mrhap" else hap.SCHEDULE_SEQUENTIAL)
    if args.unfused:
        h.set_launch(unfused=True)
    if args.rows:
        h.set_row_count(args.rows)
    if args.rb:
        h.set_launch(rows_per_block=args.rb)
    if args.sweep_launch:
        t_, c_, rb_, st_ = (int(v) for v in args.sweep_launch.split(","))
        h.set_launch(t_, c_, rb_, streaming=bool(st_))
    if args.blocks:
        h.set_launch(blocks=True)
    if not args.read_s:
        h.set_points(X)
    torch.cuda.synchronize()
    print(f"similarity and state ready: n={n} levels={rp.levels}", flush=True)
    res = h.iterate(args.sweeps)
    torch.cuda.synchronize()
    print(f"sweeps done: {res.iters}; launch {h.get_launch()}; rows {h.get_row_count()}", flush=True)
    h.close()
    return 0


def run_ceiling_form(args, torch, hap) -> dict:
    """What the row pass's read/write mixes reach on this GPU: the library's bandwidth probe over
    8192 x 8192 FP32 arrays, for a pure write (what the similarity builds do), a pure read, a
    copy, the points-mode mix (read and write rho and alpha) and the S-reading mix (read S, rho,
    alpha; write rho, alpha).  The row pass's own pattern is the probe's default (256 workgroups
    of 512 threads taking rows g, g + 256, ..., 16-byte non-temporal accesses); each mix with
    inputs is also run in place (the outputs are the last inputs, as the row pass updates rho
    and alpha), and with the probe's variants of cached loads after the first input and of
    contiguous blocks of 32 rows per workgroup; "best" is the fastest variant of each mix.  HIP
    events on the probe's stream, --steps repetitions each after two untimed ones."""
    dev = torch.device("cuda:0")
    n = 8192
    arrs = [torch.full((n, n), 1.0 + k, dtype=torch.float32, device=dev) for k in range(5)]
    sink = torch.zeros(1, dtype=torch.float32, device=dev)
    reps = max(5, args.steps)
    out = {"form": "ceiling", "arrays": f"{n} x {n} FP32", "peak_GBs": HBM_PEAK_GBS, "mixes": {}, "best": {}}
    for mix, r, w in (("write", 0, 1), ("read", 1, 0), ("copy", 1, 1), ("points_mix_2r2w", 2, 2),
                      ("s_mix_3r2w", 3, 2)):
        for inplace in ((False, True) if r and w else (False,)):
            for cached in ((False, True) if r > 1 else (False,)):
                for blocks in (False, True):
                    name = mix + ("_in_place" if inplace else "") + ("_cached" if cached else "") + \
                        ("_blocks" if blocks else "")
                    ins = arrs[:r]
                    outs = ins[r - w:] if inplace else arrs[r:r + w]
                    kw = dict(sink=sink, cached=cached, blocks=blocks)
                    for _ in range(2):
                        hap.bandwidth_probe(ins, outs, **kw)
                    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    torch.cuda.synchronize()
                    e0.record()
                    for _ in range(reps):
                        hap.bandwidth_probe(ins, outs, **kw)
                    e1.record()
                    torch.cuda.synchronize()
                    us = e0.elapsed_time(e1) * 1e3 / reps
                    gbs = (r + w) * n * n * 4 / (us * 1e-6) / 1e9
                    out["mixes"][name] = {"reads": r, "writes": w, "in_place": inplace, "cached": cached,
                                          "blocks": blocks, "avg_us": us, "GBs": gbs, "frac": gbs / HBM_PEAK_GBS}
                    if mix not in out["best"] or us < out["best"][mix]["avg_us"]:
                        out["best"][mix] = {"variant": name, "avg_us": us, "GBs": gbs, "frac": gbs / HBM_PEAK_GBS}
                    print(json.dumps({"mix": name, "avg_us": us, "GBs": gbs}), file=sys.stderr, flush=True)
    return out


def run_image_form(args, torch, hap, synth) -> dict:
    """Image-style form (Section 4): RGB pixels of the sizes of the paper's two images
    (103 x 103 and 120 x 100, from 16 colour blobs), negative Euclidean distances, random
    preferences U[-1e6, 0] per point, L = 3, damping 0.5, 30 iterations, FP32."""
    import numpy as np

    from paper_1403_7394_amd import metrics
    dev = torch.device("cuda:0")
    out = {"form": "image", "results": {}}
    for which in ("mandrill", "buttons"):
        blobs, prefs, rp = synth.workload_image(which)
        n = blobs.X.shape[0]
        L = rp.levels
        X = torch.from_numpy(blobs.X).to(dev)
        ld = n + (-n) % 4
        S = torch.empty((n, ld), dtype=torch.float32, device=dev)[:, :n]
        p = torch.from_numpy(prefs.astype(np.float32)).to(dev)
        ws = torch.empty(hap.workspace_size(n, L, hap.HAP_F32), dtype=torch.uint8, device=dev)
        times = []
        for rep in range(1 + max(1, args.steps)):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hap.build_similarity(X, S, mode=hap.BUILD_DIRECT_L2)
            h = hap.Hap(S, L, rp.damping, pref=p, workspace=ws)
            res = h.iterate(rp.max_iters)
            counts = [h.exemplars(l)[1] for l in range(L)]
            labels = h.labels()
            ns = [h.net_similarity(l) for l in range(L)]
            torch.cuda.synchronize()
            if rep > 0:
                times.append(time.perf_counter() - t0)
            h.close()
        lab = labels.cpu().numpy()
        t = float(np.mean(times))
        out["results"][which] = {
            "n": n, "levels": L, "iterations": res.iters, "seconds": t,
            "updates_per_s": n * n * L * res.iters / t,
            "exemplars_per_level": counts,
            "purity_per_level": [metrics.purity(lab[l], blobs.truth) for l in range(L)],
            "net_similarity_per_level": ns,
            "paper_exemplars_per_level": [15, 7, 6] if which == "mandrill" else [154, 25, 11],
        }
        del S, ws
    return out


def main() -> int:
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--no-cpu-baseline", action="store_true", help="skip the oracle timing")
    ap.add_argument("--no-converge-variants", action="store_true",
                    help="skip the L = 1 and kappa = 0.5 runs timed to the stop rule")
    ap.add_argument("--cpu-sweeps", type=int, default=5, help="sweeps of the oracle timed for cpu_baseline (about 13 s)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="also run a 1 GiB device copy (counter calibration under rocprofv3)")
    ap.add_argument("--form", choices=["plain", "precision", "batched", "warm", "image", "ceiling", "sweeps",
                                       "builds", "batch-once"], default="plain",
                    help="plain: the headline line; precision: the similarity build forms; "
                         "batched: many problems in one launch; warm: the learned warm start; "
                         "image: the paper's image-style workload (random preferences, Euclidean distance); "
                         "ceiling: bandwidth of the row pass's read/write mixes; "
                         "sweeps, builds, batch-once: short runs for counter profiling")
    ap.add_argument("--sweeps", type=int, default=4, help="--form sweeps: sweeps to run")
    ap.add_argument("--n", type=int, default=8192, help="--form sweeps: points")
    ap.add_argument("--rows", type=int, default=0, help="--form sweeps: update rows [0, rows) only (0: all)")
    ap.add_argument("--rb", type=int, default=0, help="--form sweeps: rows per workgroup (0: the default launch)")
    ap.add_argument("--unfused", action="store_true",
                    help="--form sweeps with --schedule mrhap: one row-pass launch per level")
    ap.add_argument("--sweep-launch", default="",
                    help="--form sweeps: row-pass shape threads,chunks,rows_per_block,streaming (empty: the default)")
    ap.add_argument("--blocks", action="store_true",
                    help="--form sweeps: each workgroup takes a contiguous block of rows (default: interleaved)")
    ap.add_argument("--copy-gib", type=float, default=1.0,
                    help="--form sweeps / batch-once: GiB of the calibration copy run first (0: none)")
    ap.add_argument("--batch-launch", default="1024,512,4",
                    help="--form batch-once (and --form batched with --batch-split): threads,workgroups,row_groups "
                         "of the persistent launch")
    ap.add_argument("--batch-split", default="",
                    help="--form batch-once / batched: split_n,max_members of the gangs that share large problems "
                         "(batched default: the autotuner's choice; batch-once default: no split)")
    ap.add_argument("--read-s-steps", type=int, default=2,
                    help="plain form: steps of the S-reading row pass timed after the headline steps "
                         "(its own roofline entry; 0: skip)")
    ap.add_argument("--form-iters", type=int, default=0, help="iterations for a form run (0 = the workload's)")
    ap.add_argument("--read-s", action="store_true", help="plain form: the row pass reads S (no points mode)")
    ap.add_argument("--schedule", choices=["sequential", "mrhap"], default="sequential",
                    help="plain form: Algorithm 1's level-sequential schedule or the MapReduce one (Section 3)")
    ap.add_argument("--kappa", type=float, default=0.0,
                    help="plain and warm forms: weight of the optional level-wise similarity update (Eq. 2.7); "
                         "> 0 makes the row pass read S")
    ap.add_argument("--warm-levels", default="3,1", help="warm form: the level counts to train and evaluate")
    args = ap.parse_args()

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py runs on one GPU only: the library has no multi-GPU path "
              "(the row-block sharding is described in the design notes)", file=sys.stderr)
        return 2

    import numpy as np
    import torch

    from paper_1403_7394_amd import hap, metrics, synth

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        return 2
    hap.load()
    if args.form == "precision":
        print(json.dumps(run_precision_form(args, torch, hap, synth)), flush=True)
        return 0
    if args.form == "batched":
        print(json.dumps(run_batched_form(args, torch, hap, synth)), flush=True)
        return 0
    if args.form == "warm":
        print(json.dumps(run_warm_form(args, torch, hap, synth)), flush=True)
        return 0
    if args.form == "image":
        print(json.dumps(run_image_form(args, torch, hap, synth)), flush=True)
        return 0
    if args.form == "ceiling":
        print(json.dumps(run_ceiling_form(args, torch, hap)), flush=True)
        return 0
    if args.form in ("sweeps", "builds", "batch-once"):
        return run_profile_form(args, torch, hap, synth)
    dev = torch.device("cuda:0")
    blobs, rp = synth.workload_plain_f32()
    n = blobs.X.shape[0]
    L = rp.levels
    X = torch.from_numpy(blobs.X).to(dev)
    S = torch.empty((n, n), dtype=torch.float32, device=dev)
    ws = torch.empty(hap.workspace_size(n, L, hap.HAP_F32), dtype=torch.uint8, device=dev)

    if args.copy_probe:
        src = torch.ones(1 << 28, dtype=torch.float32, device=dev)   # 1 GiB
        dst = torch.empty_like(src)
        torch.mul(src, 1.0, out=dst)
        torch.cuda.synchronize()
        del src, dst

    points = not args.read_s and args.kappa == 0.0
    schedule = hap.SCHEDULE_MRHAP if args.schedule == "mrhap" else hap.SCHEDULE_SEQUENTIAL

    def step(profile: bool, use_points: bool):
        hap.build_similarity(X, S)
        h = hap.Hap(S, L, rp.damping, workspace=ws, schedule=schedule, kappa=args.kappa)
        if use_points:
            h.set_points(X)
        if profile:
            # event pairs around the launches of every PROF_EVERY-th sweep: enough launches for
            # a stable average without the events' own overhead on every launch
            h.profile(True, every=PROF_EVERY)
        res = h.iterate(rp.max_iters, rp.stable_iters)
        prof = h.profile_read() if profile else None
        counts = [h.exemplars(l)[1] for l in range(L)]
        ns = h.net_similarity(-1)
        launch = h.get_launch()
        fused = bool(h.launch_flags() & hap.LAUNCH_FUSED)
        labels = h.labels()
        h.close()
        return res, counts, ns, prof, launch + (fused,), labels

    def timed(steps: int, use_points: bool):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        acc = dict(sweeps=0, row_ms=0.0, row_n=0, col_ms=0.0, col_n=0, first=0)
        for _ in range(steps):
            res, counts, ns, prof, launch, labels = step(True, use_points)
            # an early stop is detected one sweep after the stop iteration; a stop at the cap is not
            acc["sweeps"] += res.iters + 1 if (res.converged and res.iters < rp.max_iters) else res.iters
            acc["first"] += 1
            acc["row_ms"] += prof[0]
            acc["row_n"] += prof[1]
            acc["col_ms"] += prof[2]
            acc["col_n"] += prof[3]
        torch.cuda.synchronize()
        acc["elapsed"] = time.perf_counter() - t0
        acc["last"] = (res, counts, ns, launch, labels)
        return acc

    def roofline(acc, use_points: bool) -> dict:
        w = 4
        # algorithmic bytes of all row-pass launches: read S, R, A and write R, A = 5 N^2 w, or
        # 4 N^2 w in the first sweep (no alpha to finish); one word less per element in points
        # mode, where S is not read.  The MapReduce schedule's fused pass runs every level in one
        # launch and reads S once: 1 + 4L words (1 + 3L in the first sweep) per launch.
        fused = acc["last"][3][4]
        lps = 1 if fused else L
        if fused:
            first_w, steady_w = 1 + 3 * L, 1 + 4 * L
        else:
            first_w, steady_w = (3, 4) if use_points else (4, 5)
        first_launches = acc["first"] * lps
        alg_total = (first_launches * first_w + (acc["row_n"] - first_launches) * steady_w) * n * n * w
        per_launch = alg_total / max(acc["row_n"], 1)
        avg_s = acc["row_ms"] / max(acc["row_n"], 1) * 1e-3
        achieved = per_launch / avg_s / 1e9
        # the counters were taken on the plain row pass; the Eq. 2.7 instance is another kernel
        traffic = (measured_traffic(use_points, first_launches, acc["row_n"] - first_launches)
                   if args.kappa == 0.0 and not fused else None)
        return {
            "bound": "hbm",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": traffic,
            "kernel": ("row pass (sweep_flow_kernel, points mode)" if use_points else
                       "row pass (sweep_kernel, S read, Eq. 2.7 row offsets)" if args.kappa else
                       f"fused row pass of all {L} levels (sweep_fused_kernel, S read once)" if fused else
                       "row pass (sweep_kernel, S read)"),
            "words_per_element": {"first_sweep": first_w, "later_sweeps": steady_w},
            "avg_launch_us": avg_s * 1e6,
            "alg_bytes_per_launch": per_launch,
            "launches_timed": acc["row_n"],
            "launches": int(acc["sweeps"] * lps),
            "timed_every": PROF_EVERY,
        }

    for _ in range(args.warmup):
        step(False, points)
    main = timed(args.steps, points)
    res, counts, ns, launch, labels = main["last"]
    elapsed = main["elapsed"]
    sweeps = main["sweeps"]
    ms_per_step = elapsed / args.steps * 1e3
    value = n * n * L * sweeps / elapsed

    lab = labels.cpu().numpy()
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": "plain HAP, 8192 points in 2-D, 64 Gaussian blobs, FP32, L=3, damping 0.9, "
                        "median preference, 500 iterations or 50 stable",
            "row_pass": "points mode (s_ij recomputed from the points)" if points else "reads S",
            "schedule": args.schedule,
            "kappa": args.kappa,
            "n": n, "levels": L, "damping": rp.damping, "max_iters": rp.max_iters,
            "stable_iters": rp.stable_iters, "seed": blobs.seed,
        },
        "roofline": roofline(main, points),
        "sweeps_per_step": sweeps / args.steps,
        "converged": bool(res.converged),
        # the run meets the stop rule only if it converged; otherwise the step ran to the cap
        "time_to_converge_ms": ms_per_step if res.converged else None,
        "time_to_cap_ms": None if res.converged else ms_per_step,
        # the timed sweeps' kernel time only (row passes and column sums, no host work)
        "sweep_updates_per_s": (n * n * main["row_n"] / ((main["row_ms"] + main["col_ms"]) * 1e-3)
                                if main["row_ms"] > 0 else None),
        "colsum_avg_us": main["col_ms"] / max(main["col_n"], 1) * 1e3,
        "exemplars_per_level": counts,
        "net_similarity": ns,
        "purity_per_level": [metrics.purity(x, blobs.truth) for x in lab],
        "launch": {"threads": launch[0], "chunks": launch[1], "rows_per_block": launch[2],
                   "streaming": launch[3], "fused_levels": launch[4]},
    }
    # how the step's labels compare with the stored oracle runs of the same workload (written by
    # tests/golden/full_run_plain8192.py from the oracle alone); the row-ordered launch
    # (one row per workgroup) equals the FP32 oracle run at every checkpoint, which the GPU tests
    # check; the default launch sums the column partials in blocks of rows
    if (args.schedule == "sequential" and args.kappa == 0.0 and not res.converged
            and res.iters == rp.max_iters):
        gold = {}
        for dt in ("float32", "float64"):
            try:
                with np.load(os.path.join(ROOT, "tests", "golden", f"full_run_plain8192_oracle_{dt}.npz")) as z:
                    gold[dt] = z["final_labels"]
            except (OSError, KeyError):
                pass
        out["oracle_label_agreement_at_cap"] = {dt: [float(np.mean(lab[l] == g[l])) for l in range(L)]
                                                for dt, g in gold.items()}
    if points and args.read_s_steps > 0:
        # the pass the workload's configuration names (dense S read every sweep), timed the same way
        rs = timed(args.read_s_steps, False)
        out["roofline_read_s"] = roofline(rs, False)
        out["read_s"] = {"steps": args.read_s_steps, "ms_per_step": rs["elapsed"] / args.read_s_steps * 1e3,
                         "value": n * n * L * rs["sweeps"] / rs["elapsed"],
                         "labels_equal_points_mode": bool(torch.equal(rs["last"][4], labels))}
    if args.schedule == "sequential" and args.kappa == 0.0 and not args.no_converge_variants:
        # Under the literal Eq. 2.6 the L = 3 run never meets the stop rule, so its time to
        # converge does not exist; the same workload does converge at L = 1 (plain affinity
        # propagation) and with the optional Eq. 2.7 update (kappa = 0.5).  Each is timed once
        # from X on the device to labels (build, median, sweeps to the stop rule, labels).
        variants = {}
        for name, lv, kap in (("L1", 1, 0.0), ("kappa0.5", L, 0.5)):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hap.build_similarity(X, S)
            h = hap.Hap(S, lv, rp.damping, workspace=ws, kappa=kap)
            if kap == 0.0:
                h.set_points(X)
            r = h.iterate(rp.max_iters, rp.stable_iters)
            h.labels()
            torch.cuda.synchronize()
            ms = (time.perf_counter() - t0) * 1e3
            variants[name] = {"levels": lv, "kappa": kap, "iters": r.iters, "converged": bool(r.converged),
                              "time_to_converge_ms": ms if r.converged else None,
                              "exemplars_per_level": [h.exemplars(l)[1] for l in range(lv)]}
            h.close()
        out["converging_variants"] = variants
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(blobs.X, rp, args.cpu_sweeps)
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
