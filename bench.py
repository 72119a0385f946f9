#!/usr/bin/env python3
"""Throughput of LANTERN's relaxed verification on one MI355X.

A step is one lantern_verify call over one batch of synthetic rows of the
stress workload (V=16384 codebook, k=1000 neighbours, delta=0.4, 3840 draft
candidates per step, bf16 logits, neighbour table resident in HBM).  Inputs
are generated on the device before the timed region; several distinct step
buffers are rotated so that reads come from HBM rather than from the 256 MB
last-level cache.  Prints one JSON line.

The headline (`value`, `roofline`) is the plain mix of the configuration, in
which nearly every row is accepted.  The same line carries, under `variants`,
the reject-heavy and the bound-binding mixes through the same entry point and
through the decisions-only and tree entry points, and under `knn` the
neighbour-table build of the stress and the wide-latent codebooks.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--variant plain|reject|peaked] [--mode ...]
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

METRIC = "relaxed verifications/sec at V=16384,k=1000 (bf16 logits); % HBM peak"
HBM_PEAK_GBS = 8000.0
MFMA_PEAK_TFLOPS = {"bf16": 2500.0, "f32": 157.3}
# HBM bytes per launch from the rocprofv3 FETCH_SIZE / WRITE_SIZE runs summarised under profiles/
# (FETCH_SIZE scaled by the factor a plain 256 MiB copy gives in the same run).  Counters cannot be
# read from inside this process, so the figure is a record of that run: it is reported only while the
# library still has the version it was measured at, and with the file it comes from.
_FETCH_SCALE = 262144.0 / 131096.2   # what FETCH_SIZE read for a 256 MiB copy in the same run
MEASURED_TRAFFIC = {
    # (workload, variant, mode): (bytes per launch, library version, source)
    ("stress", "plain", "sample"): ((130993.5 * _FETCH_SCALE + 240.2) * 1024, 241,
                                    "profiles/verify_fast_stress_plain.md (FETCH_SIZE, WRITE_SIZE; version 241)"),
    ("stress", "reject", "sample"): ((165291.7 * _FETCH_SCALE + 285.7) * 1024, 241,
                                     "profiles/verify_fast_stress_plain.md (reject mix; version 241)"),
    ("wide_latent", "plain", "sample"): ((124432.1 * _FETCH_SCALE + 240.6) * 1024, 241,
                                         "profiles/verify_fast_stress_plain.md (wide_latent; version 241)"),
    ("stress", "plain", "greedy"): ((69189.1 * _FETCH_SCALE + 240.0) * 1024, 241,
                                    "profiles/greedy_fast_stress_plain.md (version 241)"),
}


# Per-kernel split of a table build, from the kernel trace summarised under profiles/ (events inside this
# process only bracket the whole build): us per build, reported under the same rule, and only if the parts do
# not add up to more than the build took.  The stress table takes the path with sampled thresholds and a
# filtering contraction, and so does the wide-latent table.  The thresholds' kernel contracts the rows with a sample of
# 2048 and 1024 tokens itself; its product is not counted among the contractions.
MEASURED_KNN_SPLIT = {
    # workload: ({kernel: us per build}, extra contraction flop, library version, source)
    "stress": ({"thresholds": 34.8, "filter_contraction": 105.2, "selection": 171.7, "exact_check": 4.1,
                "operands_and_norms": 8.3}, 0.0, 241,
               "profiles/knn_build_stress_and_wide_latent.md (kernel trace; version 241)"),
    "wide_latent": ({"thresholds": 22.0, "filter_contraction": 71.7, "selection": 72.8, "exact_check": 4.1,
                     "operands_and_norms": 11.7}, 0.0, 241,
                    "profiles/knn_build_stress_and_wide_latent.md (kernel trace; version 241)"),
}


def algorithmic_bytes_per_verification(V: int, k: int, logit_bytes: int) -> int:
    """Both logit rows once, one table row, token, two uniforms, two outputs."""
    return 2 * V * logit_bytes + 4 * k + 20


class Runner:
    """Inputs of one (workload, variant, mode) resident on the device, and the call that is one step."""

    def __init__(self, lantern, lib, cfg, knn, variant, mode, divergence, tree_order, nbuf, dev, stream):
        import torch
        from synth import workloads
        self.cfg, self.mode, self.variant = cfg, mode, variant
        self.delta = 0.0 if variant == "reject" else cfg.delta
        self.nbuf = nbuf
        self.rows = cfg.rows
        dcode = lantern.BF16 if cfg.logit_dtype == "bf16" else lantern.F32
        delta = float(self.delta)
        div = 1 if divergence == "jsd" else 0
        self.out_acc = [torch.empty(cfg.rows, dtype=torch.int32, device=dev) for _ in range(nbuf)]
        self.out_res = [torch.empty(cfg.rows, dtype=torch.int32, device=dev) for _ in range(nbuf)]
        out_acc, out_res = self.out_acc, self.out_res
        self.tree_info = {}
        if mode in ("tree", "tree_seq"):
            import numpy as np
            from synth import trees
            M = 60
            B = cfg.rows // M
            self.rows = B * M
            parent_host = trees.random_trees(np.random.default_rng(workloads.BASE_SEED), B, M)
            if tree_order == "level":
                parent_host = trees.level_order(parent_host)
            parent = torch.from_numpy(parent_host).to(dev).reshape(-1)
            tb = []
            for s_ in range(nbuf):
                st_, ri, tok, un = trees.tree_step(cfg, parent_host, step=s_, variant=variant, device=dev)
                tb.append((st_, torch.from_numpy(ri).to(dev), torch.from_numpy(tok).to(dev), un))
            self.distinct_rows = len(set(tb[0][1].cpu().tolist()))
            t_len = torch.empty(B, dtype=torch.int32, device=dev)
            t_path = torch.empty(B * M, dtype=torch.int32, device=dev)
            t_next = torch.empty(B, dtype=torch.int32, device=dev)
            self.t_len = t_len
            self.tree_info = {"trees": B, "candidates_per_tree": M, "tree_order": tree_order,
                              "distinct_logit_rows": self.distinct_rows}
            self.probe_src = [(t_[0].target_logits, t_[0].draft_logits) for t_ in tb]
            self.keep = (tb, parent)

            if mode == "tree_seq":
                need = int(lib.lantern_verify_trees_sequential_workspace_bytes(B, M, cfg.V))
                work = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
                self.keep = (tb, parent, work)

                def step_seq(i):
                    st_, ri, tok, un = tb[i % nbuf]
                    rc = lib.lantern_verify_trees_sequential(
                        st_.target_logits.data_ptr(), st_.draft_logits.data_ptr(), dcode, B * (M + 1), cfg.V, cfg.V,
                        ri.data_ptr(), parent.data_ptr(), B, M, tok.data_ptr(), knn.data_ptr(), cfg.k, div, delta,
                        un.data_ptr(), t_len.data_ptr(), t_path.data_ptr(), t_next.data_ptr(), work.data_ptr(),
                        work.numel(), stream.cuda_stream)
                    assert rc == 0, rc
                self.step = step_seq
                return

            def step(i):
                st_, ri, tok, un = tb[i % nbuf]
                rc = lib.lantern_verify_trees(st_.target_logits.data_ptr(), st_.draft_logits.data_ptr(), dcode,
                                              B * (M + 1), cfg.V, cfg.V, ri.data_ptr(), parent.data_ptr(), B, M,
                                              tok.data_ptr(), knn.data_ptr(), cfg.k, div, delta, un.data_ptr(),
                                              out_acc[i % nbuf].data_ptr(), t_len.data_ptr(), t_path.data_ptr(),
                                              t_next.data_ptr(), stream.cuda_stream)
                assert rc == 0, rc
            self.step = step
            return
        bufs = [workloads.make_step(cfg, step=s, device=dev, variant=variant) for s in range(nbuf)]
        self.bufs = bufs
        self.probe_src = [(b.target_logits, None if mode == "greedy" else b.draft_logits) for b in bufs]

        if mode == "greedy":
            def step(i):
                b = bufs[i % nbuf]
                rc = lib.lantern_verify_greedy(b.target_logits.data_ptr(), dcode, cfg.rows, cfg.V, cfg.V,
                                               b.draft_tokens.data_ptr(), knn.data_ptr(), cfg.k, delta,
                                               out_acc[i % nbuf].data_ptr(), out_res[i % nbuf].data_ptr(), None,
                                               stream.cuda_stream)
                assert rc == 0, rc
        elif mode == "decide":
            def step(i):
                b = bufs[i % nbuf]
                rc = lib.lantern_decide_rows(b.target_logits.data_ptr(), b.draft_logits.data_ptr(), dcode, cfg.rows,
                                             cfg.V, cfg.V, None, cfg.rows, b.draft_tokens.data_ptr(), knn.data_ptr(),
                                             cfg.k, div, delta, b.uniforms.data_ptr(), out_acc[i % nbuf].data_ptr(),
                                             None, stream.cuda_stream)
                assert rc == 0, rc
        elif div:
            def step(i):
                b = bufs[i % nbuf]
                rc = lib.lantern_verify_divergence(b.target_logits.data_ptr(), b.draft_logits.data_ptr(), dcode,
                                                   cfg.rows, cfg.V, cfg.V, b.draft_tokens.data_ptr(), knn.data_ptr(),
                                                   cfg.k, 1, delta, b.uniforms.data_ptr(),
                                                   out_acc[i % nbuf].data_ptr(), out_res[i % nbuf].data_ptr(),
                                                   None, None, None, None, None, stream.cuda_stream)
                assert rc == 0, rc
        else:
            def step(i):
                b = bufs[i % nbuf]
                lantern.verify(b.target_logits, b.draft_logits, b.draft_tokens, knn, delta, b.uniforms,
                               out_accept=out_acc[i % nbuf], out_resample=out_res[i % nbuf], stream=stream)
        self.step = step

    def algorithmic_bytes(self) -> int:
        cfg = self.cfg
        lb = 2 if cfg.logit_dtype == "bf16" else 4
        if self.mode in ("tree", "tree_seq"):   # every distinct pair of logit rows once; per verification the table row and the small items
            return 2 * cfg.V * lb * self.distinct_rows + (4 * cfg.k + 24) * self.rows
        if self.mode == "greedy":  # one logit row, the table row, token, two outputs
            return (cfg.V * lb + 4 * cfg.k + 12) * self.rows
        return algorithmic_bytes_per_verification(cfg.V, cfg.k, lb) * self.rows

    def accepted_fraction(self, steps: int) -> float:
        import torch
        if self.mode == "tree_seq":   # no per-candidate decisions: the accepted nodes over all candidates
            return float(self.t_len.float().sum().item()) / self.rows
        acc_all = torch.stack(self.out_acc[: min(self.nbuf, steps)])[:, : self.rows]
        return float((acc_all == 1).float().mean().item())


def timed(runner, steps, warmup, stream):
    """W untimed steps, then K steps between one pair of HIP events on the launch stream.
    Returns (wall seconds, average launch duration in ms: includes the gaps between launches)."""
    import torch
    for i in range(warmup):
        runner.step(i)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    ev0.record(stream)
    for i in range(steps):
        runner.step(i)
    ev1.record(stream)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    return t1 - t0, ev0.elapsed_time(ev1) / steps


def time_knn_build(lantern, codebook, k, repeats=3):
    """Median of a few builds between HIP events (the first call, untimed, loads the kernels); workspace
    and table are allocated once, outside the timed calls."""
    import torch
    V, d = codebook.shape
    code = lantern.BF16 if codebook.dtype == torch.bfloat16 else lantern.F32
    ws = torch.empty(lantern.binding.knn_workspace_bytes(code, V, d, k), dtype=torch.uint8, device=codebook.device)
    knn = torch.empty((V, k), dtype=torch.int32, device=codebook.device)
    lantern.build_knn(codebook, k, workspace=ws, out=knn)
    torch.cuda.synchronize()
    ms = []
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        lantern.build_knn(codebook, k, workspace=ws, out=knn)
        e1.record()
        torch.cuda.synchronize()
        ms.append(e0.elapsed_time(e1))
    ms.sort()
    return knn, ms[len(ms) // 2]


def time_random_table(lantern, V, k, seed=2410, repeats=3):
    """Median of a few builds of the random-selection table (Section 5.3.1) between HIP events, after one
    untimed call; the table is what the call must write (4 V k bytes), the pair keys are generated on the fly."""
    import torch
    lantern.build_random(V, k, seed)
    torch.cuda.synchronize()
    ms = []
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        out = lantern.build_random(V, k, seed)
        e1.record()
        torch.cuda.synchronize()
        ms.append(e0.elapsed_time(e1))
        del out
    ms.sort()
    mid = ms[len(ms) // 2]
    return {"table": f"V={V} k={k}", "build_ms": mid, "algorithmic_bytes": 4 * V * k,
            "hbm_frac": 4.0 * V * k / (mid * 1e-3) / 1e9 / HBM_PEAK_GBS,
            "note": "timed with the table's allocation inside the call (a cached block after the first build)"}


def knn_report(cfg, build_ms, version=None):
    """The build against the MFMA roofline of its contraction (2 V^2 d flop in the codebook's type) and
    against the HBM roofline of what it must move (codebook in, table out)."""
    flop = 2.0 * cfg.V * cfg.V * cfg.d
    peak = MFMA_PEAK_TFLOPS[cfg.cb_dtype]
    io_bytes = cfg.V * cfg.d * (2 if cfg.cb_dtype == "bf16" else 4) + 4 * cfg.V * cfg.k
    rep = {"codebook": f"V={cfg.V} d={cfg.d} {cfg.cb_dtype} k={cfg.k}", "build_ms": build_ms,
           "contraction_flop": flop, "mfma_peak_tflops": peak,
           "mfma_frac": flop / (build_ms * 1e-3) / 1e12 / peak,
           "algorithmic_bytes": io_bytes, "hbm_frac": io_bytes / (build_ms * 1e-3) / 1e9 / HBM_PEAK_GBS}
    split = MEASURED_KNN_SPLIT.get(cfg.name)
    if split is not None and version == split[2]:
        us = split[0]
        if sum(us.values()) * 1e-3 > build_ms:
            rep["split_note"] = "not reported: the recorded kernels add up to more than this build took"
            return rep
        rep["contraction_ms"] = sum(v for n, v in us.items() if n.endswith("contraction")) * 1e-3
        if "thresholds" in us:
            rep["threshold_ms"] = us["thresholds"] * 1e-3
        rep["select_ms"] = us["selection"] * 1e-3
        rep["exact_check_ms"] = us["exact_check"] * 1e-3
        # the contractions alone against the matrix-core peak of their type
        rep["contraction_mfma_frac"] = (flop + split[1]) / (rep["contraction_ms"] * 1e-3) / 1e12 / peak
        rep["split_source"] = split[3]
    return rep


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=576)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="stress", choices=["stress", "image_batch", "wide_latent", "llamagen_step", "tiny"],
                    help="stress is the headline; llamagen_step (one tree's 60 candidates per call) and tiny are "
                         "in the launch-latency regime: read ms_per_step")
    ap.add_argument("--variant", default="plain", choices=["plain", "reject", "peaked"])
    ap.add_argument("--mode", default="sample", choices=["sample", "greedy", "tree", "tree_seq", "decide"],
                    help="sample: lantern_verify (the headline); greedy: lantern_verify_greedy, target rows only; "
                         "decide: lantern_decide_rows, the decisions without resampled tokens (rejections settle in "
                         "the fp32 pass too); tree: rows_per_step/60 random draft trees of 60 candidates, siblings sharing logit rows "
                         "(lantern_verify_trees: decisions, walk, one residual draw per tree); tree_seq: the same trees "
                         "under the sequential-residual sibling rule (lantern_verify_trees_sequential)")
    ap.add_argument("--divergence", default="tvd", choices=["tvd", "jsd"],
                    help="bound on the neighbourhood: total variation (the headline) or Jensen-Shannon")
    ap.add_argument("--tree-order", default="level", choices=["level", "random"],
                    help="tree mode: candidates listed level by level with siblings next to each other (as a "
                         "drafter that expands one level at a time lists them), or in random drafting order")
    ap.add_argument("--buffers", type=int, default=6, help="distinct step inputs rotated through")
    ap.add_argument("--rows", type=int, default=None,
                    help="verifications per step, when not the workload's own (a sweep aid: the headline uses the default)")
    ap.add_argument("--cpu-seconds", type=float, default=10.0,
                    help="the CPU oracle is timed on whole steps of the workload until this much time has passed")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true",
                    help="leave out the other mixes, entry points and the wide-latent table build that the default "
                         "run reports beside the headline")
    ap.add_argument("--extra-steps", type=int, default=60, help="timed steps of each extra mix / entry point")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run one plain 256 MiB device copy, so that a counter run has a kernel of "
                         "known traffic to scale FETCH_SIZE / WRITE_SIZE by")
    ap.add_argument("--traffic-bytes", type=float, default=None,
                    help="HBM bytes per launch from rocprofv3 counters, if known")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (verifications are independent, so more GPUs "
              "would each take a share of the rows with the table replicated); run with --gpus 1",
              file=sys.stderr)
        return 2

    import torch
    import paper_2410_03355_amd as lantern
    from synth import workloads

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the library has no CPU fallback", file=sys.stderr)
        return 2
    lib = lantern.load()
    dev = "cuda:0"
    torch.cuda.set_device(0)
    cfg = workloads.CONFIGS[args.workload]
    if args.rows is not None:
        cfg = workloads.with_overrides(cfg, rows=args.rows)
    stream = torch.cuda.current_stream()
    headline = (args.workload == "stress" and args.variant == "plain" and args.mode == "sample"
                and args.divergence == "tvd" and args.rows is None)
    extras = headline and not args.no_extras

    # ---- neighbour table: built once on the device, stays resident ----
    codebook = workloads.make_codebook(cfg, device=dev)
    knn, knn_build_ms = time_knn_build(lantern, codebook, cfg.k)

    # ---- step inputs, resident in HBM before the timed region ----
    nbuf = max(1, args.buffers)
    run = Runner(lantern, lib, cfg, knn, args.variant, args.mode, args.divergence, args.tree_order, nbuf, dev, stream)
    torch.cuda.synchronize()
    greedy, tree = args.mode == "greedy", args.mode in ("tree", "tree_seq")

    for i in range(args.warmup):
        run.step(i)
    torch.cuda.synchronize()
    if args.copy_calibration:
        src = torch.empty(256 << 20, dtype=torch.uint8, device=dev).random_(0, 255)
        dst = torch.empty_like(src)
        dst.copy_(src)  # reads 256 MiB, writes 256 MiB
        torch.cuda.synchronize()
        del src, dst

    # one pair of HIP events on the launch stream brackets the K launches of the timed region
    wall, kernel_ms_avg = timed(run, args.steps, 0, stream)

    # the device's read rate for a plain stream of the same shape (same buffers, same rotation)
    sink = torch.zeros(1, dtype=torch.int32, device=dev)
    probe_src = run.probe_src
    probe_bytes = probe_src[0][0].numel() * probe_src[0][0].element_size() // 65536 * 65536
    probe_total = probe_bytes * (1 if greedy else 2)
    stream_read_gbs = None
    if probe_bytes > 0:
        for i in range(4):
            pa, pb = probe_src[i % nbuf]
            lib.lantern_probe_stream_read(pa.data_ptr(), None if pb is None else pb.data_ptr(), probe_bytes,
                                          sink.data_ptr(), stream.cuda_stream)
        pv0, pv1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        pv0.record(stream)
        n_probe = 100
        for i in range(n_probe):
            pa, pb = probe_src[i % nbuf]
            lib.lantern_probe_stream_read(pa.data_ptr(), None if pb is None else pb.data_ptr(), probe_bytes,
                                          sink.data_ptr(), stream.cuda_stream)
        pv1.record(stream)
        torch.cuda.synchronize()
        stream_read_gbs = probe_total * n_probe / (pv0.elapsed_time(pv1) * 1e-3) / 1e9

    rows = run.rows
    bytes_per_launch = run.algorithmic_bytes()
    achieved_gbs = bytes_per_launch / (kernel_ms_avg * 1e-3) / 1e9
    value = rows * args.steps / wall
    accept_frac = run.accepted_fraction(args.steps)

    traffic, traffic_note = args.traffic_bytes, None
    if traffic is None and args.divergence == "tvd" and args.rows is None:
        rec = MEASURED_TRAFFIC.get((args.workload, args.variant, args.mode))
        if rec is not None:
            if rec[1] == int(lib.lantern_version()):
                traffic, traffic_note = rec[0], rec[2]
            else:
                traffic_note = f"not reported: measured at library version {rec[1]}, this is {int(lib.lantern_version())}"

    result = {
        "metric": METRIC,
        "value": value,
        "unit": "verifications/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "logits_dtype": cfg.logit_dtype,
        "arithmetic": "fp32 pass with proven margins; rows it cannot settle, and every resampled token, in fp64",
        "data": "synthetic",
        "config": {
            "workload": f"{cfg.name}/{args.variant}/{args.mode}/{args.divergence}: V={cfg.V} d={cfg.d} k={cfg.k} delta={run.delta} "
                        f"rows_per_step={rows} logits={cfg.logit_dtype}",
            "rows_per_step": rows,
            "distinct_step_buffers": nbuf,
            "accepted_fraction": accept_frac,
            **({**run.tree_info, "mean_accepted_length": float(run.t_len.float().mean().item())} if tree else {}),
        },
        "roofline": {
            "bound": "hbm",
            "kernel": "greedy_fast" if greedy else ("trees_sequential" if args.mode == "tree_seq" else "verify_fast"),
            **({"note": "per step: verify_fast over shared rows, the tree walk, one fp64 residual draw per tree"}
               if args.mode == "tree" else {}),
            **({"note": "one workgroup per tree walks it in fp64, sibling after sibling: latency bound, 64 of 256 "
                        "compute units busy"} if args.mode == "tree_seq" else {}),
            "achieved": achieved_gbs,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved_gbs / HBM_PEAK_GBS,
            "traffic": traffic,
            **({"traffic_source": traffic_note} if traffic_note else {}),
            "algorithmic_bytes_per_launch": bytes_per_launch,
            "kernel_ms_avg": kernel_ms_avg,
            "stream_read_gbs": stream_read_gbs,
            "stream_read_note": f"plain read of {probe_total >> 20} MiB per launch from the same rotating buffers, one "
                                "workgroup per 64 KiB: what a kernel with this access pattern reaches on this device",
        },
        "knn_build_ms": knn_build_ms,
        "knn": {cfg.name: knn_report(cfg, knn_build_ms, int(lib.lantern_version()))},
    }

    if extras:
        # ---- the other mixes and entry points on the same configuration (the headline's mix accepts
        # nearly every row; the paper's acceptance rates are far lower, and rejections cost time) ----
        variants = {}
        for variant, modes in (("reject", ("sample", "decide", "tree", "tree_seq")),
                               ("peaked", ("sample", "decide", "tree", "tree_seq"))):
            variants[variant] = {}
            for mode in modes:
                r = Runner(lantern, lib, cfg, knn, variant, mode, "tvd", args.tree_order, min(nbuf, 4), dev, stream)
                torch.cuda.synchronize()
                w, kms = timed(r, args.extra_steps, 5, stream)
                b = r.algorithmic_bytes()
                variants[variant][mode] = {
                    "entry_point": {"sample": "lantern_verify", "decide": "lantern_decide_rows",
                                    "tree": "lantern_verify_trees",
                                    "tree_seq": "lantern_verify_trees_sequential"}[mode],
                    "delta": r.delta, "rows_per_step": r.rows, "steps": args.extra_steps,
                    "ms_per_step": w / args.extra_steps * 1e3, "kernel_ms_avg": kms,
                    "value": r.rows * args.extra_steps / w,
                    "accepted_fraction": r.accepted_fraction(args.extra_steps),
                    "frac": b / (kms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                    **({"mean_accepted_length": float(r.t_len.float().mean().item())} if mode in ("tree", "tree_seq") else {}),
                }
                del r
                torch.cuda.empty_cache()
        result["variants"] = variants
        result["variants_note"] = ("same configuration and table; reject: delta=0 and acceptance draws just below one "
                                   "(about 60 % of the rows rejected); peaked: logits x5 (about 45 % rejected, the bound "
                                   "cuts the neighbourhoods); sample resamples every rejected row in fp64, decide "
                                   "returns decisions only, tree walks 64 trees of 60 candidates and resamples one "
                                   "token per tree, tree_seq walks the same trees under the sequential-residual "
                                   "sibling rule (its accepted_fraction is accepted nodes / candidates); frac = algorithmic bytes / kernel time / 8 TB/s")
        wl = workloads.CONFIGS["wide_latent"]
        _, wl_ms = time_knn_build(lantern, workloads.make_codebook(wl, device=dev), wl.k)
        result["knn"][wl.name] = knn_report(wl, wl_ms, int(lib.lantern_version()))
        result["random_table"] = time_random_table(lantern, cfg.V, cfg.k)

    if not args.no_cpu_baseline and args.mode == "sample" and args.divergence == "tvd":
        import numpy as np  # noqa: F401
        import oracle  # CPU baseline leg only
        threads = min(os.cpu_count() or 1, 16, oracle.max_threads())
        knn_host = knn.cpu().numpy()
        bufs = run.bufs
        out_acc, out_res, delta = run.out_acc, run.out_res, run.delta
        host = [(b.target_logits.float().cpu().numpy(), b.draft_logits.float().cpu().numpy(),
                 b.draft_tokens.cpu().numpy(), b.uniforms.cpu().numpy()) for b in bufs]
        # untimed: the GPU's outputs of the timed region against the oracle, buffer by buffer
        mism = 0
        for i, (tl, dl, tok, un) in enumerate(host[: min(nbuf, args.steps, 2)]):
            acc, res, _ = oracle.verify(tl, dl, tok, knn_host, cfg.k, delta, un, threads=threads,
                                        want_diag=False)
            mism += int((acc != out_acc[i].cpu().numpy()).sum() + (res != out_res[i].cpu().numpy()).sum())
        # timed: the oracle alone, whole steps of the same workload until the time is up
        n_cpu = 0
        c0 = time.perf_counter()
        while True:
            tl, dl, tok, un = host[n_cpu % nbuf]
            oracle.verify(tl, dl, tok, knn_host, cfg.k, delta, un, threads=threads, want_diag=False)
            n_cpu += 1
            c1 = time.perf_counter()
            if c1 - c0 >= args.cpu_seconds:
                break
        # one thread, one step; and the table build of a sample of query rows on all threads
        s0 = time.perf_counter()
        tl, dl, tok, un = host[0]
        n_single = min(rows, 512)
        oracle.verify(tl[:n_single], dl[:n_single], tok[:n_single], knn_host, cfg.k, delta, un[:n_single], threads=1,
                      want_diag=False)
        s1 = time.perf_counter()
        cb_host = codebook.float().cpu().numpy()
        n_knn = min(cfg.V, 256)
        k0 = time.perf_counter()
        oracle.build_knn(cb_host, cfg.k, rows=(0, n_knn), threads=threads)
        k1 = time.perf_counter()
        result["cpu_baseline"] = {
            "single_thread_value": n_single / (s1 - s0),
            "knn_build_ms_extrapolated": (k1 - k0) / n_knn * cfg.V * 1e3,
            "knn_sample": f"{n_knn} of {cfg.V} query rows on {threads} threads, scaled to the whole table",
            "value": n_cpu * rows / (c1 - c0),
            "unit": "verifications/s",
            "cores": threads,
            "kind": "oracle",
            "sample": f"{n_cpu} step(s) of {rows} rows of the same workload ({c1 - c0:.1f} s), rows split over "
                      f"{threads} threads",
            "mismatches_vs_gpu": mism,
        }

    print(json.dumps(result))
    return 0


if __name__ == "__main__":
    sys.exit(main())
