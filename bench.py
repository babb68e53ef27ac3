#!/usr/bin/env python3
"""Throughput of the token-adapted encoder on one MI355X.

A step = one pass of the whole hot path over one synthetic batch: otas_prompt_prepend followed by
otas_encoder_forward (LayerNorm, QKV GEMM, attention, projection, merge metric / plan / apply,
LayerNorm, MLP GEMMs, for every layer).  Inputs and weights are resident in HBM before the timed
region.  Prints ONE JSON line: images/s of the headline workload, per-strategy images/s, the
roofline figures of the dominant kernel (the bf16 MFMA GEMM) and of the other kernels, measured
with HIP events through the library's per-launch timing, and the CPU oracle timed on a bounded
sample of the same workload.
"""
from __future__ import annotations

import argparse
import gc
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import otas_synth as synth  # noqa: E402

PEAK_BF16_TFLOPS = 2500.0      # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0          # MI355X HBM3E
RATED_MHZ = 2400.0             # the clock the data-sheet peaks are quoted at
BASELINE_METRIC = "images/sec per (prompts, r) strategy, ViT-B/16 batch 64 bf16; merge-kernel HBM GB/s"


READ_AHEAD_ROWS = 4096     # kWarmRows of the library


def algorithmic_work(cfg, lengths0, r, otas, ctx):
    """Per-kind algorithmic FLOPs / bytes of ONE forward, from the host-known length schedule and the
    library's own split-K decision (which decides whether a block's first LayerNorm is a launch of its
    own or part of the previous block's split-K reduce)."""
    D, H, F, L = cfg.D, cfg.H, cfg.F, cfg.L
    e = 4 if cfg.dtype == "f32" else 2
    if cfg.deep:   # per-layer prompting: no merging; lengths constant (replace) or + P per layer (grow)
        P = np.array([p for p, _ in cfg.strategies])
        grow = cfg.deep == "grow"
        ent = [np.asarray(lengths0) + (l * P if grow else 0) for l in range(L)]
        sched = np.stack(ent + [ent[-1]], axis=1)
    else:
        sched = np.array([otas.otas_schedule(int(n), 0, int(rr), cfg.n_lead, L) for n, rr in zip(lengths0, r)])  # [B, L+1]
    T = sched.sum(axis=0)                       # rows entering layer l (l = 0..L-1), then the output rows
    Tm = T[:L] if cfg.deep else T[1:]           # rows of layer l behind its merging module (MLP rows)
    w = {"gemm_qkv": 0.0, "gemm_proj": 0.0, "gemm_fc1": 0.0, "gemm_fc2": 0.0, "attention": 0.0,
         "merge_apply_bytes": 0.0, "layer_norm_bytes": 0.0, "splitk_reduce_bytes": 0.0,
         "merge_apply_bytes_per_layer": [], "splits": [],
         # the same three passes priced as if the residual stream were stored in the model's dtype (what the
         # method itself needs: token rows in and out, the metric rows, sizes in and out)
         "merge_apply_method_bytes": 0.0, "merge_apply_method_bytes_per_layer": [],
         "layer_norm_method_bytes": 0.0, "splitk_reduce_method_bytes": 0.0}
    # bf16 launches of up to READ_AHEAD_ROWS rows also read the next linear's weight
    ahead = lambda rows, n_out: n_out * D * e if e == 2 and rows <= READ_AHEAD_ROWS else 0
    ln1_fused = False
    for l in range(L):
        w["gemm_qkv"] += 2.0 * T[l] * D * 3 * D
        w["gemm_proj"] += 2.0 * T[l] * D * D
        w["gemm_fc1"] += 2.0 * Tm[l] * D * F
        w["gemm_fc2"] += 2.0 * Tm[l] * D * F
        w["attention"] += float(np.sum(4.0 * sched[:, l].astype(np.float64) ** 2 * D))
        if not ln1_fused:
            w["layer_norm_bytes"] += T[l] * D * (4.0 + e)            # LN1: float residual row in, operand row out
            w["layer_norm_method_bytes"] += T[l] * D * 2.0 * e
        if Tm[l] != T[l]:
            # merge-apply fused with LN2: float rows in and out, a size and a list entry per row, operand row out
            b = (T[l] + Tm[l]) * (D * 4.0 + 8.0) + Tm[l] * D * e + ahead(Tm[l], F)
            w["merge_apply_bytes"] += b
            w["merge_apply_bytes_per_layer"].append(b)
            bm = (T[l] + Tm[l]) * D * e + T[l] * (D // H) * e + 4.0 * (T[l] + Tm[l])
            w["merge_apply_method_bytes"] += bm
            w["merge_apply_method_bytes_per_layer"].append(bm)
        else:
            w["layer_norm_bytes"] += Tm[l] * D * (4.0 + e)           # LN2 on its own
            w["layer_norm_method_bytes"] += Tm[l] * D * 2.0 * e
        S = ctx.otas_splitk_factor(int(Tm[l]), D, F, ctx.otas_splitk_room(int(T[0]), int(Tm[l]))) if e == 2 and not cfg.deep else 1
        w["splits"].append(S)
        ln1_fused = S > 1 and l + 1 < L
        if S > 1:   # S float partial rows + residual row in, residual row out, next block's operand row out
            w["splitk_reduce_bytes"] += Tm[l] * D * (4.0 * (S + 2) + (e if l + 1 < L else 0))
            w["splitk_reduce_bytes"] += ahead(Tm[l], 3 * D) if l + 1 < L else 0
            w["splitk_reduce_method_bytes"] += Tm[l] * D * (e * 2 + (e if l + 1 < L else 0))   # residual in/out, operand out
    w["T"] = T.tolist()
    w["Tm"] = [int(v) for v in Tm]
    return w


class Strategy:
    """One workload resident on the GPU: context, inputs, workspace, outputs."""

    def __init__(self, name, batch=0):
        import torch
        import paper_2401_05031_amd as otas
        self.name = name
        self.cfg = cfg = synth.config(name)
        if batch and batch < cfg.B:      # the first `batch` queries of the workload: what a serving loop sends at low rates
            cfg.B = batch
            cfg.strategies = cfg.strategies[:batch]
        self.ctx = otas.Context.from_host_weights(cfg.L, cfg.D, cfg.H, cfg.F,
                                                  otas.OTAS_F32 if cfg.dtype == "f32" else otas.OTAS_BF16,
                                                  cfg.ln_eps, cfg.n_lead, synth.all_weights(cfg))
        ctx = self.ctx
        toks, prm, P, self.R = synth.batch(cfg)
        D = cfg.D
        tok_packed, self.tok_off = synth.pack(toks, D)
        prm_packed, self.prm_off = synth.pack(prm, D)
        self.t_tok = torch.from_numpy(tok_packed).to("cuda").to(ctx.torch_dtype)
        self.t_prm = torch.from_numpy(prm_packed).to("cuda").to(ctx.torch_dtype) if prm_packed.shape[0] else None
        T0 = int(self.tok_off[-1] + self.prm_off[-1])
        self.x0 = torch.empty((T0, D), dtype=ctx.torch_dtype, device="cuda")
        self.lengths0 = np.diff(self.tok_off) + np.diff(self.prm_off)
        reff, _ = ctx.trace_layout(self.lengths0, self.R)
        T_out = int(T0 - reff.sum())
        self.deep = None
        if cfg.deep:   # per-layer prompting: prompts [L, sum P, D]; block 0 (layer 0) is what prepend inserts
            assert all(r == 0 for r in self.R)
            blocks = [prm_packed] + [synth.pack([synth.query_layer_prompts(cfg, q, l) for q in range(cfg.B)], D)[0]
                                     for l in range(1, cfg.L)]
            self.deep = torch.from_numpy(np.stack(blocks, axis=0)).to("cuda").to(ctx.torch_dtype).contiguous()
            self.deep_mode = otas.OTAS_PROMPT_GROW if cfg.deep == "grow" else otas.OTAS_PROMPT_REPLACE
            T_out = T0 + (cfg.L - 1) * int(self.prm_off[-1]) if cfg.deep == "grow" else T0
        self.ws = torch.empty(ctx.otas_workspace_bytes(cfg.B, max(T0, T_out)), dtype=torch.uint8, device="cuda")
        self.x_out = torch.empty((T_out, D), dtype=torch.float32, device="cuda")
        self.sizes_out = torch.empty(T_out, dtype=torch.int32, device="cuda")

    def step(self):
        off = self.ctx.otas_prompt_prepend(self.t_tok, self.tok_off, self.t_prm, self.prm_off, self.x0)
        if self.deep is not None:
            self.ctx.otas_encoder_forward_deep(self.x0, off, self.deep_mode, self.deep, self.prm_off, self.ws,
                                               self.x_out, self.sizes_out)
        else:
            self.ctx.otas_encoder_forward(self.x0, off, self.R, 0, self.ws, self.x_out, self.sizes_out)

    def time_steps(self, steps, warmup):
        import torch
        for _ in range(warmup):
            self.step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            self.step()
        torch.cuda.synchronize()
        self.ms_step = (time.perf_counter() - t0) / steps * 1e3

    def time_single_forwards(self, runs=21):
        """Latency of ONE forward pass (prompt prepend included) as a serving batch sees it: the GPU is
        idle when the call starts and the pass is waited for; HIP events on the stream the library works
        on (the context was created on torch's current stream); median of `runs`."""
        import torch
        t = []
        for _ in range(runs):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            self.step()
            e1.record()
            e1.synchronize()
            t.append(e0.elapsed_time(e1))
        self.latency_ms = float(np.median(t))
        self.latency_runs = runs

    def measure_clock(self, steps):
        """Shader clock while this workload runs back to back: the library's one-wave probe samples it (every
        32512 clocks) beside `steps` steps; it is sized to end before they do even if the clock never drops."""
        import torch
        torch.cuda.synchronize()
        n = int(max(64, min(60000, 0.45 * steps * self.ms_step / 0.01355)))
        self.ctx.otas_clock_probe_start(n)
        for _ in range(steps):
            self.step()
        mhz = np.asarray(self.ctx.otas_clock_probe_read(), dtype=np.float64)
        torch.cuda.synchronize()
        mhz = mhz[len(mhz) // 10:]          # the first tenth covers the launch ramp
        self.clock = {"median": round(float(np.median(mhz)), 0), "p10": round(float(np.percentile(mhz, 10)), 0),
                      "p90": round(float(np.percentile(mhz, 90)), 0), "samples": int(len(mhz)), "steps": steps}

    def idle_clock(self):
        import torch
        torch.cuda.synchronize()
        self.ctx.otas_clock_probe_start(400)
        mhz = np.asarray(self.ctx.otas_clock_probe_read(), dtype=np.float64)
        return round(float(np.median(mhz[40:])), 0)

    def time_launches(self, timing_steps):
        """Per-kernel durations: the same steps again with an event pair around every launch."""
        import torch
        import paper_2401_05031_amd as otas
        ctx, cfg = self.ctx, self.cfg
        ctx.otas_timing_enable(True)
        for _ in range(timing_steps):
            self.step()
        recs = ctx.otas_timing_read_launches()
        ev_overhead_us = ctx.otas_timing_overhead_ms() * 1e3
        ctx.otas_timing_enable(False)
        n_per = len(recs) // timing_steps
        assert n_per * timing_steps == len(recs)
        per_step, per_launch = {}, {}
        for i in range(n_per):          # launch i of a step: its kind, and its mean duration over the steps
            kind = recs[i][0]
            ms = float(np.mean([recs[s * n_per + i][1] for s in range(timing_steps)]))
            per_launch.setdefault(kind, []).append(ms)
        for kind in ctx.otas_timing_kind_names():
            v = per_launch.get(kind, [])
            per_step[kind] = (float(sum(v)), len(v))
        work = algorithmic_work(cfg, self.lengths0, self.R, otas, ctx)
        assert torch.isfinite(self.x_out.float()).all()
        return {"name": self.name, "cfg": cfg, "ctx": ctx, "R": list(self.R), "ms": self.ms_step,
                "img_s": cfg.B / (self.ms_step * 1e-3),
                "latency_ms": self.latency_ms, "latency_runs": self.latency_runs, "clock": self.clock,
                "kernels": per_step, "launches": per_launch, "work": work, "ev_overhead_us": ev_overhead_us}


def measured_traffic(workload):
    """Per-launch HBM bytes per kernel family measured offline with rocprofv3 --pmc (see
    paper_2401_05031_amd/traffic.py); None for workloads that were not measured."""
    path = os.path.join(ROOT, "paper_2401_05031_amd", "hbm_traffic.json")
    try:
        d = json.load(open(path))
    except OSError:
        return {}
    return {k: v["bytes"] for k, v in d["families"].items()} if d.get("workload") == workload else {}


def rooflines(res):
    k, w = res["kernels"], res["work"]
    full = res["cfg"].B == synth.config(res["name"]).B      # the stored traffic is the full batch's
    traffic = measured_traffic(res["name"]) if full else {}
    gemm_ms = sum(k[n][0] for n in ("gemm_qkv", "gemm_proj", "gemm_fc1", "gemm_fc2"))
    gemm_launches = sum(k[n][1] for n in ("gemm_qkv", "gemm_proj", "gemm_fc1", "gemm_fc2"))
    gemm_flops = sum(w[n] for n in ("gemm_qkv", "gemm_proj", "gemm_fc1", "gemm_fc2"))
    out = {}
    ach = gemm_flops / (gemm_ms * 1e-3) / 1e12 if gemm_ms > 0 else 0.0
    out["gemm"] = {"bound": "mfma", "achieved": round(ach, 2), "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                   "frac": round(ach / PEAK_BF16_TFLOPS, 4), "traffic": traffic.get("gemm"),
                   "launches_per_step": gemm_launches, "avg_launch_us": round(gemm_ms * 1e3 / max(gemm_launches, 1), 2),
                   "flops_per_launch": gemm_flops / max(gemm_launches, 1)}
    # the same with nothing subtracted from the event readings (each launch then also carries what its event pair adds)
    raw_ms = gemm_ms + gemm_launches * res["ev_overhead_us"] * 1e-3
    if raw_ms > 0:
        out["gemm"]["achieved_without_overhead_subtraction"] = round(gemm_flops / (raw_ms * 1e-3) / 1e12, 2)
        out["gemm"]["frac_without_overhead_subtraction"] = round(gemm_flops / (raw_ms * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 4)
    for n in ("gemm_qkv", "gemm_proj", "gemm_fc1", "gemm_fc2"):
        if k[n][0] > 0:
            a = w[n] / (k[n][0] * 1e-3) / 1e12
            out[n] = {"bound": "mfma", "achieved": round(a, 2), "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                      "frac": round(a / PEAK_BF16_TFLOPS, 4), "avg_launch_us": round(k[n][0] * 1e3 / max(k[n][1], 1), 2)}
    # In merging layers of head-width-64 bf16 models the library launches attention and the merge plan as one
    # kernel (recorded as attention): its time then covers both, and no merge_plan launch is recorded.
    fused_plan = k["merge_plan"][1] == 0 and any(int(r) > 0 for r in res.get("R", []))
    if k["attention"][0] > 0:
        a = w["attention"] / (k["attention"][0] * 1e-3) / 1e12
        out["attention"] = {"bound": "mfma", "achieved": round(a, 2), "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                            "frac": round(a / PEAK_BF16_TFLOPS, 4), "traffic": traffic.get("attention"),
                            "avg_launch_us": round(k["attention"][0] * 1e3 / max(k["attention"][1], 1), 2)}
        if fused_plan:
            out["attention"]["includes_merge_plan"] = True
            out["attention"]["note"] = ("these launches also run the layer's merge plan (one kernel, the plan's "
                                        "workgroups first; its list-writing phases move into the projection's launch "
                                        "where that has workgroup slots to spare): the time covers both, the FLOP "
                                        "count attention alone")
    if k["merge_apply"][0] > 0:
        a = w["merge_apply_bytes"] / (k["merge_apply"][0] * 1e-3) / 1e9
        out["merge_apply"] = {"bound": "hbm", "achieved": round(a, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                              "frac": round(a / PEAK_HBM_GBS, 4), "traffic": traffic.get("merge_apply"),
                              "algorithmic_bytes_per_launch": round(w["merge_apply_bytes"] / max(k["merge_apply"][1], 1)),
                              "method_bytes_per_launch": round(w["merge_apply_method_bytes"] / max(k["merge_apply"][1], 1)),
                              "frac_on_method_bytes": round(w["merge_apply_method_bytes"] / (k["merge_apply"][0] * 1e-3) / 1e9 / PEAK_HBM_GBS, 4),
                              "avg_launch_us": round(k["merge_apply"][0] * 1e3 / max(k["merge_apply"][1], 1), 2)}
    if k["merge_apply"][0] > 0 and w["merge_apply_bytes_per_layer"]:
        # the largest launch (the first merging layer): later layers shrink until launch latency dominates
        b0, t0 = w["merge_apply_bytes_per_layer"][0], res["launches"]["merge_apply"][0]
        a = b0 / (t0 * 1e-3) / 1e9
        out["merge_apply_first_layer"] = {"bound": "hbm", "achieved": round(a, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                                          "frac": round(a / PEAK_HBM_GBS, 4), "algorithmic_bytes": round(b0),
                                          "method_bytes": round(w["merge_apply_method_bytes_per_layer"][0]),
                                          "frac_on_method_bytes": round(w["merge_apply_method_bytes_per_layer"][0] / (t0 * 1e-3) / 1e9 / PEAK_HBM_GBS, 4),
                                          "launch_us": round(t0 * 1e3, 2)}
    if k.get("splitk_reduce_ln", (0, 0))[0] > 0:
        a = w["splitk_reduce_bytes"] / (k["splitk_reduce_ln"][0] * 1e-3) / 1e9
        out["splitk_reduce_ln"] = {"bound": "hbm", "achieved": round(a, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                                   "frac": round(a / PEAK_HBM_GBS, 4), "launches_per_step": k["splitk_reduce_ln"][1],
                                   "frac_on_method_bytes": round(w["splitk_reduce_method_bytes"] / (k["splitk_reduce_ln"][0] * 1e-3) / 1e9 / PEAK_HBM_GBS, 4),
                                   "avg_launch_us": round(k["splitk_reduce_ln"][0] * 1e3 / k["splitk_reduce_ln"][1], 2)}
    if k["layer_norm"][0] > 0:
        a = w["layer_norm_bytes"] / (k["layer_norm"][0] * 1e-3) / 1e9
        out["layer_norm"] = {"bound": "hbm", "achieved": round(a, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                             "frac": round(a / PEAK_HBM_GBS, 4), "traffic": traffic.get("layer_norm"),
                             "frac_on_method_bytes": round(w["layer_norm_method_bytes"] / (k["layer_norm"][0] * 1e-3) / 1e9 / PEAK_HBM_GBS, 4),
                             "avg_launch_us": round(k["layer_norm"][0] * 1e3 / max(k["layer_norm"][1], 1), 2)}
    # one row per GEMM launch of a forward pass: rows, the kernel the library picks (block tile, workgroup
    # slots on 256 CUs), tiles, rounds of those slots, microseconds, TFLOP/s.  Kernels 3 and 7 have tiles of several sizes and
    # pick one by the rows: tiles and rounds are not given for them
    tiles_of = {1: (64, 64, 2048), 2: (128, 128, 768), 4: (192, 256, 256), 5: (256, 256, 256),
                6: (320, 256, 256), 8: (160, 256, 256), 9: (224, 256, 256), 10: (288, 256, 256)}
    names = {3: "128|160x128", 7: "small"}
    cfg, ctx = res["cfg"], res.get("ctx")
    if ctx is not None and not cfg.deep:
        table = []
        shapes = {"gemm_qkv": (w["T"][:cfg.L], 3 * cfg.D, cfg.D, 0), "gemm_proj": (w["T"][:cfg.L], cfg.D, cfg.D, 2),
                  "gemm_fc1": (w["Tm"], cfg.F, cfg.D, 1), "gemm_fc2": (w["Tm"], cfg.D, cfg.F, 2)}
        for kind, (rows, N, K, epi) in shapes.items():
            for l, (M, ms) in enumerate(zip(rows, res["launches"].get(kind, []))):
                S = w["splits"][l] if kind == "gemm_fc2" else 1
                # split products run the partial-output form of kernel 3 or 7 (not told apart here)
                kid = 0 if S > 1 else ctx.otas_linear_choice(M, N, K, epi)
                bm, bn, slots = tiles_of.get(kid, (0, 0, 1))
                tiles = -(-M // bm) * -(-N // bn) * S if bm else 0
                table.append({"kind": kind, "layer": l, "M": int(M), "N": N, "K": K, "kernel": kid, "tile": f"{bm}x{bn}" if bm else names.get(kid, "split"),
                              "split_k": S, "tiles": int(tiles), "rounds": round(tiles / slots, 2), "us": round(ms * 1e3, 1),
                              "tflops": round(2.0 * M * N * K / (ms * 1e-3) / 1e12, 1)})
        out["gemm_per_launch"] = table
    for n in ("merge_plan", "prompt_prepend"):
        if k[n][1] > 0:
            out[n] = {"avg_launch_us": round(k[n][0] * 1e3 / k[n][1], 2), "launches_per_step": k[n][1]}
    out["note_hbm_kernels"] = ("achieved / frac count the bytes these kernels move with the float residual stream "
                               "(4 B per element of a token row) and, in launches of up to 4096 rows, of the next "
                               "linear's weight, which they read ahead; frac_on_method_bytes prices the same launches at "
                               "what the method needs with rows in the model's dtype (2 B): the gap is the cost of "
                               "keeping the residual in float")
    out["kernel_ms_per_step"] = {n: round(v[0], 4) for n, v in k.items()}
    out["event_pair_overhead_us_subtracted"] = round(res["ev_overhead_us"], 2)
    return out


def cpu_baseline(name, n_queries):
    """The oracle, as it stands, on the host cores over a bounded sample of the same workload: float64
    arithmetic (the value), and the same sample again with float32 arithmetic (second figure)."""
    from oracle import otas_oracle as orc
    cfg = synth.config(name)
    layers = synth.all_weights(cfg)
    toks, prm, P, R = synth.batch(cfg, list(range(n_queries)))
    try:
        from threadpoolctl import threadpool_info
        threads = max([p.get("num_threads", 1) for p in threadpool_info()] + [1])
    except Exception:
        threads = len(os.sched_getaffinity(0))
    storage = "bf16" if cfg.dtype == "bf16" else "f64"
    dts = {}
    for arith in ("f64", "f32"):
        t0 = time.perf_counter()
        for q in range(n_queries):
            x0, _ = orc.prompt_prepend(toks[q], prm[q], cfg.n_lead)
            orc.encoder_forward_query(x0, layers, R[q], H=cfg.H, ln_eps=cfg.ln_eps, n_lead=cfg.n_lead,
                                      storage=storage, arith=arith)
        dts[arith] = time.perf_counter() - t0
    return {"value": round(n_queries / dts["f64"], 3), "unit": "images/s", "cores": int(threads), "kind": "oracle",
            "value_f32_arithmetic": round(n_queries / dts["f32"], 3),
            "sample": f"{n_queries} of {cfg.B} queries of {name}, NumPy oracle with bf16 storage rounding: float64 "
                      f"arithmetic {dts['f64']:.1f} s (the value), float32 arithmetic {dts['f32']:.1f} s; host has "
                      f"{len(os.sched_getaffinity(0))} usable cores"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="vitb_r16", choices=list(synth.CONFIG_NAMES))
    ap.add_argument("--others", default="vitb_plain,vitb_p10_r8,vitb_deep10_replace,vitb_deep2_grow,vitl_ragged,vith_mixed",
                    help="further workloads reported per strategy (the two large ragged ones run few steps)")
    ap.add_argument("--batch", type=int, default=0,
                    help="run the headline workload on its first BATCH queries only (latency studies and profiler runs of "
                         "small batches; the stored HBM traffic figures do not apply then and are left out)")
    ap.add_argument("--small-batches", default="1,4,8,16,32",
                    help="batch sizes whose single-forward latency is reported beside the full batch's ('' = none)")
    ap.add_argument("--cpu-queries", type=int, default=32)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-clock", action="store_true",
                    help="skip the shader-clock pass (profiler runs: the probe is a kernel that lasts as long as the steps)")
    ap.add_argument("--calibrate", action="store_true",
                    help="also run one plain device copy of 256 MiB (torch) so that a rocprofv3 --pmc run of this "
                         "command holds a kernel of known HBM traffic to scale FETCH_SIZE / WRITE_SIZE by")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU (queries are independent, so more GPUs would be plain data "
              "parallelism with no collective); --gpus must be 1", file=sys.stderr)
        sys.exit(2)
    import torch
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback", file=sys.stderr)
        sys.exit(3)

    if args.calibrate:
        a = torch.empty(256 << 20, dtype=torch.uint8, device="cuda").random_(0, 255)
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        b.copy_(a)                      # 256 MiB read + 256 MiB written
        torch.cuda.synchronize()
        del a, b
    # Wall-clock runs of every strategy first, the per-launch event passes afterwards: once timing
    # events have been recorded in a process, cross-stream dependencies cost more (measured: the
    # merge plan's fork/join adds ~170 us per layer), which must not leak into a later strategy's
    # throughput.
    names = [args.workload] + [n for n in args.others.split(",") if n and n != args.workload]
    strategies = [Strategy(n, args.batch if i == 0 else 0) for i, n in enumerate(names)]
    # Everything is set up: move what exists out of the garbage collector's sight.  With torch imported a
    # full collection takes ~38 ms on the host, and one of them landing inside a 50-step timed region
    # (the host runs at most a few steps ahead of the GPU) reads as +0.7 ms per step for that strategy.
    gc.collect()
    gc.freeze()
    for i, st in enumerate(strategies):
        big = st.cfg.L * st.cfg.D * st.cfg.B > 12 * 768 * 64 * 2      # ViT-L / ViT-H batches: 12 / 73 ms a step
        st.time_steps(args.steps if i == 0 else (max(5, args.steps // 8) if big else max(5, args.steps // 2)),
                      args.warmup if not big else min(args.warmup, 3))
    for st in strategies:
        st.time_single_forwards(21)
    # Small batches of the headline workload: median of 21 single forward passes each (prepend included), one
    # context per batch size, closed again at once.
    small = {}
    for b in [int(v) for v in args.small_batches.split(",") if v]:
        if b >= strategies[0].cfg.B:
            continue
        sb = Strategy(args.workload, b)
        sb.time_steps(5, 3)
        sb.time_single_forwards(21)
        small[str(b)] = round(sb.latency_ms, 4)
        sb.ctx.close()
        del sb
    # The clock figures are an extra: if the probe fails, the line is still printed without them.
    idle_mhz = None
    for i, st in enumerate(strategies):
        big = st.cfg.L * st.cfg.D * st.cfg.B > 12 * 768 * 64 * 2
        st.clock = None
        if args.no_clock:
            continue
        try:
            if idle_mhz is None:
                idle_mhz = st.idle_clock()
            st.measure_clock(4 if big else 20)
        except Exception as e:      # noqa: BLE001
            print(f"bench.py: shader-clock probe failed for {st.name}: {e}", file=sys.stderr)
            st.clock = None
    all_res = [st.time_launches(max(3, min(10, args.steps)) if i == 0 else 3) for i, st in enumerate(strategies)]
    head = all_res[0]
    per_strategy = {}
    for r in all_res:
        P, R = r["cfg"].strategies[0]
        mixed = len(set(r["cfg"].strategies)) > 1
        rf = rooflines(r)
        rf.pop("gemm_per_launch", None)
        per_strategy[r["name"]] = {
            "strategy": "mixed" if mixed else ({"prompts": P, "r": R, "per_layer": r["cfg"].deep} if r["cfg"].deep
                                               else {"prompts": P, "r": R}),
            "images_per_s": round(r["img_s"], 1), "ms_per_step": round(r["ms"], 4),
            "single_forward_ms_median": round(r["latency_ms"], 4), "single_forward_runs": r["latency_runs"],
            "single_forward_images_per_s": round(r["cfg"].B / (r["latency_ms"] * 1e-3), 1),
            "gemm_tflops": rf["gemm"]["achieved"],
            "shader_clock_mhz_median": r["clock"]["median"] if r["clock"] else None,
            "merge_apply_gbs": rf.get("merge_apply", {}).get("achieved"),
            "attention_tflops": rf.get("attention", {}).get("achieved"),
        }
    rf = rooflines(head)
    cfg = head["cfg"]
    out = {
        "metric": BASELINE_METRIC if cfg.B == synth.config(cfg.name).B
        else BASELINE_METRIC + f" [this run: the first {cfg.B} queries of the batch only]",
        "value": round(head["img_s"], 1), "unit": "images/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(head["ms"], 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": cfg.dtype, "data": "synthetic",
        "config": {"workload": f"{cfg.name}: L={cfg.L} D={cfg.D} H={cfg.H} F={cfg.F}, batch {cfg.B} x {cfg.n0} tokens, "
                               f"strategy (P, r) = {'mixed' if len(set(cfg.strategies)) > 1 else cfg.strategies[0]}",
                   "global_batch": cfg.B, "seq_len": cfg.n0, "parallelism": "single GPU"},
        "single_forward_ms_median": round(head["latency_ms"], 4),
        "small_batch_single_forward_ms_median": small,
        "roofline": dict({k: rf["gemm"][k] for k in ("bound", "achieved", "peak", "unit", "frac", "traffic")},
                         traffic_source="rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this command, stored in "
                                        "paper_2401_05031_amd/hbm_traffic.json (profiles/hbm_traffic_vitb_r16_pmc.md); "
                                        "not re-measured by this run"),
        "shader_clock": None if head["clock"] is None else {
            "rated_mhz": RATED_MHZ, "idle_mhz": idle_mhz, "under_load_mhz": head["clock"],
            "peak_at_measured_clock": round(PEAK_BF16_TFLOPS * head["clock"]["median"] / RATED_MHZ, 1),
            "gemm_frac_of_peak_at_measured_clock":
                round(rf["gemm"]["achieved"] / (PEAK_BF16_TFLOPS * head["clock"]["median"] / RATED_MHZ), 4),
            "note": "the data-sheet peak (roofline.peak) is 256 CUs x 4 matrix cores x 1024 FLOP per clock at 2400 MHz; "
                    "under sustained matrix work on random operands the chip lowers its clock (measured here by a "
                    "one-wave probe beside the timed steps), so the same cycles-per-tile efficiency yields a smaller "
                    "fraction of that peak"},
        "rooflines": rf,
        "per_strategy": per_strategy,
    }
    for st in strategies:
        st.ctx.close()
    if not args.no_cpu:
        out["cpu_baseline"] = cpu_baseline(args.workload, args.cpu_queries)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
