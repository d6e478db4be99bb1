#!/usr/bin/env python3
"""Benchmark of the stitched hot path on one MI355X.

Headline workload: the largest of the five benchmark configurations, C4 = bias + tanh-GELU
forward fused with the bias-gradient column sum, x, grad bf16 [16384,3072] (302 MB of minimum
traffic; two launches per step: the stitched kernel and the fold of its column partial sums).
A step is one pass of the whole subgraph over one batch.  Inputs are resident in HBM before
the timed region; the step rotates through enough independent buffer sets that no set's inputs are
still in the 256 MB Infinity Cache when its turn comes again (cold-HBM rule; outputs are stored past it).

Prints ONE JSON line: metric/value = achieved GB/s on the subgraph's minimum traffic (each
input read once + each output written once) over the whole step, plus `roofline` -- which
carries `per_config`, the same measurement for all five configurations (C2 and C5 both as the
evaluator's choice and with the LDS scheme forced), each beside the per-op GPU baseline and
beside streaming probes of the same bytes and read : write mix -- and `cpu_baseline` (the
float64 per-op oracle timed on this machine's host).  Further context (the configurations' full
records, backward patterns, packed launches, explored programs, generated kernels) goes to stderr,
one JSON line too: some 30 KB, more than a reader of the last lines of stdout keeps.
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

HBM_PEAK_GBPS = 8000.0          # MI355X published HBM3E peak
CACHE_BYTES = 256 << 20         # Infinity Cache; the inputs of a rotation must be >= 2x this


TRAFFIC_PROFILE = "profiles/stitched_kernels_hbm_traffic_pmc.md"


def _profiled_traffic(tag: str, kernel: str = ""):
    """HBM bytes per step measured with rocprofv3 --pmc (FETCH_SIZE + WRITE_SIZE, scaled by a plain copy of
    known size, summed over the step's launches).  NOT measured in this run: read from the committed counter
    summary, whose lines `TRAFFIC_BYTES_PER_STEP <config> <kernels> <bytes>` were written from such a run.
    None when the summary was taken on another kernel than the one this run times (`kernel`: the plan's name of
    its stitched kernel, launch shape included)."""
    try:
        for line in open(os.path.join(ROOT, TRAFFIC_PROFILE)):
            parts = line.split()
            if len(parts) == 4 and parts[0] == "TRAFFIC_BYTES_PER_STEP" and parts[1] == tag:
                return float(parts[3]) if not kernel or kernel == parts[2] else None
    except OSError:
        pass
    return None


def _sets_needed(input_bytes: int) -> int:
    """Buffer sets that a cold rotation takes.  Inputs alone count: they may stay in the cache, what is stored does not."""
    return max(2, -(-2 * (CACHE_BYTES + (32 << 20)) // max(1, input_bytes)))


def rotation_sets(spec, most: int) -> int:
    return min(_sets_needed(traffic_split(spec)[0]), most)


class Runner:
    """One plan + rotating device buffer sets."""

    def __init__(self, spec, scheme="auto", seed=0, n_sets=None, host_inputs=None, **opts):
        import torch
        from paper_2009_10924_amd import binding as B
        from workloads import make_inputs
        self.torch, self.B, self.spec = torch, B, spec
        self.graph = B.Graph.from_spec(spec)
        self.plan = B.Plan(self.graph, scheme, **opts)
        self.info = self.plan.info
        self.host_inputs = host_inputs if host_inputs is not None else make_inputs(spec, seed)
        first = [B.to_device(self.host_inputs[t.name], t.dtype) for t in spec.inputs]
        self.n_sets = n_sets or rotation_sets(spec, 4096)
        self.inputs = [first] + [[t.clone() for t in first] for _ in range(self.n_sets - 1)]
        self.outputs = [B.alloc_outputs(spec) for _ in range(self.n_sets)]
        self.workspaces = [self.plan.make_workspace() for _ in range(self.n_sets)]
        self.stream = torch.cuda.current_stream().cuda_stream
        self._calls = [self.plan.bind([t.data_ptr() for t in i], [t.data_ptr() for t in o],
                                      w.data_ptr() if w is not None else 0, w.numel() if w is not None else 0, self.stream)
                       for i, o, w in zip(self.inputs, self.outputs, self.workspaces)]
        self.step_no = 0

    def step(self):
        self._calls[self.step_no % self.n_sets]()
        self.step_no += 1

    def time_region(self, steps, warmup):
        """(wall seconds, event seconds) for `steps` back-to-back executes after `warmup` untimed ones."""
        torch = self.torch
        for _ in range(warmup):
            self.step()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0 = time.perf_counter()
        e0.record()
        for _ in range(steps):
            self.step()
        e1.record()
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        return wall, e0.elapsed_time(e1) * 1e-3

    def per_launch_events(self, steps):
        """Average over `steps` of an event pair around each single execute (includes the pair's own overhead)."""
        torch = self.torch
        pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
        for a, b in pairs:
            a.record()
            self.step()
            b.record()
        torch.cuda.synchronize()
        ts = sorted(a.elapsed_time(b) * 1e-3 for a, b in pairs)
        return sum(ts) / len(ts), ts[len(ts) // 2], ts[0]


def copy_ceiling(steps=50, nbytes=1 << 30):
    """GB/s (read+write) of the library's plain streaming copy over buffers far larger than the caches."""
    import torch
    from paper_2009_10924_amd import binding as B
    src = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    src.fill_(1)
    for _ in range(3):
        B.stream_copy(dst, src)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        B.stream_copy(dst, src)
    e1.record()
    torch.cuda.synchronize()
    sec = e0.elapsed_time(e1) * 1e-3 / steps
    return 2 * nbytes / sec / 1e9


def time_oracle(spec, host_inputs, min_seconds=10.0, max_repeats=50):
    """Wall-clock of the float64 per-op oracle on this host (single-threaded numpy kernels): (seconds per pass,
    passes timed, whether an untimed warm pass came first).  A first pass that already takes `min_seconds` is the
    sample itself, so that the bounded sample stays at 10-30 s of CPU work."""
    from oracle import oracle as O
    t0 = time.perf_counter()
    O.evaluate(spec, host_inputs)
    first = time.perf_counter() - t0
    if first >= min_seconds:
        return first, 1, False
    reps, t0 = 0, time.perf_counter()
    while True:
        O.evaluate(spec, host_inputs)
        reps += 1
        dt = time.perf_counter() - t0
        if dt >= min_seconds or reps >= max_repeats:
            return dt / reps, reps, True


def traffic_split(spec):
    """(input bytes, output bytes) of a subgraph: what one step must read and must write."""
    from workloads import DTYPE_BYTES
    import math
    from paper_2009_10924_amd import binding as B
    shapes = B.output_shapes(spec)
    bytes_in = sum(math.prod(t.dims) * DTYPE_BYTES[t.dtype] for t in spec.inputs)
    bytes_out = sum(math.prod(shapes[name]) * DTYPE_BYTES[dt] for name, dt in spec.outputs)
    return bytes_in, bytes_out


# (read-only GB/s, write-only GB/s) of the streaming probes on 1 GiB, measured once per run by directional_rates()
_DIRECTIONAL = None


def directional_rates():
    global _DIRECTIONAL
    if _DIRECTIONAL is None:
        gib = 1 << 30
        _DIRECTIONAL = (gib / min(probe_us(gib, 2, 0, k, steps=30) for k in (1, 2, 4)) / 1e3,
                        gib / min(probe_us(gib, 0, 1, k, steps=30) for k in (1, 2, 4)) / 1e3)
        import torch
        torch.cuda.empty_cache()
    return _DIRECTIONAL


def directional_bound_us(spec):
    """Lower bound on a step's time from its traffic alone: the data bus carries reads and writes one after the other, so
    input bytes at the best measured read-only rate plus output bytes at the best measured write-only rate (both on
    1 GiB, so without a small launch's ramp and drain) is a time no kernel with this traffic goes below.  The same-size
    streaming probe beside it is a reference kernel, not a bound: a stitched kernel can beat it by a few percent."""
    rd, wr = directional_rates()
    bytes_in, bytes_out = traffic_split(spec)
    return bytes_in / rd / 1e3 + bytes_out / wr / 1e3


def stream_mix(spec):
    """(reads, writes) of equal-sized streams whose ratio is closest to the subgraph's input : output bytes."""
    import math
    bytes_in, bytes_out = traffic_split(spec)
    ratio = bytes_in / max(1, bytes_out)
    return min(((1, 1), (2, 1), (3, 1), (4, 1), (3, 2), (1, 2)), key=lambda m: abs(math.log(ratio / (m[0] / m[1]))))


def probe_us(total_bytes, reads, writes, vecs_per_lane=2, steps=200):
    """us of the streaming probe (fs_stream_probe) that moves `total_bytes` as `reads` input and `writes` output
    streams of equal size through rotating cold buffers: the traffic-only bound for a kernel of this footprint and
    read : write mix (launch ramp and drain included)."""
    import torch
    from paper_2009_10924_amd import binding as B
    stream_bytes = max(16, (total_bytes // (reads + writes)) // 16 * 16)
    n_sets = min(_sets_needed((reads or writes) * stream_bytes), 4096)
    srcs = [torch.empty(max(16, reads * stream_bytes), dtype=torch.uint8, device="cuda").fill_(3) for _ in range(n_sets)]
    dsts = [torch.empty(max(16, writes * stream_bytes), dtype=torch.uint8, device="cuda") for _ in range(n_sets)]
    stream = torch.cuda.current_stream().cuda_stream
    calls = [B.bind_probe(d.data_ptr(), s.data_ptr(), stream_bytes, reads, writes, vecs_per_lane, stream) for d, s in zip(dsts, srcs)]
    for i in range(min(20, n_sets)):
        calls[i]()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for i in range(steps):
        calls[i % n_sets]()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) * 1e3 / steps


def grid_floor_us(workgroups, steps=400):
    """us of a launch of `workgroups` x 256 threads in which every lane loads one 128-bit vector and stores one
    (cold buffers): the fixed cost -- launch, first memory round trip, drain -- that a one-shot kernel of that grid
    pays whatever else it does."""
    return probe_us(2 * 16 * 256 * max(1, workgroups), 1, 1, vecs_per_lane=1, steps=steps)


def measure_config(name, spec, steps, warmup, with_unfused=True, scheme="auto", probes=True):
    r = Runner(spec, scheme)
    wall, ev = r.time_region(steps, warmup)
    sec = ev / steps
    out = {
        "workload": spec.name, "pattern": r.info["pattern"], "scheme": r.info["scheme"], "kernel": r.info["kernel"],
        "n_kernels": r.info["n_kernels"], "grid": r.info["grid"][0], "block": r.info["block"][0], "vgprs": r.info["vgprs"],
        "lds_bytes": r.info["lds_bytes"], "bytes_min": r.info["bytes_min"], "us": sec * 1e6,
        "GBps": r.info["bytes_min"] / sec / 1e9, "frac_of_peak": r.info["bytes_min"] / sec / 1e9 / HBM_PEAK_GBPS,
        "predicted_us": r.info["predicted_us"], "buffer_sets": r.n_sets, "launches_timed": steps,
    }
    if r.info["pattern"] == "row_generated":   # the generated kernel's own name, as kernel traces show it
        out["entry"] = [l.split()[1] for l in r.plan.describe().splitlines() if l.strip().startswith("entry ")][0]
    host = r.host_inputs
    del r
    import torch
    torch.cuda.empty_cache()
    if with_unfused:
        u = Runner(spec, "unfused", host_inputs=host, n_sets=out["buffer_sets"])   # inputs as cold as the stitched plan's
        _, evu = u.time_region(max(10, steps // 4), max(3, warmup // 4))
        secu = evu / max(10, steps // 4)
        out.update({"unfused_us": secu * 1e6, "unfused_kernels": u.info["n_kernels"],
                    "unfused_bytes_model": u.info["bytes_moved_model"], "speedup_vs_unfused": secu / sec})
        del u
        torch.cuda.empty_cache()
    if probes:
        reads, writes = stream_mix(spec)
        best = min(probe_us(out["bytes_min"], reads, writes, k, steps=max(50, min(300, steps))) for k in (1, 2, 4))
        torch.cuda.empty_cache()
        out["probe"] = {"mix": f"{reads}r:{writes}w", "us": best, "GBps": out["bytes_min"] / best / 1e3}
        out["frac_of_probe"] = best / out["us"]
        out["bound_us"] = directional_bound_us(spec)
        out["frac_of_bound"] = out["bound_us"] / out["us"]
        if out["grid"] * out["block"] * 32 < out["bytes_min"]:
            out["grid_floor_us"] = grid_floor_us(out["grid"] * out["block"] // 256)
            torch.cuda.empty_cache()
    return out


def measure_pack(name, steps, warmup):
    """Packed launch of many tiny independent subgraphs against one stitched launch each and against the
    per-op plans; every member keeps its own seeded inputs and outputs (all of it cache-resident: the
    regime is launch-bound, not bandwidth-bound)."""
    import torch
    from paper_2009_10924_amd import binding as B
    from workloads import PACK_CONFIGS, make_inputs
    specs = PACK_CONFIGS[name]()
    stream = torch.cuda.current_stream().cuda_stream
    plans = [B.Plan(B.Graph.from_spec(s), "auto") for s in specs]
    unfused = [B.Plan(B.Graph.from_spec(s), "unfused") for s in specs]
    pack = B.Pack(plans)
    dev_in = [[B.to_device(make_inputs(s, seed=i)[t.name], t.dtype) for t in s.inputs] for i, s in enumerate(specs)]
    dev_out = [B.alloc_outputs(s) for s in specs]
    packed = pack.bind([t.data_ptr() for m in dev_in for t in m], [t.data_ptr() for m in dev_out for t in m], stream)
    ws = [p.make_workspace() for p in unfused]
    sep_calls = [p.bind([t.data_ptr() for t in i], [t.data_ptr() for t in o], 0, 0, stream) for p, i, o in zip(plans, dev_in, dev_out)]
    unf_calls = [p.bind([t.data_ptr() for t in i], [t.data_ptr() for t in o], w.data_ptr() if w is not None else 0,
                        w.numel() if w is not None else 0, stream) for p, i, o, w in zip(unfused, dev_in, dev_out, ws)]

    def timed(fn, n):
        for _ in range(warmup):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(n):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e3 / n

    def all_separate():
        for c in sep_calls:
            c()

    def all_unfused():
        for c in unf_calls:
            c()

    t_pack = timed(packed, steps)
    with B.codegen(False):   # the fixed packed kernel (run-time table of members) beside the generated one
        fixed_pack = B.Pack([B.Plan(B.Graph.from_spec(s), "auto") for s in specs])
    fixed = fixed_pack.bind([t.data_ptr() for m in dev_in for t in m], [t.data_ptr() for m in dev_out for t in m], stream)
    t_fixed = timed(fixed, steps)
    t_sep = timed(all_separate, max(10, steps // 8))
    t_unf = timed(all_unfused, max(5, steps // 32))
    return {"workload": f"{name}: {len(specs)} independent tiny subgraphs (8 softmax f32 [64,128], 8 add+bias+LayerNorm f32->bf16 "
                        "[128,768], 8 softmax backward f16 [384,128], 4 RMSNorm bf16 [64,1024], 4 bias+GELU bf16 [64,3072])",
            "members": len(specs), "bytes_min": pack.info["bytes_min"],
            "packed_us": t_pack, "packed_launches": pack.info["n_kernels"], "packed_grid": pack.info["grid"], "packed_vgprs": pack.info["vgprs"],
            "packed_GBps": pack.info["bytes_min"] / t_pack / 1e3, "packed_generated": pack.info["generated"],
            "fixed_pack_us": t_fixed, "fixed_pack_vgprs": fixed_pack.info["vgprs"],
            "stitched_one_launch_each_us": t_sep, "stitched_launches": sum(p.info["n_kernels"] for p in plans),
            "unfused_us": t_unf, "unfused_launches": sum(p.info["n_kernels"] for p in unfused),
            "speedup_vs_one_launch_each": t_sep / t_pack, "speedup_vs_unfused": t_unf / t_pack,
            "predicted_us": pack.info["predicted_us"], "predicted_separate_us": pack.info["predicted_separate_us"]}


def measure_program(name, steps, warmup):
    """A multi-pattern graph cut into fusion patterns by the explorer, against the same graph one kernel per op."""
    import torch
    from paper_2009_10924_amd import binding as B
    from workloads import EXPLORE_CONFIGS, make_inputs
    spec = EXPLORE_CONFIGS[name]()
    g = B.Graph.from_spec(spec)
    t0 = time.perf_counter()
    prog = B.Program(g)
    explore_ms = (time.perf_counter() - t0) * 1e3
    info = prog.info
    host = make_inputs(spec, 0)
    first = [B.to_device(host[t.name], t.dtype) for t in spec.inputs]
    n_sets = rotation_sets(spec, 64)
    inputs = [first] + [[t.clone() for t in first] for _ in range(n_sets - 1)]
    outputs = [B.alloc_outputs(spec) for _ in range(n_sets)]
    stream = torch.cuda.current_stream().cuda_stream
    ws = [prog.make_workspace() for _ in range(n_sets)]
    calls = [prog.bind([t.data_ptr() for t in i], [t.data_ptr() for t in o], w.data_ptr(), w.numel(), stream)
             for i, o, w in zip(inputs, outputs, ws)]
    # the per-op baseline of the same ops (one plan has no place for work between its kernels: the declared matrix
    # products are left out of its graph, as their results are in place for both timings anyway)
    import dataclasses
    unf = B.Plan(B.Graph.from_spec(dataclasses.replace(spec, external=[])), "unfused")
    uws = [unf.make_workspace() for _ in range(2)]
    ucalls = [unf.bind([t.data_ptr() for t in inputs[k]], [t.data_ptr() for t in outputs[k]],
                       uws[k % 2].data_ptr() if uws[0] is not None else 0, uws[0].numel() if uws[0] is not None else 0, stream)
              for k in range(n_sets)]

    def timed(fns, n):
        for k in range(warmup):
            fns[k % len(fns)]()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for k in range(n):
            fns[k % len(fns)]()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) * 1e3 / n

    t_prog = timed(calls, steps)
    t_unf = timed(ucalls, max(5, steps // 8))
    steps_info = prog.patterns()
    return {"workload": spec.name, "ops": info["n_ops"], "patterns": info["n_patterns"], "single_ops": info["n_single_ops"],
            "launches": prog.describe().count("\nmerged ") or info["n_kernels"], "packs": info["n_packs"], "stages": info["n_stages"], "joint_folds": info["n_joint_folds"],
            "workspace_bytes": info["workspace_bytes"],
            "bytes_min": info["bytes_min"], "us": t_prog, "GBps": info["bytes_min"] / t_prog / 1e3,
            "frac_of_peak": info["bytes_min"] / t_prog / 1e3 / HBM_PEAK_GBPS,
            "unfused_us": t_unf, "unfused_launches": unf.info["n_kernels"], "speedup_vs_unfused": t_unf / t_prog,
            "predicted_us": info["predicted_us"], "delta_evaluator_gain_us": info["f_total_us"], "explore_ms": explore_ms,
            "plan": [{"ops": len(s["ops"]), "pattern": s["info"]["pattern"], "kernel": s["info"]["kernel"]} for s in steps_info],
            "buffer_sets": n_sets}


HEADLINE = "C4"
HEADLINE_TEXT = ("C4 bias + tanh-GELU forward + bias-gradient column sum, x, grad bf16 [16384,3072], bias bf16 [3072] -> "
                 "y bf16, dbias fp32 [3072], seed 0 (the largest of the five configurations; 2 launches per step)")
# per_config rows: the five configurations as the evaluator runs them, and the two whose definitions name LDS
# (C2 "reused via LDS", C5 "LDS-tiled") also with the LDS scheme forced
PER_CONFIG = (("C1", "C1", "auto"), ("C2", "C2", "auto"), ("C2_lds", "C2", "lds"), ("C3", "C3", "auto"), ("C4", "C4", "auto"),
              ("C5", "C5", "auto"), ("C5_lds", "C5", "lds"))


def _row(m, tag):
    """The compact per_config row kept inside `roofline`."""
    row = {"kernel": m["kernel"], "scheme": m["scheme"], "launches": m["n_kernels"], "bytes_min": m["bytes_min"],
           "us": round(m["us"], 3), "GBps": round(m["GBps"], 1), "frac": round(m["frac_of_peak"], 4),
           "traffic": _profiled_traffic(tag, m["kernel"]), "unfused_us": round(m["unfused_us"], 2), "unfused_launches": m["unfused_kernels"],
           "speedup_vs_unfused": round(m["speedup_vs_unfused"], 2), "launches_timed": m["launches_timed"],
           "grid": m["grid"], "block": m["block"], "vgprs": m["vgprs"], "lds_bytes": m["lds_bytes"]}
    if "probe" in m:
        # ceiling: read bytes at the read-only rate + written bytes at the write-only rate (a bound); probe: the
        # streaming kernel of the same bytes, mix and one-shot shape (a reference that includes a small launch's ramp)
        row.update({"ceiling_us": round(m["bound_us"], 3), "ceiling_GBps": round(m["bytes_min"] / m["bound_us"] / 1e3, 1),
                    "frac_of_ceiling": round(m["frac_of_bound"], 4), "probe_mix": m["probe"]["mix"],
                    "probe_us": round(m["probe"]["us"], 3), "frac_of_probe": round(m["frac_of_probe"], 4)})
    if "grid_floor_us" in m:
        row["grid_floor_us"] = round(m["grid_floor_us"], 3)
    return row


LINE_KEYS = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype",
             "data", "config", "roofline", "wall_ms_per_step", "cpu_baseline")


def split_line(result):
    """(what the line on stdout holds, the rest)"""
    return ({k: v for k, v in result.items() if k in LINE_KEYS}, {k: v for k, v in result.items() if k not in LINE_KEYS})


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2000)
    ap.add_argument("--warmup", type=int, default=100)
    ap.add_argument("--no-context", action="store_true", help="headline, per_config and ceilings only: skip the oracle timing and the patterns beyond the five configurations")
    ap.add_argument("--only", default="", help="comma-separated per_config / context names to measure (for profiling runs), e.g. C4,N2,G11")
    ap.add_argument("--oracle-seconds", type=float, default=10.0)
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on one GPU only (rows would shard across GPUs with no exchange); use --gpus 1")

    import torch
    if not torch.cuda.is_available():
        sys.exit("bench.py: no GPU visible; the hot path has no CPU fallback")
    torch.cuda.set_device(0)
    from workloads import FULL_CONFIGS
    only = set(x for x in args.only.split(",") if x)

    def wanted(name):
        return not only or name in only

    spec = FULL_CONFIGS[HEADLINE]()
    r = Runner(spec, "auto")
    bytes_min = r.info["bytes_min"]
    wall, ev = r.time_region(args.steps, args.warmup)
    sec_step = ev / args.steps
    # one more pass with an event pair around every step (upper bound of the step's own duration)
    avg_pair, med_pair, min_pair = r.per_launch_events(min(args.steps, 200))
    achieved = bytes_min / sec_step / 1e9

    roofline = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                "frac": achieved / HBM_PEAK_GBPS, "traffic": _profiled_traffic(HEADLINE, r.info["kernel"]),
                "traffic_source": f"not measured in this run: rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE summary {TRAFFIC_PROFILE} (null where that summary was taken on another kernel)",
                "scope": "whole step = stitched kernel + fold launch; algorithmic bytes / (event time of the timed region / steps)",
                "algorithmic_bytes_per_step": bytes_min, "us_per_step_region": sec_step * 1e6,
                "us_per_step_event_pair": {"avg": avg_pair * 1e6, "median": med_pair * 1e6, "min": min_pair * 1e6}}
    result = {
        "metric": "achieved HBM GB/s (% of peak) per fused subgraph; speedup vs unfused per-op",
        "value": achieved, "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": sec_step * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": HEADLINE_TEXT, "pattern": r.info["pattern"], "scheme": r.info["scheme"], "kernel": r.info["kernel"],
                   "launches_per_step": r.info["n_kernels"], "block": r.info["block"], "grid": r.info["grid"], "vgprs": r.info["vgprs"],
                   "buffer_sets": r.n_sets, "cold_hbm_rotation_bytes": r.n_sets * traffic_split(r.spec)[0]},
        "roofline": roofline,
        "wall_ms_per_step": wall / args.steps * 1e3,
    }
    host_head = r.host_inputs
    del r
    torch.cuda.empty_cache()

    # ---- all five configurations, inside `roofline` ---------------------------------------------------------------
    n_cfg = max(200, args.steps)
    per_config, details = {}, {}
    for tag, cfg, scheme in PER_CONFIG:
        if not wanted(tag):
            continue
        m = measure_config(tag, FULL_CONFIGS[cfg](), n_cfg, max(10, args.warmup), scheme=scheme)
        details[tag] = m
        per_config[tag] = _row(m, tag)
        torch.cuda.empty_cache()
    roofline["per_config"] = per_config
    if wanted("ceilings"):
        # what the memory system gives traffic-only kernels on 1 GiB per stream set (cold by size)
        gib = 1 << 30
        roofline["ceilings_GBps"] = {
            "copy_1r1w": gib / min(probe_us(gib, 1, 1, k, steps=30) for k in (1, 2, 4)) / 1e3,
            "read_only": directional_rates()[0],
            "write_only": directional_rates()[1],
            "mix_2r1w": gib / min(probe_us(gib, 2, 1, k, steps=30) for k in (1, 2, 4)) / 1e3,
            "mix_4r1w": gib / min(probe_us(gib, 4, 1, k, steps=30) for k in (1, 2, 4)) / 1e3,
            "library_copy_kernel": copy_ceiling(),
        }
        torch.cuda.empty_cache()
    if "C1" in per_config:
        # C1 is launch-bound (8 ns of traffic at peak): its floor is one launch of a 16-byte copy
        tiny_src = torch.zeros(16, dtype=torch.uint8, device="cuda")
        tiny_dst = torch.zeros(16, dtype=torch.uint8, device="cuda")
        from paper_2009_10924_amd import binding as B
        tiny = B.bind_copy(tiny_dst.data_ptr(), tiny_src.data_ptr(), 16, torch.cuda.current_stream().cuda_stream)
        for _ in range(50):
            tiny()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(2000):
            tiny()
        e1.record()
        torch.cuda.synchronize()
        per_config["C1"]["launch_floor_us"] = round(e0.elapsed_time(e1) * 1e3 / 2000, 3)

    if not args.no_context and not only:
        sec_o, reps, warmed = time_oracle(spec, host_head, args.oracle_seconds, max_repeats=20)
        result["cpu_baseline"] = {"value": bytes_min / sec_o / 1e9, "unit": "GB/s", "cores": 1, "kind": "oracle",
                                  "sample": f"full C4 batch [16384,3072] (numpy float64, one op at a time), {reps} pass(es) {'after one warm pass' if warmed else 'timed from cold'}, {sec_o:.3f} s each",
                                  "seconds_per_subgraph": sec_o, "host_cpus": os.cpu_count(),
                                  "affinity": len(os.sched_getaffinity(0))}
    del host_head
    result["per_config_details"] = details

    if not args.no_context:
        from workloads import softmax_graph
        if wanted("C1_rows_2pow20"):
            # the same kernel as C1 on 2^20 rows shows that the kernel itself streams
            result["C1_rows_2pow20"] = measure_config("C1_large", softmax_graph(1 << 20, 128, "f32"), 30, 5, with_unfused=False)
            torch.cuda.empty_cache()
        from workloads import NEXT_CONFIGS
        # patterns beyond the five configurations: softmax / LayerNorm backward, innermost-axis-moving transposes
        result["next_patterns"] = {name: measure_config(name, NEXT_CONFIGS[name](), max(50, args.steps // 4), 20)
                                   for name in ("N1", "N2", "N3", "N4", "N5", "N6") if wanted(name)}
        torch.cuda.empty_cache()
        if wanted("P1"):
            result["packing"] = measure_pack("P1", max(200, args.steps // 2), 20)
            torch.cuda.empty_cache()
        for key, name in (("explorer", "T1"), ("explorer_T2", "T2"), ("explorer_T3", "T3")):
            if wanted(name):
                result[key] = measure_program(name, max(100, args.steps // 8), 10)
                torch.cuda.empty_cache()
        # row-local patterns outside the hand-written families: one generated kernel each
        from workloads import GENERIC_CONFIGS
        from paper_2009_10924_amd import binding as B
        generic = {}
        for name in ("G1", "G2", "G3", "G4", "G5", "G6", "G7", "G8", "G9", "G10", "G11", "G12"):
            if not wanted(name):
                continue
            gspec = GENERIC_CONFIGS[name]()
            generic[name] = measure_config(name, gspec, max(50, args.steps // 8), 10)   # AUTO: the kernel generated for the pattern
            with B.codegen(False):                                                       # the interpreted row program beside it
                r = Runner(gspec, "auto")
            if r.info["pattern"] == "row_program":   # patterns with column sums have no interpreted form
                _, ev = r.time_region(50, 5)
                generic[name].update({"interpreted_us": ev / 50 * 1e6, "interpreted_kernel": r.info["kernel"]})
            del r
            torch.cuda.empty_cache()
        result["generic_patterns"] = generic
    line, context = split_line(result)
    if context:
        print(json.dumps(context), file=sys.stderr, flush=True)
    print(json.dumps(line))


if __name__ == "__main__":
    main()
