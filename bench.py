"""Benchmark: planned graph latency on one MI355X.

One step = one fluid_run of the whole layout-planned, arena-planned
transformer graph (every operator of the chain: one launch per non-view
node, except the nodes a MatMul performs in its epilogue and the products
launched together) over one batch of synthetic input already resident in
HBM.

Default workload: the 24-layer BERT-large-shaped post-LN encoder, fp32,
batch 8, seq 512, hidden 1024, 16 heads, FFN 4096 (seed 4) -- the largest
fp32 workload.  The cost table is measured on the GPU first (untimed), then
the layout plan and the Greedy-by-Size arena are computed, then W warm-up
and K timed steps run.  The same K steps are timed for the naive plan
(row-major layouts, every transpose materialised, one arena slice per
tensor) for comparison.  The other workloads (BERT-base, GPT-2-small
prefill, Llama prefill in bf16) are reported under extra_workloads.

Prints one JSON line.  Usage:
  python bench.py [--gpus 1] [--steps K] [--warmup W] [--config 4] [--extra 2,3,5]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0
PEAK_TFLOPS = {"f32": 157.3, "bf16": 2516.6}
# fp32 products summed from six bf16 ones on the bf16 matrix cores (launch
# names gemm_f32_s<tile>, conv_f32_s<tile>)
PEAK_SPLIT_TFLOPS = round(PEAK_TFLOPS["bf16"] / 6, 1)


def peak_tflops(launch_name, dtype):
    """The matrix peak of the unit that the launch's kernel runs on."""
    import re
    return PEAK_SPLIT_TFLOPS if re.match(r"(gemm|conv)_f32_s\d", launch_name) else PEAK_TFLOPS[dtype]

# HBM bytes per launch of each workload's dominant launch: two rocprofv3
# --pmc passes (FETCH_SIZE, then WRITE_SIZE) over `bench.py --kernel-only`
# (that launch alone, planned from the saved cost tables), each scaled by
# what the same counter read for the 256 MiB calibration copy (FETCH_SIZE
# counts half the bytes read, WRITE_SIZE all the bytes written).  Keyed by
# (workload, launch name, node signatures); each figure carries the hash of
# its kernel family's device sources when it was taken and is reported as
# `traffic` only while they are unchanged (else null).
TRAFFIC = {
    ('bert-large-24l-b8-s512-h1024', 'gemm_f32_s128_ak_bk_cn_eb',
     '[[\'matmul\', \'(8, 512, 1024)\', "((8, 512, 1024), (\'c\', 1024, 1024))"], [\'add\', \'(8, 512, 1024)\', "((8, 512, 1024), (\'c\', 1024))"]]'): (67907574, '132fec4696567d1e'),
    ('llama-8l-b1-s2048-h4096-prefill', 'gemm_bf16_p256x128s3_ak_bmn_cn',
     '[[\'matmul\', \'(1, 2048, 11008)\', "((1, 2048, 4096), (\'c\', 4096, 11008))"]]'): (894099167, '132fec4696567d1e'),
    ('gpt2-small-12l-b1-s512-h768-prefill', 'gemm_f32_dl32w4_ak_bmn_cn_ebg',
     '[[\'matmul\', \'(1, 512, 3072)\', "((1, 512, 768), (\'c\', 768, 3072))"], [\'add\', \'(1, 512, 3072)\', "((1, 512, 3072), (\'c\', 3072))"], [\'gelu\', \'(1, 512, 3072)\', \'((1, 512, 3072),)\']]'): (28431743, '132fec4696567d1e'),
    ('bert-base-12l-b1-s128-h768', 'gemm_f32_dl32w4_ak_bmn_cn_ebg',
     '[[\'matmul\', \'(1, 128, 3072)\', "((1, 128, 768), (\'c\', 768, 3072))"], [\'add\', \'(1, 128, 3072)\', "((1, 128, 3072), (\'c\', 3072))"], [\'gelu\', \'(1, 128, 3072)\', \'((1, 128, 3072),)\']]'): (14277143, '132fec4696567d1e'),
    ('vgg16-b1-224', 'conv_f32_s64x64_kcuv_ks4',
     '[[\'conv\', \'(1, 256, 56, 56)\', "((1, 256, 58, 58), (\'c\', 256, 256, 3, 3), (\'c\', 256))"]]'): (35250587, 'e30b4fb1ac56c921'),
}

# the device sources of each kernel family (by launch-name prefix)
FAMILY_SOURCES = {"gemm": ["k_gemm*.hip", "gemm_common.h", "split_common.h", "dev.h"],
                  "conv": ["k_conv*.hip", "gemm_common.h", "split_common.h", "dev.h"],
                  "": ["k_elementwise.hip", "k_reduce.hip", "dev.h"]}


# Cost tables measured on an MI355X for the benchmark workloads (Alg. 3's
# eval is a compile-time step: measured once per graph, kernel build and GPU
# model, then reused).  index.json records, per workload, the hash of the
# library sources the numbers depend on; a table whose sources changed is
# measured afresh instead.
STORED_TABLES = os.path.join(ROOT, "paper_2411_09242_amd", "tables")


def library_source_hash():
    """Hash of the library sources a cost table's numbers depend on: the
    device code (kernels and the measurement protocol), how a variant
    becomes launch parameters, the candidate layouts, the fusion rules, the
    graph builders and the table format."""
    import glob
    import hashlib
    d = os.path.join(ROOT, "paper_2411_09242_amd", "csrc")
    files = glob.glob(os.path.join(d, "gpu", "*"))
    for stem in ("dispatch", "kparams", "layouts", "fusion", "graph", "costtable", "prepare"):
        files += glob.glob(os.path.join(d, "host", stem + ".*"))
    h = hashlib.sha256()
    for f in sorted(files):
        h.update(os.path.relpath(f, d).encode())
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def stored_table_meta(wl):
    p = os.path.join(STORED_TABLES, "index.json")
    if not os.path.exists(p):
        return None
    with open(p) as f:
        return json.load(f).get(wl)


def kernel_source_hash(launch_name):
    import glob
    import hashlib
    d = os.path.join(ROOT, "paper_2411_09242_amd", "csrc", "gpu")
    fam = next(f for f in ("gemm", "conv", "") if launch_name.startswith(f))
    files = sorted(f for pat in FAMILY_SOURCES[fam] for f in glob.glob(os.path.join(d, pat)))
    h = hashlib.sha256()
    for f in files:
        h.update(os.path.basename(f).encode())
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def log(*a):
    print(*a, file=sys.stderr, flush=True)


class Markers:
    """ROCTx ranges around the timed regions, so that a kernel trace taken
    with rocprofv3 --marker-trace can be cut to exactly those dispatches.
    No-ops when the ROCTx library is not present."""

    def __init__(self):
        import ctypes
        self.lib = None
        for name in ("librocprofiler-sdk-roctx.so.1", "librocprofiler-sdk-roctx.so", "libroctx64.so"):
            try:
                self.lib = ctypes.CDLL(name)
                break
            except OSError:
                continue
        if self.lib is not None:
            self.lib.roctxRangePushA.argtypes = [ctypes.c_char_p]

    def push(self, name):
        if self.lib is not None:
            self.lib.roctxRangePushA(name.encode())

    def pop(self):
        if self.lib is not None:
            self.lib.roctxRangePop()


MARK = Markers()


def node_work(g, n):
    """Algorithmic work of one launch of node n: ('flop', 2MNK) for a MatMul,
    else ('bytes', inputs read once + output written once)."""
    nd = g.desc["nodes"][n]
    isz = 2 if g.dtype == "bf16" else 4
    if nd["op"] == "matmul":
        a = g.edge_shape(nd["ins"][0])
        K = a[-1]
        N = nd["out_shape"][-1]
        M = int(np.prod(nd["out_shape"][:-1]))
        return "flop", 2.0 * M * N * K
    if nd["op"] == "conv":      # 2 * output elements * (C * KH * KW)
        w = g.desc["consts"][~nd["ins"][1]]["shape"]
        return "flop", 2.0 * float(np.prod(nd["out_shape"])) * float(np.prod(w[1:]))
    b = 0
    for v in nd["ins"]:
        if v >= 0:
            b += int(np.prod(g.edge_shape(v))) * isz
    b += int(np.prod(nd["out_shape"])) * isz
    return "bytes", float(b)


def node_sig(g, n):
    """(op, output shape, input shapes) of node n; constants as ('c', ...)."""
    nd = g.desc["nodes"][n]
    return (nd["op"], tuple(nd["out_shape"]),
            tuple(tuple(g.edge_shape(v)) if v >= 0 else ("c",) + tuple(g.desc["consts"][~v]["shape"])
                  for v in nd["ins"]))


def launch_units(g, ex):
    """The launches one fluid_run enqueues, in order: per launch its kernel
    name (with the fused epilogue steps and the group size), the nodes it
    performs (node order) and its algorithmic work -- the flops of its
    products for a GEMM launch (grouped products summed; a fused bias or
    activation adds no flops), else the bytes of its one node (for a
    residual Add and its normalisation in one launch: the summands read
    once, the normalised output written once, and the sum written once when
    the launch stores it; its class is the norm's)."""
    launch, written, names = ex.schedule()
    units = [{"name": nm, "nodes": []} for nm in names]
    for n, l in enumerate(launch):
        if l >= 0:
            units[l]["nodes"].append(n)
    for i, u in enumerate(units):
        mm = [n for n in u["nodes"] if g.desc["nodes"][n]["op"] in ("matmul", "conv")]
        if mm:
            u["op"], u["kind"] = g.desc["nodes"][mm[0]]["op"], "flop"
            u["work"] = sum(node_work(g, n)[1] for n in mm)
        elif len(u["nodes"]) == 2 and g.desc["nodes"][u["nodes"][0]]["op"] == "add":
            h, n = u["nodes"]
            u["op"] = g.desc["nodes"][n]["op"]
            isz = 2 if g.dtype == "bf16" else 4
            u["kind"] = "bytes"
            out_b = int(np.prod(g.desc["nodes"][n]["out_shape"])) * isz
            u["work"] = float(sum(int(np.prod(g.edge_shape(v))) * isz for v in g.desc["nodes"][h]["ins"]) +
                              out_b * (2 if written[h] else 1))
        else:
            assert len(u["nodes"]) == 1, u
            n = u["nodes"][0]
            u["op"] = g.desc["nodes"][n]["op"]
            u["kind"], u["work"] = node_work(g, n)
        u["index"] = i
        u["sig"] = (u["name"],) + tuple(node_sig(g, n) for n in u["nodes"])
    return units


def time_steps(ex, steps, stream, torch):
    """K eager steps, an event after each: (mean ms, [per-step ms])."""
    torch.cuda.synchronize()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    ev[0].record()
    for i in range(steps):
        ex.run(stream)
        ev[i + 1].record()
    torch.cuda.synchronize()
    per = [ev[i].elapsed_time(ev[i + 1]) for i in range(steps)]
    return ev[0].elapsed_time(ev[-1]) / steps, per


def time_units(ex, units, repeat, torch, marker=None):
    """ms per pass of the given launches issued back to back exactly as
    fluid_run issues them (fluid_run_nodes over their nodes, so that fused
    epilogues and grouped products run as one launch): `repeat` passes
    captured in one HIP graph (so that host launch cost does not pace small
    kernels), one warm-up replay, then one replay between two events on the
    replay stream."""
    nodes = [n for u in units for n in u["nodes"]]
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        ex.run_nodes(nodes, 1, s.cuda_stream)
        s.synchronize()
        with torch.cuda.graph(g, stream=s):
            ex.run_nodes(nodes, repeat, s.cuda_stream)
        g.replay()
        s.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        if marker:
            MARK.push(marker)
        e0.record(s)
        g.replay()
        e1.record(s)
        s.synchronize()
        if marker:
            MARK.pop()
    torch.cuda.current_stream().wait_stream(s)
    del g
    return e0.elapsed_time(e1) / repeat


def op_class_rates(g, units, ex, steps, torch):
    """Per operator class (the operator of a launch's first node; a GEMM
    launch with a fused epilogue counts as matmul): ms per step of its
    launches back to back (one HIP graph) and the rate against the class's
    bound.  Nodes performed inside another launch are not counted again."""
    by_op = {}
    for u in units:
        by_op.setdefault(u["op"], []).append(u)
    out = {}
    for op, us in by_op.items():
        ms_c = time_units(ex, us, max(3, min(steps, 20)), torch)
        work = sum(u["work"] for u in us)
        if us[0]["kind"] == "flop":
            rate = work / (ms_c * 1e-3) / 1e12
            # the class's peak rate: its work at each launch's own peak
            peak, unit = work / sum(u["work"] / peak_tflops(u["name"], g.dtype) for u in us), "TFLOP/s"
        else:
            rate = work / (ms_c * 1e-3) / 1e9
            peak, unit = PEAK_HBM_GBS, "GB/s"
        out[op] = {"ms_per_step": round(ms_c, 4), "launches_per_step": len(us),
                   "achieved": round(rate, 2), "unit": unit, "frac": round(rate / peak, 4)}
    return dict(sorted(out.items(), key=lambda kv: -kv[1]["ms_per_step"]))


def graph_ms(ex, steps, torch, marker=None):
    """ms per step: `steps` runs captured in one HIP graph, one warm-up
    replay, one replay between two events."""
    hg = ex.capture(steps=steps)
    hg.replay()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    if marker:
        MARK.push(marker)
    e0.record()
    hg.replay()
    e1.record()
    torch.cuda.synchronize()
    if marker:
        MARK.pop()
    del hg
    return e0.elapsed_time(e1) / steps


def ablation(F, g, table, ex, steps, torch):
    """Layout DP, kernel variants and priced fusion chains switched on one
    at a time (same cost table, same Greedy-by-Size arena planner): graph
    latency, planned table total and per-operator-class times of each plan.
    Without pricing (and without the DP) a MatMul performs the nodes after
    it whenever its tile can (fusion by adjacency, after planning)."""
    out = {}
    for name, flags in (("identity_layouts_variant0", F.NO_DP | F.NO_VARIANTS),
                        ("identity_layouts_best_variant", F.NO_DP),
                        ("dp_layouts_variant0", F.NO_VARIANTS),
                        ("dp_layouts_best_variant_adjacent_fusion", F.NO_FUSION),
                        ("dp_layouts_best_variant", 0)):
        lp_a = F.LayoutPlan(g, table, flags)
        ap_a = F.ArenaPlan(g, lp_a, epilogue=True)
        ex_a = F.Executor(g, lp_a, ap_a, ex.consts, ex.inputs)
        for _ in range(2):
            ex_a.run()
        torch.cuda.synchronize()
        out[name] = {"ms_per_step": round(graph_ms(ex_a, steps, torch), 4), "table_ns": lp_a.total_ns,
                     "launches_per_step": ex_a.launches(), "priced_chains": sum(1 for t in lp_a.fuse if t),
                     "peak_arena_mb": round(ap_a.peak / 2**20, 3),
                     "op_ms": {op: c["ms_per_step"]
                               for op, c in op_class_rates(g, launch_units(g, ex_a), ex_a, steps, torch).items()}}
        del ex_a
        torch.cuda.empty_cache()
    return out


def calibration_copy(torch, mib=256):
    """A plain device-to-device copy of known size, inside its own marker
    range: HBM counters of the kernels are scaled by what the same counters
    read for this copy."""
    src = torch.empty(mib << 18, dtype=torch.float32, device="cuda").fill_(1.0)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    MARK.push(f"calibration_copy_{mib}MiB")
    dst.copy_(src)
    torch.cuda.synchronize()
    MARK.pop()
    del src, dst
    torch.cuda.empty_cache()


def cpu_baseline(cfg, budget_s=20.0, seed=4):
    """The oracle (plain NumPy, float64, as it stands) on the host, on a
    bounded sample of the workload: for the large workloads the graph of the
    first two layers at full batch and sequence (the layers are identical, so
    a step costs layers / 2 times as much), else the whole graph; median of
    the runs that fit in the budget (at least one), scaled to one step."""
    import synth_inputs
    from oracle import execute, graph as OG
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:  # noqa: BLE001
        threads = len(os.sched_getaffinity(0))
    big = cfg["arch"] != "vgg" and cfg["batch"] * cfg["seq"] * cfg["hidden"] >= 2 ** 21
    k = 2 if big and cfg["layers"] > 2 else cfg.get("layers", 1)
    og = OG.build_transformer(dict(cfg, layers=k))
    x, consts = synth_inputs.make_inputs(cfg, og.const_specs(), seed)
    times = []
    t_start = time.time()
    while True:
        t = time.time()
        execute.run_canonical(og, [x], consts)
        times.append(time.time() - t)
        if time.time() - t_start > budget_s or len(times) >= 5:
            break
    scale = cfg["layers"] / k
    what = (f"first {k} of {cfg['layers']} layers at full batch and sequence, x{scale:g}" if k < cfg["layers"]
            else f"whole {cfg['layers']}-layer graph")
    return {"value": round(1000.0 * float(np.median(times)) * scale, 3), "unit": "ms", "cores": int(threads),
            "kind": "oracle",
            "sample": f"{what}; {len(times)} run(s), median {1000.0 * float(np.median(times)):.1f} ms per run; "
                      f"float64 NumPy"}


def row_major_weights(F, g, table):
    """The same cost table without the packed-weight MatMul variants
    (10-19): the naive plan keeps every weight row-major as supplied."""
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        p = os.path.join(d, "t.json")
        table.save(p)
        with open(p) as f:
            obj = json.load(f)
        for sig in obj["sigs"] + obj.get("fused_sigs", []):
            if sig["op"] == "matmul":
                for ent in sig["entries"]:
                    ent[2] = [c if v < 10 else -1 for v, c in enumerate(ent[2])]
        with open(p, "w") as f:
            json.dump(obj, f)
        return F.CostTable.load(p, g)


def measure_workload(F, torch, cfg, x, consts, steps, warmup, reps, save_table=None, tables=None,
                     kernel_only=False, plan_steps=False):
    """Cost table (untimed), plans, then the timed regions; returns a dict.
    tables: (directory, "save" | "load") -- keep each workload's measured
    table, or plan from a kept one instead of measuring (same plan, e.g. for
    counter runs); (STORED_TABLES, "stored") -- plan from the stored table
    while the library sources are those it was measured with, else measure;
    (STORED_TABLES, "store") -- measure and store it.  kernel_only: after
    planning, launch only the dominant kernel's nodes K times (eagerly) and
    return which kernel that was."""
    g = F.Graph.transformer(cfg)
    wl = cfg["name"]
    stream = torch.cuda.current_stream().cuda_stream
    t = time.time()
    tpath = os.path.join(tables[0], wl + ".json") if tables else None
    mode = tables[1] if tables else None
    meta = stored_table_meta(wl) if mode == "stored" else None
    src = library_source_hash()
    if mode == "stored" and not (meta and meta.get("sources") == src and os.path.exists(tpath)):
        log(f"{wl}: no stored cost table for these library sources; measuring")
        mode = None
    if mode in ("load", "stored"):
        table = F.CostTable.load(tpath, g)
        table_info = {"source": "stored" if mode == "stored" else "loaded", "file": os.path.relpath(tpath, ROOT)}
        if meta:
            table_info.update({k: meta[k] for k in ("measure_s", "reps", "gpu", "sources") if k in meta})
    else:
        MARK.push(f"{wl}/cost_table")
        table = F.CostTable.measure(g, reps=reps)
        MARK.pop()
        table_info = {"source": "measured", "measure_s": round(time.time() - t, 1), "reps": reps, "sources": src}
        if mode in ("save", "store"):
            os.makedirs(tables[0], exist_ok=True)
            table.save(tpath)
        if mode == "store":
            ip = os.path.join(tables[0], "index.json")
            index = json.load(open(ip)) if os.path.exists(ip) else {}
            index[wl] = {k: v for k, v in table_info.items() if k != "source"}
            props = torch.cuda.get_device_properties(0)
            index[wl]["gpu"] = f"{props.name} ({props.gcnArchName.split(':')[0]})"
            with open(ip, "w") as f:
                json.dump(index, f, indent=1, sort_keys=True)
    t_measure = time.time() - t
    log(f"{cfg['name']}: cost table ready in {t_measure:.1f} s ({table_info['source']})")
    if save_table:
        table.save(save_table)
    lp = F.LayoutPlan(g, table)
    # operands of a MatMul live until the end of the nodes its epilogue
    # absorbs, so that every such fusion happens; the paper's lifetimes are
    # reported beside it
    apl = F.ArenaPlan(g, lp, epilogue=True)
    apl_paper = F.ArenaPlan(g, lp)
    lp_naive = F.LayoutPlan(g, row_major_weights(F, g, table), F.NO_DP)
    ap_naive = F.ArenaPlan(g, lp_naive, no_reuse=True)
    ex = F.Executor(g, lp, apl, consts, [x])
    ex_naive = F.Executor(g, lp_naive, ap_naive, consts, [x])
    del consts
    n_launch = ex.launches()
    n_launch_naive = ex_naive.launches()

    # warm-up; then, untimed for the result, each node signature's launches
    # back to back (a few passes) to find the dominant kernel, and each
    # operator class's launches back to back for the per-class rates
    for _ in range(warmup):
        ex.run(stream)
        ex_naive.run(stream)
    torch.cuda.synchronize()
    units = launch_units(g, ex)
    by_sig = {}
    for u in units:
        by_sig.setdefault(u["sig"], []).append(u)
    # dominant kernel: the launch signature (kernel instance with its fused
    # epilogue and group, and the shapes of the nodes it performs) with the
    # largest summed algorithmic time at its bound's peak (flops / MFMA peak
    # or bytes / HBM peak) -- fixed by the graph and the plan, not by timing
    # noise or by the per-dispatch overhead a tracer adds
    def ideal_ms(us):
        peak = (peak_tflops(us[0]["name"], g.dtype) * 1e12) if us[0]["kind"] == "flop" else (PEAK_HBM_GBS * 1e9)
        return sum(u["work"] for u in us) / peak
    dom_key = max(by_sig, key=lambda k: (ideal_ms(by_sig[k]), -by_sig[k][0]["index"]))
    dom = by_sig[dom_key]
    if kernel_only:
        ex.run_nodes([n for u in dom for n in u["nodes"]], steps, stream)
        torch.cuda.synchronize()
        return {"kernel": dom[0]["name"], "node_sigs": [list(map(str, x)) for x in dom_key[1:]],
                "launches": steps * len(dom)}
    if plan_steps:   # only the plan's own steps, eagerly (for a kernel trace of the graph)
        ms, _ = time_steps(ex, steps, stream, torch)
        return {"steps": steps, "eager_ms_per_step": round(ms, 4), "launches_per_step": len(units)}
    op_classes = op_class_rates(g, units, ex, steps, torch)

    # timed region 1: K eager steps (whole graph, no per-launch events)
    MARK.push(f"{wl}/eager_timed")
    ms_eager, per_step = time_steps(ex, steps, stream, torch)
    MARK.pop()
    # timed region 1b: the dominant kernel alone -- the launches of its nodes
    # back to back, K times over, with the bindings of a run (the arena holds
    # the data of the last step), replayed as one HIP graph between two
    # events on the replay stream
    launches = steps * len(dom)
    avg_ms = time_units(ex, dom, steps, torch, marker=f"{wl}/kernel_timed") / len(dom)
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    # timed region 2 (the reported latency): the same K steps captured into
    # one HIP graph; one warm-up replay, then one timed replay
    hg = ex.capture(steps=steps)
    hg.replay()
    torch.cuda.synchronize()
    MARK.push(f"{wl}/graph_timed")
    ev0.record()
    hg.replay()
    ev1.record()
    torch.cuda.synchronize()
    MARK.pop()
    ms_step = ev0.elapsed_time(ev1) / steps
    del hg
    hg_naive = ex_naive.capture(steps=steps)
    hg_naive.replay()
    torch.cuda.synchronize()
    MARK.push(f"{wl}/naive_graph_timed")
    ev0.record()
    hg_naive.replay()
    ev1.record()
    torch.cuda.synchronize()
    MARK.pop()
    ms_naive = ev0.elapsed_time(ev1) / steps
    del hg_naive
    ms_naive_eager, _ = time_steps(ex_naive, steps, stream, torch)

    kind, work = dom[0]["kind"], dom[0]["work"]
    tkey = (wl, dom[0]["name"], str([list(map(str, x)) for x in dom_key[1:]]))
    entry = TRAFFIC.get(tkey)
    traffic = entry[0] if entry and entry[1] == kernel_source_hash(dom[0]["name"]) else None
    if kind == "flop":
        achieved = work / (avg_ms * 1e-3) / 1e12
        peak = peak_tflops(dom[0]["name"], g.dtype)
        roof = {"bound": "mfma", "achieved": round(achieved, 2), "peak": peak, "unit": "TFLOP/s",
                "frac": round(achieved / peak, 4), "traffic": traffic}
    else:
        achieved = work / (avg_ms * 1e-3) / 1e9
        roof = {"bound": "hbm", "achieved": round(achieved, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                "frac": round(achieved / PEAK_HBM_GBS, 4), "traffic": traffic}
    roof.update({"kernel": dom[0]["name"], "node_sigs": [list(map(str, x)) for x in dom_key[1:]],
                 "avg_launch_us": round(avg_ms * 1e3, 3), "launches": launches,
                 "positions_in_step": [u["index"] for u in dom],
                 "work_per_launch": work, "work_unit": "flop" if kind == "flop" else "byte"})

    abl = ablation(F, g, table, ex, steps, torch)

    # planned vs naive outputs (same inputs, different layouts and kernels)
    out = ex.run(stream)[0].float()
    out_n = ex_naive.run(stream)[0].float()
    torch.cuda.synchronize()
    agree = float((out - out_n).abs().max().item())
    res = {
        "ms_per_step": round(ms_step, 4), "eager_ms": round(ms_eager, 4),
        "eager_step_ms_p10_p50_p90": [round(float(np.percentile(per_step, q)), 4) for q in (10, 50, 90)],
        "naive_ms": round(ms_naive, 4), "naive_eager_ms": round(ms_naive_eager, 4),
        "speedup_vs_naive": round(ms_naive / ms_step, 3),
        "peak_arena_mb": round(apl.peak / 2**20, 3), "naive_arena_mb": round(ap_naive.peak / 2**20, 3),
        "max_live_lower_bound_mb": round(apl.lower_bound / 2**20, 3),
        "paper_lifetimes_arena_mb": round(apl_paper.peak / 2**20, 3),
        "paper_lifetimes_launches_per_step": F.fluid_run_launches(g.h, lp.h, apl_paper.h),
        "launches_per_step": n_launch, "naive_launches_per_step": n_launch_naive,
        "plan_table_ns": lp.total_ns, "naive_table_ns": lp_naive.total_ns, "guard_used": lp.guard_used,
        "fusion_priced": lp.fusion_priced, "priced_chains": sum(1 for t in lp.fuse if t),
        "planned_vs_naive_max_abs_diff": agree, "cost_table": table_info,
        "roofline": roof,
        "op_classes": op_classes,
        "ablation": abl,
    }
    del ex, ex_naive
    torch.cuda.empty_cache()
    return res


def device_inputs(torch, F, cfg, seed):
    """Synthetic inputs drawn on the GPU (same distributions as the seeded
    host recipe: x ~ N(0,1), weights 0.02 N(0,1), biases/beta 0, gamma 1,
    RoPE tables from positions; for the convolutional workload an image batch
    and sqrt(2 / fan_in) N(0,1) weights); used for the extra workloads to keep the
    benchmark short.  Timing does not depend on the values."""
    import synth_inputs
    g = F.Graph.transformer(cfg)
    dt = torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)
    conv = cfg["arch"] == "vgg"
    xs = ((cfg["batch"], cfg["channels"], cfg["image"], cfg["image"]) if conv
          else (cfg["batch"], cfg["seq"], cfg["hidden"]))
    x = torch.randn(xs, generator=gen, device="cuda").to(dt)
    consts = []
    for c in g.desc["consts"]:
        shape, role = tuple(c["shape"]), c["role"]
        cdt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        if role == "weight":
            fan_in = (int(np.prod(shape[1:])) if len(shape) == 4 else shape[0]) if conv else 0
            std = float(np.sqrt(2.0 / fan_in)) if conv else 0.02
            a = (std * torch.randn(shape, generator=gen, device="cuda")).to(cdt)
        elif role == "gamma":
            a = torch.ones(shape, device="cuda", dtype=cdt)
        elif role in ("rope_cos", "rope_sin"):
            c_, s_ = synth_inputs.rope_tables(shape[0], 2 * shape[1], cfg.get("rope_base", 10000.0))
            a = torch.from_numpy(c_ if role == "rope_cos" else s_).cuda()
        else:
            a = torch.zeros(shape, device="cuda", dtype=cdt)
        consts.append(a)
    return x, consts


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--config", type=int, default=4)
    ap.add_argument("--extra", default="2,3,5,6", help="extra workloads to report ('' for none)")
    ap.add_argument("--reps", type=int, default=7, help="timed launches per cost-table entry")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--save-table", default=None)
    ap.add_argument("--tables-dir", default=None, help="directory for every workload's cost table")
    ap.add_argument("--tables-mode", choices=("save", "load"), default="save")
    ap.add_argument("--measure", action="store_true",
                    help="measure every cost table (default: the stored tables while the sources match)")
    ap.add_argument("--store-tables", nargs="?", const=STORED_TABLES, default=None, metavar="DIR",
                    help="measure every cost table and store it (default: with the library)")
    ap.add_argument("--kernel-only", action="store_true",
                    help="launch only each workload's dominant kernel (for counter runs); prints what ran")
    ap.add_argument("--plan-steps", action="store_true",
                    help="run only the plan's steps, eagerly (for a kernel trace of the whole graph)")
    a = ap.parse_args()
    if a.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on exactly one GPU: the executor has no multi-GPU path "
              "(one GPU's share of a sharded graph runs the same kernels).", file=sys.stderr)
        sys.exit(2)

    import torch
    import synth_inputs
    from paper_2411_09242_amd import fluid as F

    F.load()
    torch.cuda.init()
    calibration_copy(torch)
    cfg = synth_inputs.config(a.config)
    log(f"workload {cfg['name']}")
    if a.kernel_only or a.plan_steps:   # values do not matter for which kernels run or the bytes they move
        x, consts = device_inputs(torch, F, cfg, a.config)
    else:
        x, consts = synth_inputs.make_inputs(cfg, F.Graph.transformer(cfg).const_specs(), a.config)
    if a.tables_dir:
        tables = (a.tables_dir, a.tables_mode)
    elif a.store_tables:
        tables = (a.store_tables, "store")
    else:
        tables = None if a.measure else (STORED_TABLES, "stored")
    r = measure_workload(F, torch, cfg, x, consts, a.steps, a.warmup, a.reps, a.save_table, tables, a.kernel_only,
                         a.plan_steps)
    if a.kernel_only or a.plan_steps:
        print(json.dumps({"kernel_only" if a.kernel_only else "plan_steps": True, "workload": cfg["name"], **r}),
              flush=True)
        return
    res = {
        "metric": "graph latency (ms) + peak arena MB vs naive plan; kernel % of roofline",
        "value": r["ms_per_step"], "unit": "ms", "n_gpus": 1, "steps": a.steps, "warmup": a.warmup,
        "ms_per_step": r["ms_per_step"], "higher_is_better": False, "scaling": "weak",
        "vs_baseline": None, "dtype": cfg["dtype"], "data": "synthetic",
        "config": dict({"workload": cfg["name"]},
                       **{k: cfg[k] for k in ("arch", "layers", "batch", "seq", "hidden", "heads", "ffn", "channels",
                                              "image", "stages", "fc", "classes") if k in cfg},
                       parallelism="none (1 GPU)"),
        "timing": "value: K steps captured in one HIP graph, one timed replay; roofline: the "
                  "dominant kernel's launches (all nodes of its signature) back to back K times over, "
                  "replayed as one HIP graph between two HIP events, per-launch mean",
    }
    res.update({k: v for k, v in r.items() if k != "ms_per_step"})
    extras = {}
    for idx in [int(s) for s in a.extra.split(",") if s.strip()]:
        if idx == a.config:
            continue
        c = synth_inputs.config(idx)
        log(f"extra workload {c['name']}")
        xe, ce = device_inputs(torch, F, c, idx)
        st = max(5, a.steps // 2) if idx in (4, 5) else a.steps
        e = measure_workload(F, torch, c, xe, ce, st, max(2, a.warmup // 2), max(2, a.reps // 2), None, tables)
        e.update({"workload": c["name"], "dtype": c["dtype"], "steps": st,
                  "data": "synthetic, drawn on the GPU"})
        extras[f"cfg{idx}"] = e
        del xe, ce
        torch.cuda.empty_cache()
    if extras:
        res["extra_workloads"] = extras
    if not a.no_cpu_baseline:
        log("cpu baseline (oracle) ...")
        res["cpu_baseline"] = cpu_baseline(cfg, seed=a.config)
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
