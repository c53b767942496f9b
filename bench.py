#!/usr/bin/env python3
"""Decode-attention benchmark on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W]

One step is one call of the whole path -- plan (host), split-partial kernel,
and the log-sum-exp merge of the chunk states when the plan splits (inside
the split launch or in a second launch, as the plan says) -- over synthetic
N(0,1) bf16 inputs already resident in HBM.  Calls are captured in HIP
graphs and replayed; HIP events on the replay stream bracket the timed
replays, and the variants of a workload are interleaved round by round with
the order rotated (the paper times with CUDA-graph replay and A/B
interleaving, Section 5).  Every timed launch is first checked against the
fp64 oracle (sampled sequences on 1 GiB shapes); a launch that disagrees is
reported and the run exits with status 3.

Printed: one JSON line.  `value` is microseconds per call of the planned
launch on the high-load shape (B=32, H_Q=64, H_KV=8, D=128, L_K=8192, 1 GiB of
K/V), with its HBM roofline and counter traffic, its split sweep and one
split as the paper launches it.  Beside it: the Llama-3.1-70B GQA decode
shape (B=1, L_K=512) against one split, a split sweep, both merges and a cold
cache; B=1 contexts of 1024-8192 keys; the low-head workloads (MQA, pure MQA,
varlen GQA) against the paper's one-split launch; the same shapes with every
call reading its cache from HBM; batches of mixed lengths under the
per-sequence schedule; the high-load call beside a GEMM on reserved CUs; a
plain 1 GiB read kernel (the HBM read ceiling); and the fp64 oracle timed on
the host cores (a reported baseline only).  Compact summaries come last.
"""

from __future__ import annotations

import argparse
import contextlib
import gc
import hashlib
import json
import math
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "decode-attention µs/call + achieved HBM GB/s (% of peak), heuristic vs num_splits=1"
HBM_PEAK_GBS = 8000.0
PROFILE_TRAFFIC = os.path.join(ROOT, "profiles", "traffic.json")
KERNEL_SOURCES = [os.path.join(ROOT, "paper_2604_00028_amd", "csrc", f)
                  for f in ("decode_attn.hip", "plan.cpp", "plan.h", "cost_model.inc", "split_table.inc")]
SWEEP = (1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64)
HIGHLOAD_SWEEP = (1, 2, 3, 4, 6, 8, 12, 16)
LONG_SWEEP = (1, 2, 4, 8, 12, 16, 24)
# The paper's regression matrix (Section 5.3): Batch x L_K x H_KV, here with H_Q = 8 * H_KV.
REG_B = (1, 2, 4, 8)
REG_L = (128, 256, 384, 512, 576, 640, 768, 1024, 2048, 4096, 8192)
REG_HKV = (1, 2, 4, 8, 32)
REG_SWEEP = (1, 2, 3, 4, 6, 8, 12, 16, 24, 32)
PROFILE_REGRESSION = os.path.join(ROOT, "profiles", "regression_matrix.md")


def log(msg: str) -> None:
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200, help="calls per timed replay")
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--rounds", type=int, default=7, help="interleaved timed replays per variant")
    ap.add_argument("--highload-steps", type=int, default=20)
    ap.add_argument("--no-highload", action="store_true")
    ap.add_argument("--no-long", action="store_true", help="skip the L_K = 1024/2048/8192 block")
    ap.add_argument("--no-small", action="store_true", help="skip the MQA / low-tile / varlen block")
    ap.add_argument("--no-streamed", action="store_true", help="skip the K/V-streamed-from-HBM block")
    ap.add_argument("--no-ragged", action="store_true", help="skip the mixed-length (per-sequence schedule) block")
    ap.add_argument("--no-cu-margin", action="store_true",
                    help="skip the cu_margin block (decode beside a GEMM on reserved CUs)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--lk", type=int, default=8192, help="with --only long: L_K of the B=1 Llama-70B GQA shape")
    ap.add_argument("--shape", default="1,32,1,512", help="with --only shape: B,H_Q,H_KV,L_K (fixed layout)")
    ap.add_argument("--occupancy-summary", metavar="DIR", default=None,
                    help="summarise rocprofv3 occupancy counter runs DIR/occ_<pass>_<case> into "
                         "profiles/occupancy_heuristic_vs_s1.md")
    ap.add_argument("--only", choices=("headline", "highload", "long", "shape", "ragged", "copy", "readprobe"),
                    default=None,
                    help="time only the planned launch of one workload, a plain 1 GiB device copy (the reference "
                         "for HBM traffic counters) or the 1 GiB read probe, for profiler runs")
    ap.add_argument("--num-splits", type=int, default=0, help="with --only: force num_splits")
    ap.add_argument("--combine", type=int, default=-1,
                    help="with --only and a forced num_splits > 1: merge the chunk states in a second launch (0) or "
                         "inside the split launch (1); -1 leaves it to the planner")
    ap.add_argument("--pack-gqa", type=int, default=-1,
                    help="with --only: force pack_gqa (2: one workgroup per KV head and chunk, the paper's launch)")
    ap.add_argument("--regression", metavar="OUT_JSON", default=None,
                    help="time the paper's 160-configuration regression matrix (heuristic, num_splits=1, the "
                         "paper's policy and fixed splits) and write the results to OUT_JSON")
    ap.add_argument("--regression-summary", metavar="IN_JSON", default=None,
                    help="summarise a --regression result into profiles/regression_160_configs.md")
    ap.add_argument("--schedule-sweep", metavar="OUT_JSON", default=None,
                    help="time per-sequence schedules (modelled and fixed chunk lengths) against uniform launches "
                         "on mixed-length batches and write the results to OUT_JSON")
    ap.add_argument("--schedule-sweep-summary", metavar="IN_JSON", default=None,
                    help="summarise a --schedule-sweep result into profiles/schedule_mixed_length_batches.md")
    ap.add_argument("--mixed-sweep", metavar="OUT_JSON", default=None,
                    help="time the dealt launch against the launch with one split count on batches of mixed and "
                         "equal lengths and write the results to OUT_JSON")
    ap.add_argument("--mixed-sweep-summary", metavar="IN_JSON", default=None,
                    help="summarise a --mixed-sweep result into profiles/dealt_route_mixed_batches.md")
    ap.add_argument("--waves-sweep", metavar="OUT_JSON", default=None,
                    help="time one-split launches of two waves per workgroup against four on shapes of 192-1024 "
                         "workgroups (the planner's own wave count and the other one) and write OUT_JSON")
    ap.add_argument("--waves-sweep-summary", metavar="IN_JSON", default=None,
                    help="summarise a --waves-sweep result into profiles/two_waves_vs_four_waves.md")
    ap.add_argument("--calibrate", metavar="OUT_JSON", default=None,
                    help="time every launch the planner can choose (split count, tile width, V slices, merge) over "
                         "the calibration shapes, each output checked against the oracle, and write the sweep that "
                         "paper_2604_00028_amd/calibrate.py fits the cost model to")
    ap.add_argument("--calibrate-set", choices=("warm", "streamed"), default="warm",
                    help="with --calibrate: K/V resident between calls (warm) or read from HBM on every call")
    ap.add_argument("--traffic-summary", metavar="DIR", default=None,
                    help="derive per-launch HBM traffic from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE output "
                         "directories DIR/pmc_<COUNTER>_<workload> and write profiles/traffic.json")
    return ap.parse_args()


@contextlib.contextmanager
def no_gc():
    """No cyclic garbage collection inside: one that frees an older variant's
    graph during a capture ends the process."""
    gc.collect()
    gc.disable()
    try:
        yield
    finally:
        gc.enable()


class Variant:
    """K calls of one launch configuration captured in a HIP graph."""

    def __init__(self, name, da, torch, q, k, v, L, s, pack, steps, kv_copies=None, cu=None, plan=None):
        self.name = name
        B, H_Q, D = q.shape
        H_KV = k.shape[-2]
        # plan given: run it as it is (da_decode_attn_planned); else the library plans from (s, pack)
        self.plan = plan if plan is not None else da.da_make_plan(B, H_Q, H_KV, L, D, s, pack)
        nbytes = da.da_workspace_bytes(B, H_Q, D, self.plan.num_splits)
        self.ws = torch.zeros(max(nbytes, 256), dtype=torch.uint8, device="cuda") if nbytes else None
        self.out = torch.empty((B, H_Q, D), dtype=torch.bfloat16, device="cuda")
        self.steps = steps
        s_res, p_res = self.plan.num_splits, self.plan.pack_gqa
        kvs = kv_copies if kv_copies else [(k, v)]
        # the same launch on the same data: variants with equal keys pool their timings (pack_gqa only
        # names the packing a tile width comes from, so plans that differ in it alone are one launch)
        self.key = (launch_key(self.plan), q.data_ptr(), kvs[0][0].data_ptr(), len(kvs),
                    None if cu is None else cu.data_ptr())

        def call(i):
            kk, vv = kvs[i % len(kvs)]
            if plan is not None:
                da.da_decode_attn_planned(q, kk, vv, plan, cu, out=self.out, L_K_max=L if cu is not None else None,
                                          workspace=self.ws)
            else:
                da.da_decode_attn(q, kk, vv, cu, out=self.out, L_K_max=L if cu is not None else None,
                                  num_splits=s_res, pack_gqa=p_res, workspace=self.ws)

        self.call = call
        for i in range(3):
            call(i)
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with no_gc(), torch.cuda.graph(self.graph):
            for i in range(steps):
                call(i)
        self.graph.replay()
        torch.cuda.synchronize()
        self.times = []

    def sample(self, torch):
        """The output of one eager call on the first K/V copy, written over
        NaNs: a launch that leaves any output unwritten (shared `out`
        buffers would otherwise hold another launch's result) fails the
        check."""
        self.out.fill_(float("nan"))
        self.call(0)
        torch.cuda.synchronize()
        return self.out.clone()

    def timed(self, torch) -> float:
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        self.graph.replay()
        b.record()
        torch.cuda.synchronize()
        us = a.elapsed_time(b) * 1000.0 / self.steps
        self.times.append(us)
        return us

    @property
    def median(self) -> float:
        return statistics.median(self.times)


class Timed:
    """K calls of any launch (call(i) issues call i, writing `out`) captured
    in a HIP graph."""

    def __init__(self, torch, call, steps, out=None, name=""):
        self.steps = steps
        self.call = call
        self.out = out
        self.name = name
        for i in range(3):
            call(i)
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with no_gc(), torch.cuda.graph(self.graph):
            for i in range(steps):
                call(i)
        self.graph.replay()
        torch.cuda.synchronize()
        self.times = []

    timed = Variant.timed
    median = Variant.median
    sample = Variant.sample


def interleave(torch, variants, rounds):
    """Time every variant `rounds` times, round-robin.  Variants that issue
    the same launch on the same data (a forced split count that the planner
    would choose anyway, say) are one configuration: they pool their
    timings, so that run-to-run noise is not reported as a difference
    between them."""
    n = len(variants)
    for r in range(rounds):
        # each round starts at another variant, so that no launch is always timed in the same place
        # (a fixed order biased equal launches by a few percent at a few microseconds)
        for j in range(n):
            variants[(r + j) % n].timed(torch)
    groups = {}
    for var in variants:
        key = getattr(var, "key", None)
        if key is not None:
            groups.setdefault(key, []).append(var)
    for same in groups.values():
        if len(same) > 1:
            pooled = [t for var in same for t in var.times]
            for var in same:
                var.times = list(pooled)


def algorithmic_bytes(B, H_Q, H_KV, L, D=128):
    from workloads import algorithmic_bytes as ab
    return ab(B, H_Q, H_KV, B * L, D)


def kernel_source_sha() -> str:
    """Hash of the sources that decide which kernel runs and what it reads:
    the kernels, and the planner and its constants that pick the variant."""
    h = hashlib.sha256()
    for path in KERNEL_SOURCES:
        h.update(open(path, "rb").read())
    return h.hexdigest()


def traffic_for(workload: str):
    """HBM bytes per launch from the committed rocprofv3 counter summary, if
    it was taken on the current kernel source; else None."""
    try:
        with open(PROFILE_TRAFFIC) as f:
            t = json.load(f)
        if t.get("kernel_source_sha256") != kernel_source_sha():
            return None
        w = t["workloads"][workload]
        return int(w["fetch_bytes"] + w["write_bytes"])
    except (OSError, KeyError, ValueError):
        return None


def low_head_run(args, da, torch, np, dev) -> dict:
    """The low-head workloads (configs 1 to 4): MQA decode (B=1, H_Q=8,
    H_KV=1, L_K=128), the Llama-3.1-70B GQA shape at B=1 (L_K = 128 ... 512),
    the pure-MQA low-tile sweep (B in {1,2,4} x L_K in {64..512}, H_Q=32,
    H_KV=1) and the varlen batched GQA batch.  Per shape: the heuristic's
    launch against two one-split baselines -- the paper's launch (one split,
    one workgroup per (sequence, KV head) with the whole group in it:
    pack_gqa = 2, no V slices) and one split as the planner makes it (its
    tile width and V slices) -- and a sweep of fixed split counts, each as
    the MI355X policy plans it.  Every launch is checked against the oracle
    before it is timed."""
    from workloads import algorithmic_bytes as ab, config_shapes, make_inputs
    res = {}
    K = max(args.steps, 100)
    for cid, sweep in ((1, (2, 4, 8)), (2, (2, 3, 4, 8, 16)), (3, SWEEP[1:]), (4, SWEEP[1:])):
        for sh in config_shapes(cid):
            inp = make_inputs(sh)
            q, k, v = dev(inp.q), dev(inp.k), dev(inp.v)
            cu = None if inp.cu_seqlens_k is None else torch.from_numpy(inp.cu_seqlens_k).cuda()
            L = sh.L_K
            log(f"timing {sh.name}")
            hv = Variant("heuristic", da, torch, q, k, v, L, 0, -1, K, cu=cu)
            s1_plan = Variant("s1_same_plan", da, torch, q, k, v, L, 1, -1, K, cu=cu)
            s1_paper = Variant("s1_paper_launch", da, torch, q, k, v, L, 1, 2, K, cu=cu)
            fixed = [Variant(f"s{s}", da, torch, q, k, v, L, s, 1, K, cu=cu) for s in sweep if s <= max(L, 1)]
            allv = [hv, s1_plan, s1_paper] + fixed
            validate(torch, OracleFull(np, inp), allv, sh.name)
            interleave(torch, allv, args.rounds)
            sw = {1: round(s1_plan.median, 3), **{x.plan.num_splits: round(x.median, 3) for x in fixed}}
            best = min(sw, key=sw.get)
            nbytes = ab(sh.B, sh.H_Q, sh.H_KV, int(inp.lengths.sum()), varlen=cu is not None)
            gbs = nbytes / (hv.median * 1e-6) / 1e9
            q25, q75 = np.percentile(hv.times, [25, 75])
            res[sh.name] = {"config": cid, "B": sh.B, "H_Q": sh.H_Q, "H_KV": sh.H_KV, "L_K": L,
                            "heuristic_us": round(hv.median, 3), "heuristic_iqr_us": [round(q25, 3), round(q75, 3)],
                            "plan": plan_brief(hv.plan),
                            "s1_paper_launch_us": round(s1_paper.median, 3),
                            "speedup_vs_s1_paper_launch": round(s1_paper.median / hv.median, 3),
                            "s1_same_plan_us": round(s1_plan.median, 3),
                            "speedup_vs_s1_same_plan": round(s1_plan.median / hv.median, 3),
                            "best_fixed": best, "best_fixed_us": sw[best],
                            "vs_best_fixed": round(hv.median / sw[best], 3),
                            "hbm_gbs": round(gbs, 1), "hbm_frac": round(gbs / HBM_PEAK_GBS, 5), "sweep_us": sw}
            del q, k, v, allv
    return res


def table_holds(which: str, B: int, H_Q: int, H_KV: int, L: int) -> bool:
    """Whether the generated split table ("warm" or "streamed") holds the shape."""
    from paper_2604_00028_amd import calibrate as cal
    if not hasattr(table_holds, "shapes"):
        t = cal.parse_table(open(cal.TABLE_SPLIT).read())
        table_holds.shapes = {w: {e[:4] for e in t[w]} for w in ("warm", "streamed")}
    return (B, H_Q, H_KV, L) in table_holds.shapes[which]


def launch_key(p) -> tuple:
    """What a plan launches: every field but pack_gqa, which only names the
    packing its tile width comes from."""
    return tuple(v for k, v in sorted(p.as_dict().items()) if k != "pack_gqa")


def plan_brief(p) -> str:
    """s, heads per tile, V slices, merge, (when not four) waves per
    workgroup and (when held to one) workgroups per CU of a plan, e.g.
    's4 h8 v4 fused', 's1 h8 v1 w2' or 's1 h8 v1 w2 1/cu'."""
    merge = "" if p.num_splits == 1 else (" fused" if p.combine else " 2-launch")
    waves = "" if p.group_waves == 4 else f" w{p.group_waves}"
    per_cu = " 1/cu" if getattr(p, "wg_per_cu", 0) == 1 else ""
    return f"s{p.num_splits} h{p.heads_per_tile} v{p.v_slices}{merge}{waves}{per_cu}"


class OracleFull:
    """The fp64 oracle over a whole problem given as host inputs (any
    layout), for launches that take the same inputs."""

    def __init__(self, np, inp):
        from oracle import decode_attention
        self.np = np
        self.O, _ = decode_attention(inp.q, inp.k, inp.v, inp.lengths, inp.cu_seqlens_k)

    def check(self, torch, out) -> tuple:
        np = self.np
        from oracle import bf16_bits_to_f64
        got = bf16_bits_to_f64(out.view(torch.int16).cpu().numpy().view(np.uint16))
        if not np.all(np.isfinite(got)):
            return False, float("inf"), float("inf")
        d = np.abs(got - self.O)
        return bool(d.max() <= 2e-2 and d.mean() <= 2e-3), float(d.max()), float(d.mean())


STREAMED_SHAPES = ((1, 64, 8, 128), (1, 64, 8, 256), (1, 64, 8, 384), (1, 64, 8, 512), (1, 64, 8, 1024),
                   (1, 64, 8, 2048), (4, 64, 8, 512), (8, 64, 8, 1024), (1, 8, 1, 128), (1, 8, 1, 512),
                   (1, 32, 1, 512), (4, 32, 1, 512), (16, 32, 4, 512))
STREAMED_SWEEP = (1, 2, 3, 4, 6, 8, 12, 16)


def streamed_run(args, da, torch) -> dict:
    """K/V streamed from HBM: every call of a timed replay reads its own copy
    of the cache (>= 1 GiB per replay, more than L2 + MALL hold), as each
    layer's cache is evicted by the rest of a decode step.  num_splits = 1,
    the warm-calibrated policy, the streamed policy, the streamed split
    table's plan and fixed splits."""
    res = {}
    for B, H_Q, H_KV, L in STREAMED_SHAPES:
        kvb = 2 * B * L * H_KV * 256
        copies = max(1, min(4096, -(-(1 << 30) // kvb)))
        gen = torch.Generator(device="cuda").manual_seed(17)
        q = torch.randn(B, H_Q, 128, device="cuda", generator=gen).to(torch.bfloat16)
        K = torch.empty(copies, B, L, H_KV, 128, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        V = torch.empty_like(K).normal_(generator=gen)
        kvs = [(K[i], V[i]) for i in range(copies)]
        steps = max(copies, 20)
        warm = da.da_choose_splits(B, H_Q, H_KV, L)
        cold = da.da_choose_splits(B, H_Q, H_KV, L, policy=da.POLICY_STREAMED)
        splits = sorted(set(STREAMED_SWEEP) | {warm.num_splits, cold.num_splits})
        log(f"timing streamed B={B} H_Q={H_Q} H_KV={H_KV} L_K={L} ({copies} copies)")
        # every launch as the streamed policy plans it for that split count (tile width, cache hint),
        # through the planned entry point; the warm policy's own plan beside them
        plans = {s: da.da_make_plan(B, H_Q, H_KV, L, 128, s, -1, policy=da.POLICY_STREAMED) for s in splits}
        var = {s: Variant(str(s), da, torch, q, K[0], V[0], L, s, 1, steps, kv_copies=kvs, plan=plans[s])
               for s in splits}
        wv = Variant("warm", da, torch, q, K[0], V[0], L, 0, -1, steps, kv_copies=kvs, plan=warm)
        # the streamed split table's plan (the launch its sweep measured fastest on this shape, if it holds it)
        tab = da.da_choose_splits(B, H_Q, H_KV, L, policy=da.POLICY_TABLE_STREAMED)
        tv = Variant("table", da, torch, q, K[0], V[0], L, 0, -1, steps, kv_copies=kvs, plan=tab)
        import numpy as np
        validate(torch, OracleRows(np, torch, q, K[0], V[0], range(min(B, 2))), list(var.values()) + [wv, tv],
                 f"streamed B={B} H_Q={H_Q} H_KV={H_KV} L_K={L}")
        interleave(torch, list(var.values()) + [wv, tv], args.rounds)
        us = {s: round(v.median, 3) for s, v in var.items()}
        iqr = lambda v: [round(x, 3) for x in np.percentile(v.times, [25, 75])]
        best = min(us, key=us.get)
        res[f"b{B}_h{H_Q}_kv{H_KV}_l{L}"] = {
            "B": B, "H_Q": H_Q, "H_KV": H_KV, "L_K": L, "s1_us": us[1],
            "warm_policy": warm.num_splits, "warm_policy_us": round(wv.median, 3),
            "streamed_policy": cold.num_splits, "streamed_policy_us": us[cold.num_splits],
            "s1_iqr_us": iqr(var[1]), "streamed_policy_iqr_us": iqr(var[cold.num_splits]),
            "streamed_plan": plan_brief(var[cold.num_splits].plan),
            "streamed_nontemporal": cold.kv_nontemporal,
            "streamed_speedup_vs_s1": round(us[1] / us[cold.num_splits], 3),
            "streamed_speedup_vs_warm_policy": round(wv.median / us[cold.num_splits], 3),
            "best_fixed": best, "best_fixed_us": us[best],
            "streamed_vs_best": round(us[cold.num_splits] / us[best], 3),
            "table_plan": plan_brief(tab), "table_held": table_holds("streamed", B, H_Q, H_KV, L),
            "table_us": round(tv.median, 3),
            "table_vs_best": round(tv.median / us[best], 3), "sweep_us": us}
        del K, V, kvs, var, wv, tv
    return res


def ragged_run(args, da, torch, np) -> dict:
    """Per-sequence schedules against the uniform plan on batches of mixed
    lengths: the scheduled launch (metadata made on the host, copied once),
    the uniform plan made for the longest sequence, and fixed split counts."""
    from workloads import algorithmic_bytes as ab, ragged_batches
    res = {}
    for name, lens, H_Q, H_KV in ragged_batches():
        B, tot, L = len(lens), sum(lens), max(lens)
        gen = torch.Generator(device="cuda").manual_seed(7)
        q = torch.randn(B, H_Q, 128, device="cuda", generator=gen).to(torch.bfloat16)
        kv_bytes = 2 * tot * H_KV * 256
        copies = max(1, min(16, -(-(512 << 20) // kv_bytes)))   # keep the working set out of L2 and MALL
        kvs = [(torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16),
                torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16)) for _ in range(copies)]
        cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
        out = torch.empty(B, H_Q, 128, dtype=torch.bfloat16, device="cuda")
        steps = 10 if kv_bytes > (256 << 20) else 100
        sched, meta = da.da_make_schedule(lens, H_Q, H_KV, L)
        # host cost of the planner itself (C call, buffers prepared once)
        import ctypes
        c_lens = (ctypes.c_int32 * B)(*lens)
        c_meta = (ctypes.c_uint8 * sched.meta_bytes)()
        c_out = da.DaSchedule()
        t0 = time.perf_counter()
        for _ in range(50):
            da.load().da_make_schedule(c_lens, B, H_Q, H_KV, L, 128, -1, 0, 0, 0, c_meta, sched.meta_bytes,
                                       ctypes.byref(c_out))
        plan_us = (time.perf_counter() - t0) / 50 * 1e6
        meta_dev = meta.cuda()
        # zero-filled: the arrival counters of merges inside the split launch start at zero
        ws_s = torch.zeros(max(da.da_schedule_workspace_bytes(sched), 256), dtype=torch.uint8, device="cuda")
        ws_u = torch.zeros(da.da_workspace_bytes(B, H_Q, 128, 64), dtype=torch.uint8, device="cuda")
        plan = da.da_choose_splits(B, H_Q, H_KV, L)
        log(f"timing ragged batch {name}")
        sv = Timed(torch, lambda i: da.da_decode_attn_scheduled(q, *kvs[i % copies], sched, meta_dev, cu_seqlens_k=cu,
                                                                out=out, workspace=ws_s), steps, out, "scheduled")
        fixed = sorted({1, 2, 4, 8, 16, 32, plan.num_splits})
        uv = {s: Timed(torch, lambda i, s=s: da.da_decode_attn(q, *kvs[i % copies], cu, out=out, L_K_max=L,
                                                               num_splits=s, pack_gqa=plan.pack_gqa, workspace=ws_u),
                       steps, out, f"uniform s{s}") for s in fixed}
        longest = max(range(B), key=lambda b: lens[b])
        validate(torch, OracleVarlen(np, torch, q, kvs[0][0], kvs[0][1], lens, [0, longest]),
                 [sv] + list(uv.values()), f"ragged {name}")
        interleave(torch, [sv] + list(uv.values()), max(3, args.rounds // 2))
        u_us = {s: round(v.median, 2) for s, v in uv.items()}
        best = min(u_us, key=u_us.get)
        nbytes = ab(B, H_Q, H_KV, tot, varlen=True)
        gbs = nbytes / (sv.median * 1e-6) / 1e9
        res[name] = {"B": B, "H_Q": H_Q, "H_KV": H_KV, "keys": tot, "L_K_max": L,
                     "scheduled_us": round(sv.median, 2), "chunk_tiles": sched.chunk_tiles,
                     "workgroups": sched.num_items, "max_splits": sched.max_splits, "kv_fetch": sched.kv_fetch,
                     "plan_host_us": round(plan_us, 1),
                     "uniform_plan_splits": plan.num_splits, "uniform_plan_us": u_us[plan.num_splits],
                     "speedup_vs_uniform_plan": round(u_us[plan.num_splits] / sv.median, 3),
                     "best_uniform_splits": best, "best_uniform_us": u_us[best],
                     "vs_best_uniform": round(sv.median / u_us[best], 3), "uniform_us": u_us,
                     "hbm_gbs": round(gbs, 1), "hbm_frac": round(gbs / HBM_PEAK_GBS, 4)}
        del kvs, sv, uv
    return res


SCHED_GRID = (1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64)
PROFILE_SCHEDULE = os.path.join(ROOT, "profiles", "schedule_mixed_length_batches.md")


def schedule_sweep_run(args, da, torch, np) -> None:
    """For every mixed-length batch of the fit and check sets: the modelled
    schedule, schedules at the chunk lengths that cut the longest sequence
    into 1..64 pieces, and the uniform launch at every split count."""
    from workloads import schedule_batches
    rows = []
    for kind in ("fit", "check"):
        for name, lens, H_Q, H_KV in schedule_batches(kind):
            B, tot, L = len(lens), sum(lens), max(lens)
            gen = torch.Generator(device="cuda").manual_seed(11)
            kv_bytes = 2 * tot * H_KV * 256
            copies = max(1, min(16, -(-(512 << 20) // kv_bytes)))
            q = torch.randn(B, H_Q, 128, device="cuda", generator=gen).to(torch.bfloat16)
            kvs = [(torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16),
                    torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16))
                   for _ in range(copies)]
            cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
            out = torch.empty(B, H_Q, 128, dtype=torch.bfloat16, device="cuda")
            steps = 10 if kv_bytes > (256 << 20) else (40 if kv_bytes > (32 << 20) else 200)
            ws = torch.zeros(da.da_workspace_bytes(B, H_Q, 128, 64) + 4096, dtype=torch.uint8, device="cuda")
            log(f"schedule sweep {kind}/{name}")
            plan = da.da_choose_splits(B, H_Q, H_KV, L)
            uni = {s: Timed(torch, lambda i, s=s: da.da_decode_attn(q, *kvs[i % copies], cu, out=out, L_K_max=L,
                                                                    num_splits=s, pack_gqa=plan.pack_gqa,
                                                                    workspace=ws), steps, out, f"uniform s{s}")
                   for s in sorted(set(SCHED_GRID) | {plan.num_splits})}
            t_max = -(-L // 32)
            chunks = sorted({-(-t_max // s) for s in SCHED_GRID}, reverse=True)
            scheds = {}   # (chunk, merge) -> (schedule, metadata, timed launch); chunk 0: as modelled
            for c in [0] + chunks:
                sc, meta = da.da_make_schedule(lens, H_Q, H_KV, L, chunk_tiles=c)
                md = meta.cuda()
                # either merge of the split sequences (the second launch, or inside the split launch
                # where the tiles have arrival counters); the modelled schedule as it comes
                combs = [sc.combine] if c == 0 or sc.state_rows == 0 else \
                    [0, 1] if sc.tiles <= MAX_ARRIVAL_TILES else [0]
                for k in combs:
                    sk = da.DaSchedule.from_buffer_copy(sc)
                    sk.combine = k
                    scheds[(c, k)] = (sk, md, Timed(torch, lambda i, sk=sk, md=md: da.da_decode_attn_scheduled(
                        q, *kvs[i % copies], sk, md, cu_seqlens_k=cu, out=out, workspace=ws), steps, out,
                        f"chunk {c} merge {k}"))
            auto = next(v for key, v in scheds.items() if key[0] == 0)
            longest = max(range(B), key=lambda b: lens[b])
            validate(torch, OracleVarlen(np, torch, q, kvs[0][0], kvs[0][1], lens, sorted({0, longest})),
                     list(uni.values()) + [x[2] for x in scheds.values()], f"schedule sweep {name}")
            interleave(torch, list(uni.values()) + [x[2] for x in scheds.values()], 5)
            rows.append({"set": kind, "batch": name, "B": B, "H_Q": H_Q, "H_KV": H_KV, "keys": tot, "L_K_max": L,
                         "uniform_plan_splits": plan.num_splits,
                         "uniform_us": {s: round(v.median, 3) for s, v in uni.items()},
                         "auto_chunk": auto[0].chunk_tiles, "auto_workgroups": auto[0].num_items,
                         "auto_us": round(auto[2].median, 3), "auto_hpt": auto[0].heads_per_tile,
                         "auto_combine": auto[0].combine,
                         "chunk_us_by_combine": {c: {k: round(v[2].median, 3) for (cc, k), v in scheds.items()
                                                     if cc == c} for c in chunks},
                         "chunk_hpt": {c: next(v[0].heads_per_tile for (cc, _), v in scheds.items() if cc == c)
                                       for c in chunks}})
            del kvs, uni, scheds
    with open(args.schedule_sweep, "w") as f:
        json.dump({"device_cus": da.da_device_info()[0], "kernel_source_sha256": kernel_source_sha(),
                   "validated": VALIDATION["validated"], "invalid": VALIDATION["invalid"], "rows": rows}, f)
    log(f"wrote {args.schedule_sweep}")


def schedule_sweep_summary(path: str) -> None:
    d = json.load(open(path))
    lines = ["# Per-sequence schedule on mixed-length batches (MI355X)", "",
             "Made by `python bench.py --schedule-sweep sched.json` then "
             "`python bench.py --schedule-sweep-summary sched.json`.", "",
             "Per batch: the modelled schedule (`auto`: its chunk length, in 32-key tiles, and the merge of its "
             "split sequences, `f` inside the split launch, `2` a second launch), the fastest of the schedules "
             "whose chunk cuts the longest sequence into 1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48 or 64 pieces, "
             "each with either merge (`grid best`), the "
             "uniform launch planned for the longest sequence (`uniform plan`) and the fastest uniform split "
             "count (`uniform best`).  Times in microseconds per call, HIP-graph replay, medians of 5 "
             "interleaved replays.  `fit`: the batches the schedule model was fitted to; `check`: drawn "
             "afterwards and never fitted.  `auto` is what the library made with the constants compiled in when "
             "the sweep ran (fitted to an earlier sweep of the same batches); calibration_summary.md evaluates the "
             "constants fitted to this sweep.", "",
             "| set | batch | B | H_Q/H_KV | keys | auto chunk | auto | grid best | auto/grid | uniform plan (s) "
             "| uniform best (s) | plan/auto | best/auto |",
             "|---|---|---|---|---|---|---|---|---|---|---|---|---|"]
    stats = {}
    for r in d["rows"]:
        gb = min(us for by in r["chunk_us_by_combine"].values() for us in by.values())
        uu = {int(k): v for k, v in r["uniform_us"].items()}
        ub = min(uu, key=uu.get)
        up = uu[r["uniform_plan_splits"]]
        a = r["auto_us"]
        stats.setdefault(r["set"], []).append((a / gb, up / a, uu[ub] / a))
        lines.append(f"| {r['set']} | {r['batch']} | {r['B']} | {r['H_Q']}/{r['H_KV']} | {r['keys']} | "
                     f"{r['auto_chunk']} {'f' if r.get('auto_combine') else '2'} | {a:.2f} | {gb:.2f} | {a / gb:.3f} | {up:.2f} ({r['uniform_plan_splits']}) "
                     f"| {uu[ub]:.2f} ({ub}) | {up / a:.2f} | {uu[ub] / a:.3f} |")
    lines.append("")
    for k, v in stats.items():
        g = [x[0] for x in v]
        p = [x[1] for x in v]
        b = [x[2] for x in v]
        lines.append(f"- {k}: auto/grid-best mean {sum(g) / len(g):.3f}, worst {max(g):.3f}; "
                     f"speedup over the uniform plan {min(p):.2f}x to {max(p):.2f}x; "
                     f"best uniform / auto {min(b):.3f} to {max(b):.3f}")
    with open(PROFILE_SCHEDULE, "w") as f:
        f.write("\n".join(lines) + "\n")
    print("\n".join(lines))


PROFILE_MIXED = os.path.join(ROOT, "profiles", "dealt_route_mixed_batches.md")
MIXED_BATCHES = (220, 2711)    # batches, seed
MIXED_LINES = ((60, 1.4), (60, 1.7), (80, 1.4), (80, 1.7), (80, 2.0), (100, 1.7), (150, 1.7))  # tiles, ratio


def mixed_sweep_run(args, da, torch, np) -> None:
    """For every batch of workloads.mixed_batches: the dealt launch and the
    launch with one split count, each with enough K/V copies in turn that none
    stays cached, and over one copy again and again."""
    from workloads import mixed_batches
    rows = []
    cus = da.da_device_info()[0]
    for n, (lens, H_Q, H_KV, page) in enumerate(mixed_batches(*MIXED_BATCHES)):
        B, tot, L = len(lens), sum(lens), max(lens)
        need = da.da_dealt_workspace_bytes(B, H_Q, H_KV)
        if not need:
            continue
        log(f"mixed sweep {n}: B={B} {H_Q}/{H_KV} page={page}")
        gen = torch.Generator(device="cuda").manual_seed(n)
        kv_bytes = tot * H_KV * 512
        copies = max(2, min(16, -(-(640 << 20) // kv_bytes)))
        new = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)  # noqa: E731
        q, out = new(B, H_Q, 128), torch.empty(B, H_Q, 128, dtype=torch.bfloat16, device="cuda")
        starts = np.concatenate([[0], np.cumsum(lens)])
        kvs = [(new(tot, H_KV, 128), new(tot, H_KV, 128)) for _ in range(copies)]
        orc = OracleVarlen(np, torch, q, *kvs[0], lens, sorted({0, lens.index(L)}))
        if page is None:
            cu, pool = torch.from_numpy(starts.astype(np.int32)).cuda(), tot
            own = lambda i, c, ws: da.da_decode_attn(q, *kvs[i % c], cu, out=out, L_K_max=L, workspace=ws)  # noqa: E731
            deal = lambda i, c, ws: da.da_decode_attn_dealt(q, *kvs[i % c], L, cu, out=out, workspace=ws)  # noqa: E731
        else:
            pages = [-(-x // page) for x in lens]
            order = torch.randperm(sum(pages), generator=torch.Generator().manual_seed(n))
            table, pool, at = torch.zeros(B, max(pages), dtype=torch.int32), sum(pages) * page, 0
            for b, m in enumerate(pages):
                table[b, :m] = order[at:at + m].to(torch.int32)
                at += m

            def paged(x):
                y = torch.zeros(pool, H_KV, 128, dtype=torch.bfloat16, device="cuda")
                for b, m in enumerate(pages):
                    key = torch.arange(lens[b])
                    y[(table[b].long()[key // page] * page + key % page).cuda()] = x[int(starts[b]):int(starts[b + 1])]
                return y.view(-1, page, H_KV, 128)

            kvs = [(paged(a), paged(b)) for a, b in kvs]
            bt, sl = table.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
            own = lambda i, c, ws: da.da_decode_attn_paged(q, *kvs[i % c], bt, sl, L, out=out, workspace=ws)  # noqa: E731
            deal = lambda i, c, ws: da.da_decode_attn_dealt(  # noqa: E731
                q, *kvs[i % c], L, block_table=bt, seq_lens=sl, out=out, workspace=ws)
        ws = torch.zeros(max(need, da.da_workspace_bytes(B, H_Q, 128, 64)), dtype=torch.uint8, device="cuda")
        steps = max(copies, 8 if kv_bytes > (256 << 20) else 24 if kv_bytes > (32 << 20) else 100)
        row = {"B": B, "H_Q": H_Q, "H_KV": H_KV, "page": page, "keys": tot, "longest": L, "mb": round(kv_bytes / 1e6)}
        for what, c in (("turn", copies), ("repeat", 1)):
            vs = [Timed(torch, lambda i, f=f: f(i, c, ws), steps, out, name) for name, f in (("one", own), ("dealt", deal))]
            validate(torch, orc, vs, f"mixed sweep {n}")
            interleave(torch, vs, 5)
            row[what] = [round(v.median, 2) for v in vs]
        heads = heads_per_tile(H_Q, H_KV, 32)
        groups, tiles = cus // (H_Q // heads), -(-L // 32)
        row["wide"] = heads > 16
        row["share"] = min(pool // 32 + B, B * tiles) / groups
        row["chunk"] = tiles / max(1, cus // (B * (H_Q // heads)))
        row["taken"] = bool(da.da_prefers_dealt(B, H_Q, H_KV, L, pool))
        rows.append(row)
        del kvs, vs
    with open(args.mixed_sweep, "w") as f:
        json.dump({"device_cus": cus, "kernel_source_sha256": kernel_source_sha(), "validated": VALIDATION["validated"],
                   "invalid": VALIDATION["invalid"], "rows": rows}, f)
    log(f"wrote {args.mixed_sweep}")


def mixed_sweep_summary(path: str) -> None:
    d = json.load(open(path))
    gain = lambda r, what: r[what][0] / r[what][1]  # noqa: E731
    least = lambda r: min(gain(r, "turn"), gain(r, "repeat"))  # noqa: E731
    mean = lambda v: math.exp(sum(map(math.log, v)) / len(v)) if v else 1.0  # noqa: E731
    lines = ["# Where the dealt launch pays (MI355X)", "",
             "Made by `python bench.py --mixed-sweep mixed.json` then `python bench.py --mixed-sweep-summary "
             f"mixed.json`: {len(d['rows'])} batches (`workloads.mixed_batches{MIXED_BATCHES}`), each output checked "
             f"against the oracle ({d['validated']} launches, {len(d['invalid'])} invalid).  Times are those of the "
             "launch with one split count over those of the dealt launch, HIP-graph replay, medians of 5: with "
             "640 MB of batches in turn, and one batch over and over.  `excess`: the longest chunk of one split "
             "count less the even share, in 32-key tiles; `ratio`: the one over the other.  A batch counts as "
             "slower below 0.985x in either.", "",
             "| batches with | taken | turn | repeat | slower | worst |", "|---|---|---|---|---|---|"]

    def line(name, rows):
        lines.append(f"| {name} | {len(rows)} | {mean([gain(r, 'turn') for r in rows]):.2f}x | "
                     f"{mean([gain(r, 'repeat') for r in rows]):.2f}x | {sum(least(r) < 0.985 for r in rows)} | "
                     f"{min(map(least, rows), default=1.0):.3f}x |")

    rows, taken = d["rows"], [r for r in d["rows"] if r["taken"]]
    line("the library's lines (`da_prefers_dealt`)", taken)
    line("all", rows)
    for wide in (False, True):
        for excess, ratio in MIXED_LINES + (((320, 1.7), (320, 3.0)) if wide else ()):
            line(f"{'wide' if wide else 'narrow'} head tiles, excess >= {excess}, ratio >= {ratio}",
                 [r for r in rows if r["wide"] == wide and r["chunk"] - r["share"] >= excess
                  and r["chunk"] >= ratio * r["share"]])
    lines += ["", "Every batch taken, slowest first:", "",
              "| B | heads | page | keys | longest | MB | share | excess | turn us | repeat us | turn | repeat |",
              "|---|---|---|---|---|---|---|---|---|---|---|---|"]
    for r in sorted(taken, key=least):
        lines.append(f"| {r['B']} | {r['H_Q']}/{r['H_KV']} | {r['page'] or '-'} | {r['keys']} | {r['longest']} | {r['mb']} "
                     f"| {r['share']:.0f} | {r['chunk'] - r['share']:.0f} | {r['turn'][0]} -> {r['turn'][1]} | "
                     f"{r['repeat'][0]} -> {r['repeat'][1]} | {gain(r, 'turn'):.2f}x | {gain(r, 'repeat'):.2f}x |")
    with open(PROFILE_MIXED, "w") as f:
        f.write("\n".join(lines) + "\n")
    print("\n".join(lines[:28]))


def cu_margin_run(args, da, torch, np) -> dict:
    """cu_margin with a concurrent kernel.  A quarter of the CUs (8 of every
    32 mask bits) is reserved for a bf16 GEMM on a CU-masked stream; the
    high-load decode runs on the rest, scheduled for the whole chip
    (cu_margin 0) or for the CUs it has (cu_margin = reserved).  Also: the
    same pair on two unmasked streams, and each kernel alone."""
    from paper_2604_00028_amd.streams import cu_mask_stream, destroy_stream, split_masks
    cus = da.da_device_info()[0]
    lens = [8192] * 32
    B, H_Q, H_KV, tot = 32, 64, 8, sum(lens)
    gen = torch.Generator(device="cuda").manual_seed(13)
    q = torch.randn(B, H_Q, 128, device="cuda", generator=gen).to(torch.bfloat16)
    k = torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16)
    v = torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    out = torch.empty(B, H_Q, 128, dtype=torch.bfloat16, device="cuda")
    A = torch.randn(8192, 8192, device="cuda", generator=gen).to(torch.bfloat16)
    Bm = torch.randn(8192, 8192, device="cuda", generator=gen).to(torch.bfloat16)
    plain_d, plain_g = torch.cuda.Stream(), torch.cuda.Stream()
    calls, gemms, rounds = 20, 8, max(3, args.rounds // 2)

    def decode_fn(margin):
        sched, meta = da.da_make_schedule(lens, H_Q, H_KV, 8192, cu_margin=margin)
        md = meta.cuda()
        ws = torch.zeros(max(da.da_schedule_workspace_bytes(sched), 256), dtype=torch.uint8, device="cuda")
        return sched, lambda s: da.da_decode_attn_scheduled(q, k, v, sched, md, cu_seqlens_k=cu, out=out,
                                                            workspace=ws, stream=s)

    def run(dstream, dfn, gstream):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        torch.cuda.synchronize()
        if gstream is not None:
            ev[2].record(gstream)
            with torch.cuda.stream(gstream):
                for _ in range(gemms):
                    torch.matmul(A, Bm)
            ev[3].record(gstream)
        if dfn is not None:
            ev[0].record(dstream)
            for _ in range(calls):
                dfn(dstream)
            ev[1].record(dstream)
        torch.cuda.synchronize()
        d = ev[0].elapsed_time(ev[1]) * 1000 / calls if dfn is not None else None
        g = ev[2].elapsed_time(ev[3]) * 1000 / gemms if gstream is not None else None
        return d, g

    gs = ds = None
    try:
        reserve_w, decode_w = split_masks(cus, 8)
        gs, n_res = cu_mask_stream(reserve_w)
        ds, n_dec = cu_mask_stream(decode_w)
        s0, f0 = decode_fn(0)
        sm, fm = decode_fn(n_res)
        cases = {"decode_alone_full_chip": (plain_d, f0, None),
                 "decode_alone_masked_plan_full_chip": (ds, f0, None),
                 "decode_alone_masked_plan_margin": (ds, fm, None),
                 "concurrent_masked_plan_full_chip": (ds, f0, gs),
                 "concurrent_masked_plan_margin": (ds, fm, gs),
                 "concurrent_unmasked_plan_full_chip": (plain_d, f0, plain_g),
                 "gemm_alone_full_chip": (None, None, plain_g),
                 "gemm_alone_reserved": (None, None, gs)}
        orc = OracleVarlen(np, torch, q, k, v, lens, [0, 31])
        for st, fn, gst in cases.values():   # warm every path once, checking each decode's output
            run(st, fn, gst)
            if fn is not None:
                ok, mx, mean = orc.check(torch, out)
                VALIDATION["validated"] += 1
                if not ok:
                    VALIDATION["invalid"].append({"what": "cu_margin", "launch": "scheduled decode",
                                                  "max_abs": mx, "mean_abs": mean})
        times = {name: [] for name in cases}
        for _ in range(rounds):
            for name, (st, fn, gst) in cases.items():
                times[name].append(run(st, fn, gst))
        res = {"workload": "highload_b32_h64_kv8_l8192 + bf16 GEMM 8192^3", "reserved_cus": n_res,
               "decode_cus": n_dec, "workgroups_plan_full_chip": s0.num_items,
               "workgroups_plan_margin": sm.num_items}
        for name, ts in times.items():
            d = [x[0] for x in ts if x[0] is not None]
            g = [x[1] for x in ts if x[1] is not None]
            res[name] = {"decode_us": round(statistics.median(d), 2) if d else None,
                         "gemm_us": round(statistics.median(g), 1) if g else None}
        res["margin_speedup_concurrent"] = round(res["concurrent_masked_plan_full_chip"]["decode_us"] /
                                                 res["concurrent_masked_plan_margin"]["decode_us"], 3)
        return res
    except Exception as e:  # the reservation is an optional part of the report
        return {"error": f"{type(e).__name__}: {e}"}
    finally:
        for s in (gs, ds):
            if s is not None:
                destroy_stream(s)


def host_cores():
    """(cores this process may run on, BLAS threads NumPy uses, CPU model)."""
    cores = len(os.sched_getaffinity(0))
    try:
        from threadpoolctl import threadpool_info
        blas = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        blas = None
    model = ""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return cores, blas, model


def copy_run(args, torch):
    """A plain device-to-device copy of 1 GiB (torch's copy kernel), steps
    times: bytes read and written per launch are known exactly."""
    n = 1 << 30
    src = torch.empty(n, dtype=torch.uint8, device="cuda")
    src.fill_(1)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    steps = max(1, args.highload_steps)
    a = torch.cuda.Event(enable_timing=True)
    b = torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(steps):
        dst.copy_(src)
    b.record()
    torch.cuda.synchronize()
    us = a.elapsed_time(b) * 1000.0 / steps
    print(json.dumps({"workload": "copy_1GiB", "bytes_read": n, "bytes_written": n, "launches": steps,
                      "us_per_copy": round(us, 2), "gbps": round(2 * n / (us * 1e-6) / 1e9, 1)}), flush=True)


# (workgroups, loads per thread) of the grid-stride probe, and of the one-region-per-wave probe
PROBE_GRID = ((256, 4), (256, 8), (256, 16), (512, 4), (512, 8), (1024, 4), (2048, 4), (4096, 4))
PROBE_WAVES = ((256, 8), (256, 16))


def read_probe_run(torch, steps: int = 20) -> dict:
    """The HBM read ceiling: a kernel that only reads 1 GiB with 16-byte
    loads (libhbm_probe.so, csrc/hbm_probe.hip), at 1-16 workgroups per CU
    and 4-16 loads per thread in flight, with and without the nontemporal
    hint; microseconds per launch from HIP events around `steps` launches on
    the current stream, after two warm-up launches.  The fastest
    configuration's rate is the practical ceiling the decode kernel's
    achieved bandwidth is set against."""
    import ctypes
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2604_00028_amd", "libhbm_probe.so"))
    for f in (lib.hbm_read_probe, lib.hbm_read_probe_waves):
        f.restype = ctypes.c_int
        f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                      ctypes.c_int, ctypes.c_void_p]
    n = 1 << 30
    src = torch.empty(n, dtype=torch.uint8, device="cuda")
    src.fill_(3)
    sink = torch.empty(max(w for w, _ in PROBE_GRID) * 256, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream()
    grid = {}
    # the grid-stride front at 1-16 workgroups per CU, and one region per wave at one workgroup per CU (the
    # decode kernel's pattern at high load), with and without the nontemporal hint
    configs = [(f"wg{w}x{u}", lib.hbm_read_probe, w, u) for w, u in PROBE_GRID] + \
              [(f"waves{w}x{u}", lib.hbm_read_probe_waves, w, u) for w, u in PROBE_WAVES]
    for tag, fn, wgs, loads in configs:
        for nt in (0, 1):
            def launch():
                rc = fn(src.data_ptr(), n, sink.data_ptr(), sink.numel() * 4, wgs, loads, nt, stream.cuda_stream)
                if rc != 0:
                    raise RuntimeError(f"read probe {tag} failed ({rc})")
            launch()
            launch()
            a = torch.cuda.Event(enable_timing=True)
            b = torch.cuda.Event(enable_timing=True)
            a.record(stream)
            for _ in range(steps):
                launch()
            b.record(stream)
            torch.cuda.synchronize()
            us = a.elapsed_time(b) * 1000.0 / steps
            grid[f"{tag}_{'nt' if nt else 'plain'}"] = round(n / (us * 1e-6) / 1e9, 1)
    best = max(grid, key=grid.get)
    del src, sink
    return {"bytes": n, "best_gbps": grid[best], "best": best, "frac_of_peak": round(grid[best] / HBM_PEAK_GBS, 4),
            "wave_regions_1wg_per_cu_gbps": max(grid["waves256x8_nt"], grid["waves256x16_nt"]), "gbps": grid}


def only_run(args, da, torch, np, dev):
    """Planned (or forced) launch of one workload, nothing else: the command
    the rocprofv3 summaries are taken from."""
    from workloads import config_shapes, custom_shape, make_inputs
    if args.only == "copy":
        copy_run(args, torch)
        return
    if args.only == "readprobe":
        print(json.dumps({"workload": "read_probe_1GiB", **read_probe_run(torch, max(1, args.highload_steps))}),
              flush=True)
        return
    if args.only == "ragged":
        ragged_only(args, da, torch, np)
        return
    if args.only == "long":
        sh = custom_shape(1, 64, 8, args.lk)
        inp = make_inputs(sh, seed=3000 + args.lk)
    elif args.only == "shape":
        B, H_Q, H_KV, L = (int(x) for x in args.shape.split(","))
        sh = custom_shape(B, H_Q, H_KV, L, name=f"b{B}_h{H_Q}_kv{H_KV}_l{L}")
        inp = make_inputs(sh, seed=5000 + B * 7 + L)
    else:
        sh = config_shapes(2)[3] if args.only == "headline" else config_shapes(5)[0]
        inp = make_inputs(sh)
    q, k, v = dev(inp.q), dev(inp.k), dev(inp.v)
    # the oracle on every row, or on two sampled sequences of a 1 GiB call
    oracle = OracleRows(np, torch, q, k, v, [0, sh.B - 1]) if args.only == "highload" else OracleFull(np, inp)
    del inp
    K = args.highload_steps if args.only == "highload" else args.steps
    plan = da.da_make_plan(sh.B, sh.H_Q, sh.H_KV, sh.L_K, 128, args.num_splits, args.pack_gqa)
    if args.combine >= 0:
        plan = with_combine(da, plan, args.combine)
    var = Variant(args.only, da, torch, q, k, v, sh.L_K, 0, -1, K, plan=plan)
    validate(torch, oracle, [var], sh.name)
    if VALIDATION["invalid"]:
        log(f"{sh.name}: the launch disagrees with the oracle")
        sys.exit(3)
    interleave(torch, [var], args.rounds)
    nbytes = algorithmic_bytes(sh.B, sh.H_Q, sh.H_KV, sh.L_K)
    gbs = nbytes / (var.median * 1e-6) / 1e9
    print(json.dumps({"workload": sh.name, "us_per_call": round(var.median, 3), "plan": plan_brief(var.plan),
                      "calls": K * (args.rounds + 1) + 3, "achieved_gbps": round(gbs, 1),
                      "frac": round(gbs / HBM_PEAK_GBS, 4)}), flush=True)


def ragged_only(args, da, torch, np):
    """The scheduled launch of the ragged high-load batch alone."""
    from workloads import algorithmic_bytes as ab, ragged_batches
    name, lens, H_Q, H_KV = ragged_batches()[0]
    B, tot, L = len(lens), sum(lens), max(lens)
    gen = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn(B, H_Q, 128, device="cuda", generator=gen).to(torch.bfloat16)
    k = torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16)
    v = torch.randn(tot, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    out = torch.empty(B, H_Q, 128, dtype=torch.bfloat16, device="cuda")
    sched, meta = da.da_make_schedule(lens, H_Q, H_KV, L)
    meta_dev = meta.cuda()
    ws = torch.zeros(max(da.da_schedule_workspace_bytes(sched), 256), dtype=torch.uint8, device="cuda")
    K = args.highload_steps
    var = Timed(torch, lambda i: da.da_decode_attn_scheduled(q, k, v, sched, meta_dev, cu_seqlens_k=cu, out=out,
                                                             workspace=ws), K, out, "scheduled")
    longest = max(range(B), key=lambda b: lens[b])
    validate(torch, OracleVarlen(np, torch, q, k, v, lens, [0, longest]), [var], name)
    if VALIDATION["invalid"]:
        log(f"{name}: the launch disagrees with the oracle")
        sys.exit(3)
    interleave(torch, [var], args.rounds)
    gbs = ab(B, H_Q, H_KV, tot, varlen=True) / (var.median * 1e-6) / 1e9
    print(json.dumps({"workload": name, "us_per_call": round(var.median, 3), "chunk_tiles": sched.chunk_tiles,
                      "workgroups": sched.num_items, "calls": K * (args.rounds + 1) + 3,
                      "achieved_gbps": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4)}), flush=True)


TRAFFIC_WORKLOADS = {"headline": "llama70b_gqa_b1_l512", "highload": "highload_b32_h64_kv8_l8192",
                     "ragged": "ragged_highload_b32_h64_kv8"}


def counter_avg(path: str, kernel_prefix: str, counter: str) -> float:
    """Mean per-dispatch value (KiB) of one counter for kernels whose name
    starts with kernel_prefix, from a rocprofv3 counter_collection.csv."""
    import csv
    vals = [float(r["Counter_Value"]) for r in csv.DictReader(open(path))
            if r["Kernel_Name"].startswith(kernel_prefix) and r["Counter_Name"] == counter]
    if not vals:
        raise ValueError(f"no {counter} rows for {kernel_prefix} in {path}")
    return sum(vals) / len(vals)


def traffic_summary(d: str) -> None:
    """Scale each counter by what it reads for a plain copy of known size
    (1 GiB read, 1 GiB written per launch), then write profiles/traffic.json."""
    f = lambda c, w: os.path.join(d, f"pmc_{c}_{w}", "run_counter_collection.csv")
    copy_kib = float(1 << 20)
    fetch_scale = copy_kib / counter_avg(f("FETCH_SIZE", "copy"), "__amd_rocclr_copyBuffer", "FETCH_SIZE")
    write_scale = copy_kib / counter_avg(f("WRITE_SIZE", "copy"), "__amd_rocclr_copyBuffer", "WRITE_SIZE")
    out = {"kernel_source_sha256": kernel_source_sha(),
           "fetch_scale": round(fetch_scale, 4), "write_scale": round(write_scale, 4),
           "command": "rocprofv3 --pmc <FETCH_SIZE|WRITE_SIZE> --output-format csv -d DIR/pmc_<counter>_<w> -o run "
                      "-- python3 bench.py --only <w> --steps 20 --rounds 1 --highload-steps 3",
           "workloads": {}}
    for w, name in TRAFFIC_WORKLOADS.items():
        fk = counter_avg(f("FETCH_SIZE", w), "void (anonymous namespace)::split_partial_kernel", "FETCH_SIZE")
        wk = counter_avg(f("WRITE_SIZE", w), "void (anonymous namespace)::split_partial_kernel", "WRITE_SIZE")
        out["workloads"][name] = {"fetch_kib_counter": round(fk, 2), "write_kib_counter": round(wk, 2),
                                  "fetch_bytes": int(fk * 1024 * fetch_scale), "write_bytes": int(wk * 1024 * write_scale)}
    with open(PROFILE_TRAFFIC, "w") as fh:
        json.dump(out, fh, indent=1)
        fh.write("\n")
    print(json.dumps(out))


OCC_CASES = (  # (case, --only workload, extra flags, label); s = 1 as the paper launches it
    ("headline_heur", "headline", "", "Llama-70B GQA B=1 L_K=512, heuristic (s=1, 4 V slices)"),
    ("headline_s1", "headline", "--num-splits 1 --pack-gqa 2",
     "Llama-70B GQA B=1 L_K=512, num_splits=1, one workgroup per KV head"),
    ("long2048_heur", "long", "--lk 2048", "Llama-70B GQA B=1 L_K=2048, heuristic"),
    ("long2048_s1", "long", "--lk 2048 --num-splits 1 --pack-gqa 2",
     "Llama-70B GQA B=1 L_K=2048, num_splits=1, one workgroup per KV head"),
    ("long8192_heur", "long", "--lk 8192", "Llama-70B GQA B=1 L_K=8192, heuristic"),
    ("long8192_s1", "long", "--lk 8192 --num-splits 1 --pack-gqa 2",
     "Llama-70B GQA B=1 L_K=8192, num_splits=1, one workgroup per KV head"),
    ("highload_heur", "highload", "", "high load B=32 L_K=8192, heuristic"),
    ("highload_s4", "highload", "--num-splits 4", "high load B=32 L_K=8192, num_splits=4"),
)
OCC_PASSES = {"raw": "GRBM_GUI_ACTIVE SQ_BUSY_CU_CYCLES SQ_WAVE_CYCLES SQ_WAVES",
              "occ": "MeanOccupancyPerActiveCU"}
PROFILE_OCCUPANCY = os.path.join(ROOT, "profiles", "occupancy_heuristic_vs_s1.md")


def occupancy_summary(d: str) -> None:
    """Per case, the split kernel's dispatches: duration, GPU-active cycles,
    busy CUs, mean occupancy of the busy CUs and occupancy in percent of 32
    waves per CU."""
    import csv
    kp = "void (anonymous namespace)::split_partial_kernel"
    lines = ["# Active CUs and occupancy: heuristic vs num_splits = 1 (MI355X, rocprofv3 counters)", "",
             "Commands (MI355X, one GPU), for each case and pass:", "", "```",
             "cd /tmp && export TMPDIR=/tmp && cd $REPO",
             "rocprofv3 --pmc GRBM_GUI_ACTIVE SQ_BUSY_CU_CYCLES SQ_WAVE_CYCLES SQ_WAVES --kernel-trace --stats \\",
             "    --output-format csv -d $OUT/occ_raw_<case> -o run -- \\",
             "    python3 bench.py --only <workload> <flags> --steps 20 --rounds 1 --highload-steps 3",
             "rocprofv3 --pmc MeanOccupancyPerActiveCU --output-format csv -d $OUT/occ_occ_<case> -o run -- \\",
             "    python3 bench.py --only <workload> <flags> --steps 20 --rounds 1 --highload-steps 3",
             "python3 bench.py --occupancy-summary $OUT   # writes this file", "```", "",
             "Per split-kernel dispatch, mean over the dispatches of the run. GRBM_GUI_ACTIVE comes summed over the "
             "8 XCDs and is divided by 8. Busy CUs = SQ_BUSY_CU_CYCLES / GPU-active cycles (the profiler's "
             "SIMD_UTILIZATION without the division by the CU count); over the kernel's own duration = "
             "SQ_BUSY_CU_CYCLES / (duration x clock), the clock taken as GPU-active cycles / duration of the "
             "longest case. For kernels of a few microseconds the GPU-active window also spans the dispatch, "
             "so the first figure reads low. MeanOccupancyPerActiveCU is the profiler's derived metric. "
             "Occupancy = 4 x SQ_WAVE_CYCLES / (GPU-active cycles x 256 CUs x 32 waves), the profiler's "
             "OccupancyPercent. The busy count follows the SIMDs of a CU that hold a wave: the high-load "
             "heuristic runs one workgroup of two waves per CU (every CU busy, two of its four SIMDs), so it "
             "reads about half the CUs. Kernel times under counter collection vary from box to box for the "
             "short launches (the L_K=8192 heuristic case took 8.8 us in an earlier take on another box); the "
             "benchmark's graph-replay times are the reference.", "",
             "| case | workgroups | waves | kernel us | GPU-active cycles | busy CUs (GPU-active) | busy CUs "
             "(kernel time) | MeanOccupancyPerActiveCU | occupancy |",
             "|---|---|---|---|---|---|---|---|---|"]

    def read(case, pas):
        path = os.path.join(d, f"occ_{pas}_{case}")
        rows = list(csv.DictReader(open(os.path.join(path, "run_counter_collection.csv"))))
        by, grid = {}, None
        for r in rows:
            if not r["Kernel_Name"].startswith(kp):
                continue
            by.setdefault(r["Counter_Name"], []).append(float(r["Counter_Value"]))
            if grid is None and r.get("Grid_Size") and r.get("Workgroup_Size"):
                grid = int(float(r["Grid_Size"])) // int(float(r["Workgroup_Size"]))
        dur = None
        stats = os.path.join(path, "run_kernel_stats.csv")
        if os.path.exists(stats):
            for r in csv.DictReader(open(stats)):
                if r["Name"].startswith(kp):
                    dur = float(r["AverageNs"]) / 1000.0
        return {k: sum(v) / len(v) for k, v in by.items()}, grid, dur

    got = []
    for case, _, _, label in OCC_CASES:
        try:
            raw, grid, dur = read(case, "raw")
            occ, _, _ = read(case, "occ")
        except FileNotFoundError:
            continue
        got.append((label, raw, occ, grid, dur))
    longest = max(got, key=lambda x: x[4] or 0.0)
    clock = (longest[1]["GRBM_GUI_ACTIVE"] / 8.0) / longest[4]   # cycles per microsecond
    for label, raw, occ, grid, dur in got:
        active = raw["GRBM_GUI_ACTIVE"] / 8.0
        busy = raw["SQ_BUSY_CU_CYCLES"]
        occp = 100.0 * 4.0 * raw["SQ_WAVE_CYCLES"] / (active * 256 * 32)
        lines.append(f"| {label} | {grid} | {raw['SQ_WAVES']:.0f} | {dur:.2f} | {active:,.0f} | {busy / active:.1f} | "
                     f"{busy / (dur * clock):.1f} | {occ.get('MeanOccupancyPerActiveCU', float('nan')):.2f} | "
                     f"{occp:.2f}% |")
    lines += ["", f"Clock estimate: {clock:,.0f} cycles per microsecond."]
    with open(PROFILE_OCCUPANCY, "w") as f:
        f.write("\n".join(lines) + "\n")
    print("\n".join(lines))


def regression_run(args, da, torch) -> None:
    """Every configuration of the matrix (the paper's Batch x L_K x H_KV
    sweep, Section 5.3, plus the L_K = 576/640/768 boundary of Section 4.1):
    the MI355X heuristic, one split launched as the paper launches it (the
    whole group in one workgroup, no V slices), one split as the planner
    makes it, the paper's and the evolved policy's own plans, and fixed
    split counts, each checked against the oracle (sampled sequences) and
    then timed as graph-replayed calls interleaved over rounds (median and
    IQR per launch, no pooling of equal launches)."""
    import numpy as np
    results = []
    gen = torch.Generator(device="cuda")
    for B in REG_B:
        for H_KV in REG_HKV:
            H_Q = 8 * H_KV
            for L in REG_L:
                gen.manual_seed(B * 100000 + H_KV * 10000 + L)
                q = torch.randn((B, H_Q, 128), generator=gen, device="cuda").to(torch.bfloat16)
                k = torch.randn((B, L, H_KV, 128), generator=gen, device="cuda").to(torch.bfloat16)
                v = torch.randn((B, L, H_KV, 128), generator=gen, device="cuda").to(torch.bfloat16)
                est_us = 5.0 + 2.0 * B * L * H_KV * 256 / 5e6
                K = int(max(10, min(100, 2000.0 / est_us)))
                paper = da.da_choose_splits(B, H_Q, H_KV, L, policy=da.POLICY_PAPER)
                evolved = da.da_choose_splits(B, H_Q, H_KV, L, policy=da.POLICY_EVOLVED)
                heur = da.da_choose_splits(B, H_Q, H_KV, L)
                table = da.da_choose_splits(B, H_Q, H_KV, L, policy=da.POLICY_TABLE)
                splits = sorted({s for s in REG_SWEEP if s == 1 or s * 8 <= L})
                variants = {s: Variant(f"s{s}", da, torch, q, k, v, L, s, 1, K) for s in splits}
                own = {"heuristic": Variant("heuristic", da, torch, q, k, v, L, 0, -1, K, plan=heur),
                       "paper": Variant("paper", da, torch, q, k, v, L, 0, -1, K, plan=paper),
                       "evolved": Variant("evolved", da, torch, q, k, v, L, 0, -1, K, plan=evolved),
                       "table": Variant("table", da, torch, q, k, v, L, 0, -1, K, plan=table),
                       "s1_paper_launch": Variant("s1_paper_launch", da, torch, q, k, v, L, 1, 2, K),
                       # the same launch as s = 1 once more: how far apart two identical launches time
                       "s1_repeat": Variant("s1_repeat", da, torch, q, k, v, L, 0, -1, K, plan=variants[1].plan)}
                allv = list(variants.values()) + list(own.values())
                validate(torch, OracleRows(np, torch, q, k, v, [0] if B == 1 else [0, B - 1]), allv,
                         f"regression B={B} H_KV={H_KV} L_K={L}")
                for r in range(args.rounds):     # interleaved and rotated, no pooling: every launch keeps its times
                    for j in range(len(allv)):
                        allv[(r + j) % len(allv)].timed(torch)
                sw = {s: round(x.median, 3) for s, x in variants.items()}
                best = min(sw, key=sw.get)
                iqr = lambda x: [round(t, 3) for t in np.percentile(x.times, [25, 75])]
                row = {"B": B, "H_Q": H_Q, "H_KV": H_KV, "L_K": L,
                       "heuristic_plan": plan_brief(heur), "heuristic_splits": heur.num_splits,
                       "heuristic_us": round(own["heuristic"].median, 3), "heuristic_iqr": iqr(own["heuristic"]),
                       "s1_paper_launch_us": round(own["s1_paper_launch"].median, 3),
                       "s1_paper_launch_iqr": iqr(own["s1_paper_launch"]),
                       "s1_us": sw[1], "s1_iqr": iqr(variants[1]), "s1_repeat_us": round(own["s1_repeat"].median, 3),
                       "paper_splits": paper.num_splits, "paper_us": round(own["paper"].median, 3),
                       "evolved_splits": evolved.num_splits, "evolved_us": round(own["evolved"].median, 3),
                       "table_plan": plan_brief(table), "table_us": round(own["table"].median, 3),
                       "table_iqr": iqr(own["table"]),
                       "table_held": table_holds("warm", B, H_Q, H_KV, L),
                       # the heuristic's launch is the paper's one-split launch itself (pack_gqa only names it)
                       "same_launch_as_s1_paper": launch_key(heur) == launch_key(own["s1_paper_launch"].plan),
                       "best_fixed": best, "best_fixed_us": sw[best], "sweep_us": sw}
                results.append(row)
                log(f"B={B} H_KV={H_KV} L_K={L}: heuristic {row['heuristic_plan']} {row['heuristic_us']} us, "
                    f"s=1 paper launch {row['s1_paper_launch_us']}, best s={best} {sw[best]}")
                del q, k, v, variants, own, allv
    json.dump({"configs": results, "validated": VALIDATION["validated"], "invalid": VALIDATION["invalid"],
               "kernel_source_sha256": kernel_source_sha()}, open(args.regression, "w"), indent=1)
    worst_s1 = max(r["heuristic_us"] / r["s1_paper_launch_us"] for r in results)
    worst_best = max(r["heuristic_us"] / r["best_fixed_us"] for r in results)
    print(json.dumps({"regression_configs": len(results), "validated": VALIDATION["validated"],
                      "invalid": len(VALIDATION["invalid"]),
                      "worst_heuristic_over_s1_paper_launch": round(worst_s1, 3),
                      "worst_heuristic_over_best_fixed": round(worst_best, 3)}), flush=True)
    if VALIDATION["invalid"]:
        sys.exit(3)


def regression_summary(path: str) -> None:
    d = json.load(open(path))
    rows = d["configs"]
    n = len(rows)
    r_p1 = [r["heuristic_us"] / r["s1_paper_launch_us"] for r in rows]
    r_s1 = [r["heuristic_us"] / r["s1_us"] for r in rows]
    r_best = [r["heuristic_us"] / r["best_fixed_us"] for r in rows]
    r_paper = [r["heuristic_us"] / r["paper_us"] for r in rows]
    r_evo = [r["heuristic_us"] / r["evolved_us"] for r in rows if r["B"] == 1]
    # noise floor of the method: two timings of the same launch (s = 1 as planned, twice) per shape
    rep = [abs(r["s1_repeat_us"] / r["s1_us"] - 1) for r in rows if "s1_repeat_us" in r]
    floor = max(rep) if rep else 0.0
    # slower than one split beyond noise: under 0.99x its speed, the heuristic's interquartile range
    # above the one-split launch's, and further apart than two timings of one launch ever were
    beyond = lambda r, key: (r["heuristic_us"] > r[key + "_us"] / 0.99 and
                             r["heuristic_iqr"][0] > r[key + "_iqr"][1] and
                             r["heuristic_us"] > r[key + "_us"] * (1 + floor))
    slower_p1 = [r for r in rows if beyond(r, "s1_paper_launch")]
    slower_s1 = [r for r in rows if beyond(r, "s1")]
    under99_p1 = sum(x > 1 / 0.99 for x in r_p1)
    same_p1 = [r for r in rows if r.get("same_launch_as_s1_paper")]
    under99_same = sum(r["heuristic_us"] / r["s1_paper_launch_us"] > 1 / 0.99 for r in same_p1)
    over5 = sum(x > 1.05 for x in r_best)
    bnd = [r for r in rows if r["L_K"] in (576, 640, 768)]
    held = [r for r in rows if r.get("table_held")]
    table_lines = []
    if held:
        t_h = [r["table_us"] / r["heuristic_us"] for r in held]
        t_b = [r["table_us"] / min(r["best_fixed_us"], r["heuristic_us"]) for r in held]
        h_b = [r["heuristic_us"] / min(r["best_fixed_us"], r["table_us"]) for r in held]
        diff = [r for r in held if r["table_plan"] != r["heuristic_plan"]]
        table_lines = [
            f"* Policy TABLE (the configuration-specific split table, learned from the calibration sweep, which "
            f"was timed in another run) on the {len(held)} shapes it holds: a plan other than the heuristic's in {len(diff)}; "
            f"its time over the heuristic's mean {statistics.mean(t_h):.3f}x, best {min(t_h):.3f}x, worst "
            f"{max(t_h):.3f}x; over the faster of the heuristic and the best fixed split: within 5% in "
            f"{sum(x <= 1.05 for x in t_b)} of {len(held)}, worst {max(t_b):.3f}x (the heuristic over the faster of "
            f"the table and the best fixed split: within 5% in {sum(x <= 1.05 for x in h_b)}, worst "
            f"{max(h_b):.3f}x). Every other shape the table plans as the heuristic does."]
    lines = [
        f"# Regression matrix: {n} decode shapes (the paper's Section 5.3 sweep and its L_K >= 640 boundary) "
        "on MI355X",
        "",
        "Batch in {1, 2, 4, 8} x L_K in {128, 256, 384, 512, 576, 640, 768, 1024, 2048, 4096, 8192} x H_KV in",
        "{1, 2, 4, 8, 32}, H_Q = 8 * H_KV, D = 128, bf16, synthetic inputs. Each shape times, as graph-replayed",
        "calls interleaved over rounds (median; each launch keeps its own times, equal launches are not pooled):",
        "the MI355X heuristic; one split launched as the paper launches it (`pack_gqa = 2`: one workgroup per",
        "KV head with the whole group, no V slices); one split as the planner makes it (its tile width and V",
        "slices); the paper's policy (policy PAPER); the evolved single-batch setting of its Fig. 1 (policy",
        "EVOLVED); the configuration-specific split table (policy TABLE); and fixed splits s in",
        "{1, 2, 3, 4, 6, 8, 12, 16, 24, 32} (s <= L_K / 8) as the library plans them. Every launch was checked",
        "against the fp64 oracle (sampled sequences) before it was timed:",
        f"{d.get('validated', 0)} launches, {len(d.get('invalid', []))} invalid.",
        "",
        "Command (MI355X, one GPU):",
        "",
        "```",
        "python3 bench.py --regression $OUT/regression.json --rounds 5",
        "python3 bench.py --regression-summary $OUT/regression.json   # writes this file",
        "```",
        "",
        f"* Shapes: {n}.",
        (f"* Noise floor: two timings of the same launch (one split as planned, timed twice in the same run) "
         f"differ by {statistics.mean(rep) * 100:.1f}% on average and by up to {floor * 100:.1f}%; the "
         f"interquartile ranges understate this, so 'beyond noise' below also requires a gap larger than "
         f"{floor * 100:.1f}%.") if rep else "",
        f"* Heuristic vs one split as the paper launches it: at least 0.99x its speed in {n - under99_p1} of {n} "
        f"shapes (worst {max(r_p1):.3f}x its time); slower beyond noise in {len(slower_p1)}; "
        f"faster by more than 1% in {sum(x < 0.99 for x in r_p1)}; mean {statistics.mean(r_p1):.3f}x its time, "
        f"best {min(r_p1):.3f}x." + (
            f" In {len(same_p1)} shapes the heuristic's launch is the paper's launch itself (the same kernel, grid "
            f"and cache hint; only the name of the packing differs), so their gap is the noise of timing one launch "
            f"twice; {under99_same} of the shapes under 0.99x are among them." if "same_launch_as_s1_paper" in rows[0]
            else ""),
        f"* Heuristic vs one split as the planner makes it: worst {max(r_s1):.3f}x its time; slower beyond noise in "
        f"{len(slower_s1)}; faster by more than 1% in {sum(x < 0.99 for x in r_s1)}.",
        f"* Heuristic vs the best fixed split: within 5% in {n - over5} of {n}; worst {max(r_best):.3f}x, "
        f"mean {statistics.mean(r_best):.3f}x.",
        f"* Heuristic vs the paper's policy: mean {statistics.mean(r_paper):.3f}x its time, "
        f"best {min(r_paper):.3f}x, worst {max(r_paper):.3f}x.",
        f"* Heuristic vs the evolved single-batch setting (Fig. 1; batch 1 only, {len(r_evo)} shapes): mean "
        f"{statistics.mean(r_evo):.3f}x its time, best {min(r_evo):.3f}x, worst {max(r_evo):.3f}x.",
        f"* The L_K = 576, 640, 768 boundary ({len(bnd)} shapes): heuristic vs the paper's one-split launch "
        f"{min(r['heuristic_us'] / r['s1_paper_launch_us'] for r in bnd):.3f}x to "
        f"{max(r['heuristic_us'] / r['s1_paper_launch_us'] for r in bnd):.3f}x its time; vs the paper's policy "
        f"{min(r['heuristic_us'] / r['paper_us'] for r in bnd):.3f}x to "
        f"{max(r['heuristic_us'] / r['paper_us'] for r in bnd):.3f}x." if bnd else "",
        *table_lines,
        "",
        "IQR columns: 25th-75th percentile of the per-replay microseconds.",
        "",
        "| B | H_KV | L_K | heuristic plan | us (IQR) | s = 1 paper launch us (IQR) | vs it | s = 1 planned us | "
        "paper s | paper us | evolved s | evolved us | table plan | table us | best s | best us | vs best |",
        "|---|---|---|---|---|---|---|---|---|---|---|---|---|---|---|---|---|",
    ]
    for r, a, c in zip(rows, r_p1, r_best):
        hi, pi = r["heuristic_iqr"], r["s1_paper_launch_iqr"]
        tp = (r["table_plan"] + (" (held)" if r["table_held"] else "")) if "table_plan" in r else ""
        lines.append(f"| {r['B']} | {r['H_KV']} | {r['L_K']} | {r['heuristic_plan']} | {r['heuristic_us']} "
                     f"({hi[0]}-{hi[1]}) | {r['s1_paper_launch_us']} ({pi[0]}-{pi[1]}) | {1 / a:.2f}x | "
                     f"{r['s1_us']} | {r['paper_splits']} | {r['paper_us']} | {r['evolved_splits']} | "
                     f"{r['evolved_us']} | {tp} | {r.get('table_us', '')} | {r['best_fixed']} | "
                     f"{r['best_fixed_us']} | {c:.3f} |")
    open(PROFILE_REGRESSION, "w").write("\n".join(lines) + "\n")
    print(f"wrote {PROFILE_REGRESSION}")


# ---------------------------------------------------------------- two waves against four

PROFILE_WAVES = os.path.join(ROOT, "profiles", "two_waves_vs_four_waves.md")
# (B, H_Q, H_KV, L_K), all planned unsplit with one V slice and one workgroup reading each key: 192-256
# workgroups (one per CU), 264-320 (the two-wave rule's upper range), 384-576 with 2-8 KV heads (past it,
# four waves, or two held to one workgroup per CU over 2-4 full rounds of chunks of >= 2048 keys) and pure
# MQA at 384-1152 (two waves up to 768 over chunks of >= 1024 keys and up to 1024 over >= 2048, four over 512
# and past 1024)
WAVES_SHAPES = ((24, 64, 8, 8192), (28, 64, 8, 2048), (32, 64, 8, 8192), (256, 8, 1, 4096),
                (33, 64, 8, 1024), (36, 64, 8, 1024), (40, 64, 8, 512), (39, 64, 8, 2048), (40, 64, 8, 2048),
                (300, 8, 1, 512), (300, 8, 1, 1024), (300, 16, 1, 2048), (80, 32, 4, 2048), (80, 64, 4, 1024),
                (17, 128, 16, 512), (20, 128, 16, 1024),
                (48, 64, 8, 1024), (56, 64, 8, 1024), (64, 64, 8, 1024), (72, 64, 8, 1024), (192, 16, 2, 1024),
                (96, 32, 4, 4096),
                (384, 8, 1, 1024), (448, 8, 1, 1024), (512, 16, 1, 4096), (640, 8, 1, 1024), (768, 32, 1, 2048),
                (640, 8, 1, 512), (60, 64, 8, 2048), (64, 64, 8, 4096), (96, 64, 8, 2048), (128, 32, 4, 8192),
                (128, 64, 8, 4096), (128, 64, 8, 2048), (1024, 16, 1, 2048), (1152, 8, 1, 4096))


def wave_forms(da, plan, H_KV):
    """(two-wave, four-wave) forms of a one-split plan, one of them the plan
    itself: four waves fetch straight into LDS with one workgroup per CU and
    through registers into LDS where CUs hold more (chunks of >= 512 keys);
    two waves fetch through registers, K straight into the operand layout
    where key rows hold one KV head and each CU holds one workgroup.  The
    form that is not the plan lets CUs hold several workgroups at once."""
    other = da.DaPlan.from_buffer_copy(plan)
    other.wg_per_cu = 0  # the other form lets CUs hold several workgroups
    lone = plan.grid <= plan.num_cus
    if plan.group_waves == 2:
        other.group_waves, other.kv_fetch = 4, 2 if lone else 1
        return plan, other
    other.group_waves, other.combine = 2, 0
    other.kv_fetch = 0 if H_KV == 1 and lone else 1
    return other, plan


def waves_sweep_run(args, da, torch, np) -> None:
    """Each shape of WAVES_SHAPES launched with two and with four waves per
    workgroup (the planner's plan and its other wave count, same split,
    tile and merge), each output checked against the oracle on the first
    and last sequence, then timed as graph-replayed calls interleaved over
    rounds."""
    rows = []
    gen = torch.Generator(device="cuda")
    for B, H_Q, H_KV, L in WAVES_SHAPES:
        gen.manual_seed(B * 100000 + H_KV * 10000 + L)
        q = torch.randn((B, H_Q, 128), generator=gen, device="cuda").to(torch.bfloat16)
        k = torch.randn((B, L, H_KV, 128), generator=gen, device="cuda").to(torch.bfloat16)
        v = torch.randn((B, L, H_KV, 128), generator=gen, device="cuda").to(torch.bfloat16)
        plan = da.da_choose_splits(B, H_Q, H_KV, L)
        if plan.num_splits != 1 or plan.v_slices != 1 or plan.heads_per_tile != H_Q // H_KV:
            log(f"waves sweep: B={B} H_Q={H_Q} H_KV={H_KV} L_K={L} planned {plan_brief(plan)}; skipped")
            continue
        two, four = wave_forms(da, plan, H_KV)
        est_us = 5.0 + 2.0 * B * L * H_KV * 256 / 5e6
        K = int(max(10, min(100, 2000.0 / est_us)))
        vs = [Variant("two", da, torch, q, k, v, L, 0, -1, K, plan=two),
              Variant("four", da, torch, q, k, v, L, 0, -1, K, plan=four)]
        validate(torch, OracleRows(np, torch, q, k, v, [0, B - 1]), vs, f"waves B={B} H_Q={H_Q} H_KV={H_KV} L_K={L}")
        interleave(torch, vs, args.rounds)
        iqr = lambda x: [round(t, 3) for t in np.percentile(x.times, [25, 75])]
        row = {"B": B, "H_Q": H_Q, "H_KV": H_KV, "L_K": L, "grid": plan.grid, "cus": plan.num_cus,
               "planned_waves": plan.group_waves, "two_fetch": two.kv_fetch, "four_fetch": four.kv_fetch,
               "two_per_cu": two.wg_per_cu,
               "two_us": round(vs[0].median, 3), "two_iqr": iqr(vs[0]),
               "four_us": round(vs[1].median, 3), "four_iqr": iqr(vs[1]),
               "two_over_four": round(vs[0].median / vs[1].median, 4)}
        rows.append(row)
        log(f"waves B={B} H_Q={H_Q} H_KV={H_KV} L_K={L} grid {plan.grid}: two {row['two_us']} four "
            f"{row['four_us']} ({row['two_over_four']})")
        del q, k, v, vs
        torch.cuda.empty_cache()
    json.dump({"rows": rows, "validated": VALIDATION["validated"], "invalid": VALIDATION["invalid"],
               "kernel_source_sha256": kernel_source_sha(), "rounds": args.rounds},
              open(args.waves_sweep, "w"), indent=1)
    print(json.dumps({"waves_shapes": len(rows), "validated": VALIDATION["validated"],
                      "invalid": len(VALIDATION["invalid"])}), flush=True)
    if VALIDATION["invalid"]:
        sys.exit(3)


def waves_sweep_summary(path: str) -> None:
    d = json.load(open(path))
    rows = d["rows"]
    fetch = {0: "operand layout", 1: "registers to LDS", 2: "direct to LDS"}
    lines = ["# Two waves per workgroup against four, one-split launches of 192-1024 workgroups", "",
             "Each shape launched with the planner's wave count and with the other one (same split, tile and merge; "
             "the fetch path each wave count takes there), every output checked against the oracle on the first "
             f"and last sequence ({d['validated']} launches validated, {len(d['invalid'])} invalid), then timed as "
             f"graph-replayed calls interleaved over {d['rounds']} rounds: median us per call (IQR).", "",
             "Command (MI355X, one GPU):", "", "```",
             "cd $REPO && python3 bench.py --waves-sweep $OUT/waves.json --rounds %d" % d["rounds"],
             "python3 bench.py --waves-sweep-summary $OUT/waves.json", "```", "",
             "| B | H_Q | H_KV | L_K | workgroups / CUs | planned | two waves us (fetch) | four waves us (fetch) | "
             "two / four |", "|---|---|---|---|---|---|---|---|---|"]
    for r in rows:
        ti, fi = r["two_iqr"], r["four_iqr"]
        held = ", one workgroup per CU" if r.get("two_per_cu") else ""
        lines.append(f"| {r['B']} | {r['H_Q']} | {r['H_KV']} | {r['L_K']} | {r['grid']} / {r['cus']} | "
                     f"{r['planned_waves']} | {r['two_us']} ({ti[0]}-{ti[1]}, {fetch[r['two_fetch']]}{held}) | "
                     f"{r['four_us']} ({fi[0]}-{fi[1]}, {fetch[r['four_fetch']]}) | {r['two_over_four']:.3f} |")
    lines += [""]
    for name, lo, hi, mqa in (("up to one workgroup per CU", 0, 1.0, None),
                              ("up to 5/4 (the two-wave rule)", 1.0, 1.25, None),
                              ("past 5/4, 2-16 KV heads", 1.25, 99, False), ("past 5/4, pure MQA", 1.25, 99, True)):
        x = [r["two_over_four"] for r in rows if lo < r["grid"] / r["cus"] <= hi and
             (mqa is None or (r["H_KV"] == 1) == mqa)]
        if x:
            lines.append(f"* {name}: two / four {min(x):.3f}-{max(x):.3f} over {len(x)} shapes.")
    planned_right = sum((r["two_over_four"] < 1) == (r["planned_waves"] == 2) for r in rows)
    lines.append(f"* The planner's wave count is the faster one on {planned_right} of {len(rows)} shapes.")
    open(PROFILE_WAVES, "w").write("\n".join(lines) + "\n")
    print(f"wrote {PROFILE_WAVES}")


# ---------------------------------------------------------------- validation

class OracleRows:
    """The fp64 oracle on chosen sequences of a problem held on the device
    (fixed layout), computed once; every timed launch of that problem is
    compared with it before it is timed (the paper's harness rejects invalid
    candidates, Section 3.2)."""

    def __init__(self, np, torch, q, k, v, picks):
        from oracle import decode_attention
        bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
        self.picks = list(picks)
        self.np = np
        self.O, _ = decode_attention(bits(q[self.picks]), bits(k[self.picks]), bits(v[self.picks]))

    def check(self, torch, out) -> tuple:
        np = self.np
        from oracle import bf16_bits_to_f64
        got = bf16_bits_to_f64(out[self.picks].view(torch.int16).cpu().numpy().view(np.uint16))
        if not np.all(np.isfinite(got)):
            return False, float("inf"), float("inf")
        d = np.abs(got - self.O)
        return bool(d.max() <= 2e-2 and d.mean() <= 2e-3), float(d.max()), float(d.mean())


class OracleVarlen(OracleRows):
    """OracleRows for a varlen batch ([sum L_b, H_KV, D] with the lengths)."""

    def __init__(self, np, torch, q, k, v, lens, picks):
        from oracle import decode_attention
        bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
        self.picks = list(picks)
        self.np = np
        starts = np.concatenate([[0], np.cumsum(lens)])
        ks = [bits(k[int(starts[b]):int(starts[b + 1])]) for b in self.picks]
        vs = [bits(v[int(starts[b]):int(starts[b + 1])]) for b in self.picks]
        sub_lens = np.array([lens[b] for b in self.picks], dtype=np.int64)
        cu = np.concatenate([[0], np.cumsum(sub_lens)]).astype(np.int32)
        self.O, _ = decode_attention(bits(q[self.picks]), np.concatenate(ks), np.concatenate(vs), sub_lens, cu)


VALIDATION = {"validated": 0, "invalid": []}


def validate(torch, oracle, variants, what):
    """Check each launch's output (first K/V copy) against the oracle rows;
    record the count and any failure."""
    for var in variants:
        ok, mx, mean = oracle.check(torch, var.sample(torch))
        VALIDATION["validated"] += 1
        if not ok:
            VALIDATION["invalid"].append({"what": what, "launch": var.name,
                                          "max_abs": mx, "mean_abs": mean})
            log(f"INVALID {what} {var.name}: max-abs {mx:.3e} mean-abs {mean:.3e}")


# ---------------------------------------------------------------- calibration sweep

CAL_HEADS = ((1, 8, 1), (1, 64, 8), (1, 32, 1), (2, 32, 1), (4, 32, 1), (16, 32, 4), (4, 64, 8), (8, 64, 8),
             (32, 64, 8), (2, 128, 2), (1, 256, 32), (4, 256, 32))
CAL_L = (64, 128, 256, 384, 512, 640, 768, 1024, 2048, 4096, 8192)
CAL_SPLITS = {"warm": (1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64), "streamed": (1, 2, 3, 4, 6, 8, 12, 16, 24, 32)}
L2_BYTES = 8 << 22
RESIDENT_BYTES = 288 << 20
MAX_ARRIVAL_TILES = 4096


def heads_per_tile(H_Q, H_KV, cap):
    g = H_Q // H_KV
    if g <= cap:
        return g
    return max(h for h in range(1, cap + 1) if g % h == 0)


def calibration_plans(da, B, H_Q, H_KV, L, s, which, cus):
    """Every launch the planner can choose for s chunks per sequence (packing
    on): each packed tile width, each V slice count the planner considers
    (one workgroup per CU, K/V within L2) and each merge of the chunk states,
    with the fetch path and cache hint the planner would give them."""
    policy = da.POLICY_STREAMED if which == "streamed" else da.POLICY_MI355X
    base = da.da_make_plan(B, H_Q, H_KV, L, 128, s, 1, num_cus=cus, policy=policy)
    g = H_Q // H_KV
    kv = B * L * H_KV * 512
    out = []
    for w in sorted({heads_per_tile(H_Q, H_KV, 32), heads_per_tile(H_Q, H_KV, 16)}):
        tiles = B * H_Q // w
        for vs in (1, 2, 4):
            grid = tiles * s if vs == 1 else vs * 8 * -(-(tiles * s) // 8)
            if vs > 1 and (grid > cus or kv > L2_BYTES):
                continue
            chunk = -(-L // s)
            tpw = -(-(-(-chunk // 4)) // 32)   # 32-key tiles each of the four waves walks
            fetch = 2 if grid <= cus else (1 if tpw >= 2 else 0)
            readers = (g // w) * vs
            nt = (1 if readers == 1 else 0) if which == "streamed" else int(readers == 1 and kv > RESIDENT_BYTES)
            for comb in ((0, 1) if s > 1 and tiles <= MAX_ARRIVAL_TILES else (0,)):
                p = da.DaPlan.from_buffer_copy(base)
                p.heads_per_tile, p.tiles, p.v_slices, p.grid = w, tiles, vs, grid
                p.kv_fetch, p.kv_nontemporal, p.combine = fetch, nt, comb
                p.group_waves = 4    # the model prices four-wave launches (two waves are a rule on top)
                out.append(p)
    return out


def calibrate_run(args, da, torch, np) -> None:
    which = args.calibrate_set
    cus = da.da_device_info()[0]
    shapes = []
    t0 = time.perf_counter()
    for B, H_Q, H_KV in CAL_HEADS:
        for L in CAL_L:
            kvb = B * L * H_KV * 512
            if kvb > (1 << 30) or (which == "streamed" and kvb < (256 << 10)):
                continue
            gen = torch.Generator(device="cuda").manual_seed(B * 1000003 + H_Q * 1009 + L)
            q = torch.randn(B, H_Q, 128, device="cuda", generator=gen).to(torch.bfloat16)
            if which == "streamed":
                copies = max(1, min(4096, -(-(512 << 20) // kvb)))   # more than MALL + L2 (288 MiB)
                K = torch.empty(copies, B, L, H_KV, 128, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
                V = torch.empty_like(K).normal_(generator=gen)
                kvs = [(K[i], V[i]) for i in range(copies)]
                steps = max(copies, 20)
            else:
                K = torch.randn(1, B, L, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16)
                V = torch.randn(1, B, L, H_KV, 128, device="cuda", generator=gen).to(torch.bfloat16)
                kvs = [(K[0], V[0])]
                est = max(3.0, kvb / 5e6)
                steps = int(max(10, min(200, 2000.0 / est)))
            picks = [0] if B == 1 else [0, B - 1]
            orc = OracleRows(np, torch, q, kvs[0][0], kvs[0][1], picks)
            variants = []
            for s in CAL_SPLITS[which]:
                if s > 1 and s * 4 > L:
                    continue
                for p in calibration_plans(da, B, H_Q, H_KV, L, s, which, cus):
                    name = f"{p.heads_per_tile},{s},{p.v_slices},{p.combine}"
                    variants.append(Variant(name, da, torch, q, kvs[0][0], kvs[0][1], L, s, 1, steps,
                                            kv_copies=kvs if which == "streamed" else None, plan=p))
            validate(torch, orc, variants, f"calibration {which} B={B} H_Q={H_Q} H_KV={H_KV} L={L}")
            interleave(torch, variants, args.rounds)
            launches = [[v.plan.heads_per_tile, v.plan.num_splits, v.plan.v_slices, v.plan.combine,
                         round(v.median, 3)] for v in variants]
            shapes.append({"B": B, "H_Q": H_Q, "H_KV": H_KV, "L": L, "launches": launches})
            best = min(launches, key=lambda x: x[4])
            log(f"calibration {which} B={B} H_Q={H_Q} H_KV={H_KV} L={L}: {len(variants)} launches, best "
                f"{best} ({time.perf_counter() - t0:.0f} s)")
            del q, K, V, kvs, variants
            torch.cuda.empty_cache()
    out = {"set": which, "device_cus": cus, "kernel_source_sha256": kernel_source_sha(),
           "command": f"python3 bench.py --calibrate OUT.json --calibrate-set {which} --rounds {args.rounds}",
           "validated": VALIDATION["validated"], "invalid": VALIDATION["invalid"], "shapes": shapes}
    with open(args.calibrate, "w") as f:
        json.dump(out, f, separators=(",", ":"))
    log(f"wrote {args.calibrate}: {len(shapes)} shapes, {VALIDATION['validated']} launches validated, "
        f"{len(VALIDATION['invalid'])} invalid")
    if VALIDATION["invalid"]:
        sys.exit(3)


def main():
    args = parse()
    if args.traffic_summary:
        traffic_summary(args.traffic_summary)
        return
    if args.regression_summary:
        regression_summary(args.regression_summary)
        return
    if args.occupancy_summary:
        occupancy_summary(args.occupancy_summary)
        return
    if args.mixed_sweep_summary:
        mixed_sweep_summary(args.mixed_sweep_summary)
        return
    if args.schedule_sweep_summary:
        schedule_sweep_summary(args.schedule_sweep_summary)
        return
    if args.waves_sweep_summary:
        waves_sweep_summary(args.waves_sweep_summary)
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}); the decode kernel shards by "
              f"(sequence, KV head) with no exchange, so no multi-GPU figure is produced.", file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch

    import paper_2604_00028_amd as da
    from workloads import config_shapes, custom_shape, make_inputs

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)
    torch.cuda.set_device(0)
    cus, is950 = da.da_device_info()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).cuda()
    if args.only:
        only_run(args, da, torch, np, dev)
        return
    if args.regression:
        regression_run(args, da, torch)
        return
    if args.mixed_sweep:
        mixed_sweep_run(args, da, torch, np)
        return
    if args.schedule_sweep:
        schedule_sweep_run(args, da, torch, np)
        return
    if args.calibrate:
        calibrate_run(args, da, torch, np)
        return
    if args.waves_sweep:
        waves_sweep_run(args, da, torch, np)
        return

    # ---------------- headline: the high-load shape (B=32, H_Q=64, H_KV=8, L_K=8192, 1 GiB of K/V)
    K = args.steps
    shh = config_shapes(5)[0]
    log(f"device cus={cus} gfx950={is950}; generating {shh.name}")
    inh = make_inputs(shh)
    qh, kh, vh = dev(inh.q), dev(inh.k), dev(inh.v)
    for _ in range(args.warmup):
        da.da_decode_attn(qh, kh, vh)
    torch.cuda.synchronize()
    hh = Variant("heuristic", da, torch, qh, kh, vh, shh.L_K, 0, -1, K)
    h1_plan = Variant("s1_same_plan", da, torch, qh, kh, vh, shh.L_K, 1, -1, K)
    h1_paper = Variant("s1_paper_launch", da, torch, qh, kh, vh, shh.L_K, 1, 2, K)
    hs = [Variant(f"s{x}", da, torch, qh, kh, vh, shh.L_K, x, 1, K) for x in HIGHLOAD_SWEEP if x != 1]
    log("validating and timing high-load variants")
    validate(torch, OracleRows(np, torch, qh, kh, vh, [0, 31]), [hh, h1_plan, h1_paper] + hs, shh.name)
    interleave(torch, [hh, h1_plan, h1_paper] + hs, args.rounds)
    value = hh.median
    hsw = {1: round(h1_plan.median, 3), **{x.plan.num_splits: round(x.median, 3) for x in hs}}
    hbest = min(hsw, key=hsw.get)
    hbytes = algorithmic_bytes(shh.B, shh.H_Q, shh.H_KV, shh.L_K)
    achieved = hbytes / (value * 1e-6) / 1e9
    q25, q75 = np.percentile(hh.times, [25, 75])
    high = {"workload": shh.name, "us_per_call": round(value, 3), "iqr_us": [round(q25, 3), round(q75, 3)],
            "plan": plan_brief(hh.plan), "s1_same_plan_us": round(h1_plan.median, 3),
            "s1_paper_launch_us": round(h1_paper.median, 3), "best_fixed": hbest, "best_fixed_us": hsw[hbest],
            "vs_best_fixed": round(value / hsw[hbest], 3), "sweep_us": hsw, "algorithmic_bytes": hbytes,
            "kv_bytes_unique": 2 * shh.B * shh.L_K * shh.H_KV * 256,
            "kv_bytes_per_query_head": 2 * shh.B * shh.L_K * shh.H_Q * 256}
    cpu = None if args.no_cpu_baseline else cpu_baseline_highload(inh, args.cpu_seconds)
    del qh, kh, vh, hh, h1_plan, h1_paper, hs, inh
    torch.cuda.empty_cache()

    # ---------------- the Llama-3.1-70B GQA decode at B=1, L_K=512 in detail (config 2)
    shapes = {x.L_K: x for x in config_shapes(2)}
    sh = shapes[512]
    inp = make_inputs(sh)
    q, k, v = dev(inp.q), dev(inp.k), dev(inp.v)
    Kl = max(args.steps, 100)
    log(f"timing {sh.name} in detail")
    heur = Variant("heuristic", da, torch, q, k, v, sh.L_K, 0, -1, Kl)
    base = Variant("s1_same_plan", da, torch, q, k, v, sh.L_K, 1, -1, Kl)
    paper_s1 = Variant("s1_paper_launch", da, torch, q, k, v, sh.L_K, 1, 2, Kl)
    pol = {name: Variant(name, da, torch, q, k, v, sh.L_K, 0, -1, Kl,
                         plan=da.da_choose_splits(sh.B, sh.H_Q, sh.H_KV, sh.L_K, policy=code))
           for name, code in (("paper", da.POLICY_PAPER), ("evolved", da.POLICY_EVOLVED),
                              ("streamed", da.POLICY_STREAMED), ("table", da.POLICY_TABLE))}
    sweep = [Variant(f"s{x}", da, torch, q, k, v, sh.L_K, x, 1, Kl) for x in SWEEP if x != 1]
    # the same split counts with the chunk states merged by a second launch
    two = [Variant(f"s{x}_two_launch", da, torch, q, k, v, sh.L_K, 0, -1, Kl,
                   plan=with_combine(da, da.da_make_plan(sh.B, sh.H_Q, sh.H_KV, sh.L_K, 128, x, 1), 0))
           for x in (2, 4, 8)]
    unpacked = [Variant("s1_unpacked", da, torch, q, k, v, sh.L_K, 1, 0, Kl)]
    ncopy = 256   # cold cache: cycle through 256 distinct KV copies (512 MiB > L2 + MALL)
    copies = [(torch.randn_like(k, dtype=torch.float32).to(torch.bfloat16),
               torch.randn_like(v, dtype=torch.float32).to(torch.bfloat16)) for _ in range(ncopy)]
    cold = [Variant(n, da, torch, q, k, v, sh.L_K, s_, p_, Kl, kv_copies=copies)
            for n, s_, p_ in (("cold_heuristic", 0, -1), ("cold_s1_paper_launch", 1, 2))]
    allv = [heur, base, paper_s1] + list(pol.values()) + sweep + two + unpacked
    validate(torch, OracleFull(np, inp), allv, sh.name)
    validate(torch, OracleRows(np, torch, q, copies[0][0], copies[0][1], [0]), cold, sh.name + " cold")
    # the cold-cache pair streams 512 MiB per replay through L2 and the MALL: timed on its own, so that
    # its evictions do not land between the warm launches' replays
    interleave(torch, allv, args.rounds)
    interleave(torch, cold, args.rounds)
    sweep_us = {1: round(base.median, 3), **{x.plan.num_splits: round(x.median, 3) for x in sweep}}
    best_s = min(sweep_us, key=sweep_us.get)
    detail = {"workload": sh.name, "heuristic_us": round(heur.median, 3), "plan": plan_brief(heur.plan),
              "s1_same_plan_us": round(base.median, 3), "s1_paper_launch_us": round(paper_s1.median, 3),
              "speedup_vs_s1_paper_launch": round(paper_s1.median / heur.median, 3),
              "hbm_gbs": round(algorithmic_bytes(sh.B, sh.H_Q, sh.H_KV, sh.L_K) / (heur.median * 1e-6) / 1e9, 1),
              "policies": {n: {"plan": plan_brief(x.plan), "us": round(x.median, 3)} for n, x in pol.items()},
              "best_fixed": best_s, "vs_best_fixed": round(heur.median / sweep_us[best_s], 3),
              "sweep_us": sweep_us,
              "sweep_plans": {x.plan.num_splits: plan_brief(x.plan) for x in sweep},
              "two_launch_us": {x.plan.num_splits: round(x.median, 3) for x in two},
              "unpacked_s1_us": round(unpacked[0].median, 3),
              "cold_us": {"heuristic": round(cold[0].median, 3), "s1_paper_launch": round(cold[1].median, 3)}}
    del copies, cold, allv

    # ---------------- longer Llama GQA contexts at B=1, where splits pay on MI355X
    longer = {}
    if not args.no_long:
        for L in (1024, 2048, 8192):
            shL = custom_shape(1, 64, 8, L)
            inL = make_inputs(shL, seed=3000 + L)
            qL, kL, vL = dev(inL.q), dev(inL.k), dev(inL.v)
            log(f"timing L_K={L}")
            hv = Variant("heuristic", da, torch, qL, kL, vL, L, 0, -1, Kl)
            pv = Variant("s1_paper_launch", da, torch, qL, kL, vL, L, 1, 2, Kl)
            sv = [Variant(f"s{x}", da, torch, qL, kL, vL, L, x, 1, Kl) for x in LONG_SWEEP]
            validate(torch, OracleFull(np, inL), [hv, pv] + sv, shL.name)
            interleave(torch, [hv, pv] + sv, args.rounds)
            sw = {x.plan.num_splits: round(x.median, 3) for x in sv}
            longer[L] = {"heuristic_us": round(hv.median, 3), "plan": plan_brief(hv.plan),
                         "s1_paper_launch_us": round(pv.median, 3),
                         "speedup_vs_s1_paper_launch": round(pv.median / hv.median, 3),
                         "s1_same_plan_us": sw[1], "best_fixed": min(sw, key=sw.get),
                         "best_fixed_us": min(sw.values()), "vs_best_fixed": round(hv.median / min(sw.values()), 3),
                         "sweep_us": sw}
            del qL, kL, vL, hv, pv, sv

    low = None if args.no_small else low_head_run(args, da, torch, np, dev)
    streamed = None if args.no_streamed else streamed_run(args, da, torch)
    ragged = None if args.no_ragged else ragged_run(args, da, torch, np)
    margin = None if args.no_cu_margin else cu_margin_run(args, da, torch, np)
    log("timing the HBM read probe")
    probe = read_probe_run(torch)

    result = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "us/call",
        "n_gpus": 1,
        "steps": K,
        "warmup": args.warmup,
        "ms_per_step": round(value / 1000.0, 6),
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": shh.name, "B": shh.B, "H_Q": shh.H_Q, "H_KV": shh.H_KV, "head_dim": shh.D,
                   "L_K": shh.L_K, "num_splits": 0, "pack_gqa": -1, "plan": high["plan"], "num_cus": cus},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic_for(shh.name)},
        "cpu_baseline": cpu,
        "speedup_vs_s1_same_plan": round(high["s1_same_plan_us"] / value, 3),
        "speedup_vs_s1_paper_launch": round(high["s1_paper_launch_us"] / value, 3),
        "vs_best_fixed": high["vs_best_fixed"],
        "validated": VALIDATION["validated"],
        "invalid": VALIDATION["invalid"],
        "high_load": high,
        "llama70b_b1_l512": detail,
        "long_lk": longer,
        "low_head": low,
        "streamed": streamed,
        "ragged": ragged,
        "cu_margin": margin,
        "hbm_read_probe": probe,
    }
    # compact summaries last, where a tail of the output shows them
    if low:
        sp = {n: r["speedup_vs_s1_paper_launch"] for n, r in low.items()}
        result["low_head_summary"] = {
            "speedup_vs_s1_paper_launch": sp, "min": min(sp.values()), "max": max(sp.values()),
            "llama70b_b1_l512_us": [detail["heuristic_us"], detail["s1_paper_launch_us"]],
            "vs_best_fixed_worst": max(r["vs_best_fixed"] for r in low.values())}
    if streamed:
        result["streamed_summary"] = {n: r["streamed_speedup_vs_s1"] for n, r in streamed.items()}
        result["streamed_vs_best_summary"] = {
            "streamed_policy": {n: r["streamed_vs_best"] for n, r in streamed.items()},
            "table_streamed_policy": {n: r["table_vs_best"] for n, r in streamed.items()}}
    result["high_load_summary"] = {"us": high["us_per_call"], "gbs": round(achieved, 1),
                                   "frac": round(achieved / HBM_PEAK_GBS, 4), "plan": high["plan"],
                                   "s1_paper_launch_us": high["s1_paper_launch_us"],
                                   "best_fixed_us": high["best_fixed_us"], "validated": VALIDATION["validated"],
                                   "read_probe_gbps": probe["best_gbps"],
                                   "frac_of_read_probe": round(achieved / probe["best_gbps"], 4)}
    print(json.dumps(result), flush=True)
    if VALIDATION["invalid"]:
        log(f"{len(VALIDATION['invalid'])} timed launches disagree with the oracle")
        sys.exit(3)


def with_combine(da, plan, combine):
    """A copy of a plan with the merge of its chunk states set (a second
    launch: 0; inside the split launch: 1)."""
    p = da.DaPlan.from_buffer_copy(plan)
    p.combine = combine if p.num_splits > 1 else 0
    if p.combine == 1 and p.group_waves == 2:
        # the in-launch merge runs in four-wave launches: K/V straight into LDS with one workgroup per CU,
        # through registers into LDS where some CUs hold two (two-wave chunks hold at least 512 keys)
        p.group_waves, p.kv_fetch = 4, 2 if p.grid <= p.num_cus else 1
    return p


def cpu_baseline_highload(inp, seconds: float):
    """The fp64 oracle as it stands, on the host cores, on a bounded sample
    of the high-load call: passes over its first 8 of 32 sequences for about
    `seconds`, scaled to one call."""
    from oracle import decode_attention
    cores, blas, model = host_cores()
    n_seq = 8
    q, k, v = inp.q[:n_seq], inp.k[:n_seq], inp.v[:n_seq]
    decode_attention(q, k, v)
    n = 0
    t0 = time.perf_counter()
    while time.perf_counter() - t0 < seconds:
        decode_attention(q, k, v)
        n += 1
    dt = time.perf_counter() - t0
    per_call = dt / n * (inp.q.shape[0] / n_seq)
    return {"value": round(per_call * 1e6, 1), "unit": "us/call", "cores": cores, "blas_threads": blas,
            "cpu_model": model, "kind": "oracle",
            "sample": f"{n} passes over {n_seq} of the {inp.q.shape[0]} sequences of the high-load call "
                      f"(fp64 NumPy, {seconds:.0f} s budget), scaled to one call"}


if __name__ == "__main__":
    main()
