"""The workloads by which the speed of the framework is measured: gradient
aggregation and momentum-SGD calls through `paper_1511_00175_amd.Plan`, from a
launch-bound step of tens of thousands of parameters to the largest networks
in `workloads/tables.py`.

A case names its segment table (`net` with a run of a network's layers, `flat`
for one segment, `ragged` for random odd lengths and gaps), the worker count,
the replicas' storage type, the summation order and the call:
  step        Plan.step: reduce, average, SGD, write back
  step_out    the same, and keep the raw sum
  step_bcast  the same, and send w' to every worker's copy
  composed    Plan.tree_reduce, Plan.sgd_step, Plan.broadcast, one after another
  reduce      Plan.tree_reduce alone (one node's share of a larger tree)
  noalloc     Plan.step_noalloc, the entry point for callers that cannot allocate
"""
import math

import numpy as np
import torch

import paper_1511_00175_amd as fc
from workloads import gen, tables

NETS = ("nin", "googlenet", "googlenet_caffe_bias", "alexnet", "vgg19")
OPS = ("step", "step", "step", "step_out", "step_bcast", "composed", "reduce", "noalloc")
MU = 0.9
MIN_ELEMS, MAX_ELEMS = 4_000, 140_000_000
MAX_BYTES = 10_000_000_000  # of a drawn case: below the largest listed one's


def listed():
    return [
        # GoogLeNet's 58 layers from 128 workers: the benchmark's headline step
        {"name": "googlenet_k128", "op": "step", "table": "net", "net": "googlenet", "first": 0, "layers": 0,
         "K": 128, "dtype": "f32", "order": "tree"},
        # VGG-19 from 16 workers: the largest model, several rounds of the chip
        {"name": "vgg19_k16", "op": "step", "table": "net", "net": "vgg19", "first": 0, "layers": 0,
         "K": 16, "dtype": "f32", "order": "tree"},
        # AlexNet from 128 workers with 16-bit gradients: the most bytes
        {"name": "alexnet_k128_f16", "op": "step", "table": "net", "net": "alexnet", "first": 0, "layers": 0,
         "K": 128, "dtype": "f16", "order": "tree"},
        # NiN from 32 workers, the new weights sent back to each of them
        {"name": "nin_k32_bcast", "op": "step_bcast", "table": "net", "net": "nin", "first": 0, "layers": 0,
         "K": 32, "dtype": "f32", "order": "tree"},
        # parameter-server order in three calls, each bias with its own rate and decay
        {"name": "googlenet_k16_composed", "op": "composed", "table": "net", "net": "googlenet_caffe_bias",
         "first": 0, "layers": 0, "K": 16, "dtype": "f32", "order": "linear"},
        # one of 8 nodes reduces its 16 of 128 workers' 16-bit gradients
        {"name": "alexnet_leaf_k16_f16", "op": "reduce", "table": "net", "net": "alexnet", "first": 0, "layers": 0,
         "K": 16, "dtype": "f16", "order": "tree"},
        # the owner of about an eighth of GoogLeNet adds 8 nodes' partial sums and updates
        {"name": "owner_k8_out", "op": "step_out", "table": "net", "net": "googlenet", "first": 27, "layers": 12,
         "K": 8, "dtype": "f32", "order": "tree"},
        # one inception module aggregated as soon as its gradients are there, 16-bit gradients
        {"name": "module_k128_f16", "op": "step", "table": "net", "net": "googlenet", "first": 3, "layers": 6,
         "K": 128, "dtype": "f16", "order": "tree"},
        # the first layers of NiN from 32 workers, by a caller that cannot allocate
        {"name": "layers_k32_noalloc", "op": "noalloc", "table": "net", "net": "nin", "first": 0, "layers": 5,
         "K": 32, "dtype": "f32", "order": "tree"},
        # the smallest earnest step: three convolutions, 8 workers; latency only
        {"name": "conv_k8", "op": "step", "table": "net", "net": "nin", "first": 0, "layers": 3,
         "K": 8, "dtype": "f32", "order": "tree"},
        # one flat vector of 2^20 elements, 4 workers: launch-bound
        {"name": "flat_k4", "op": "step", "table": "flat", "n": 1 << 20, "K": 4, "dtype": "f32", "order": "tree"},
        # the most workers a plan takes, odd segment lengths, parameter-server order
        {"name": "ragged_k1000", "op": "step", "table": "ragged", "segments": 24, "longest": 701, "table_seed": 5,
         "K": 1000, "dtype": "f32", "order": "linear"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _elem_bytes(case):
    """Bytes of one pass per parameter that the call cannot do without."""
    K, rep = case["K"], case["K"] * (2 if case["dtype"] == "f16" else 4)
    return {"step": rep + 16, "step_out": rep + 20, "step_bcast": rep + 16 + 4 * K, "noalloc": rep + 16,
            "reduce": rep + 4, "composed": rep + 4 + 4 * K + 16}[case["op"]]


def draw(rng):
    case = {"op": rng.choice(OPS), "K": _log(rng, 1, 1024), "dtype": rng.choice(("f32", "f32", "f16")),
            "order": rng.choice(("tree", "tree", "linear"))}
    most = min(MAX_ELEMS, MAX_BYTES // _elem_bytes(case))
    if case["op"] == "noalloc":
        most = min(most, fc.FC_NOALLOC_MAX_ELEMS // 2)  # gaps and padding count as well
    n = _log(rng, MIN_ELEMS, most)
    kind = rng.choice(("net", "flat", "ragged"))
    if kind == "net":
        # a run of layers of about n parameters
        net = rng.choice(NETS)
        sizes = [L.weights + L.out_ch for L in tables.get(net).layers]
        fits = [i for i, x in enumerate(sizes) if x <= n]
        if fits:
            first = rng.choice(fits)
            count, total = 1, sizes[first]
            while first + count < len(sizes) and total + sizes[first + count] <= n:
                total += sizes[first + count]
                count += 1
            return dict(case, table="net", net=net, first=first, layers=count)
        kind = "flat"
    if kind == "flat":
        return dict(case, table="flat", n=n)
    segments = _log(rng, 2, 128)
    return dict(case, table="ragged", segments=segments, longest=max(3, min(2 * n, most) // segments),
                table_seed=rng.randrange(1 << 20))


def _workload(case):
    """The case's table and recipes as a workloads.tables.Workload."""
    if case["table"] == "net":
        wl = tables.get(case["net"])
        if case["layers"]:
            wl.layers = wl.layers[case["first"]:case["first"] + case["layers"]]
            wl.segments, wl.padded = tables.lay_out(wl.layers,
                                                    caffe_bias_mults=case["net"].endswith("caffe_bias"))
    else:
        wl = tables.flat()
        layer = wl.layers[0]
        if case["table"] == "flat":
            rows = [(0, case["n"], 1.0, 1.0)]
        else:
            rows, _ = gen.random_table(np.random.default_rng(case["table_seed"]), case["segments"], case["longest"], 4)
        wl.segments = [tables.Segment(f"s{j}", r[0], r[1], 1, False, layer) for j, r in enumerate(rows)]
        wl.padded = -(-(rows[-1][0] + rows[-1][1]) // tables.ALIGN) * tables.ALIGN
    wl.K, wl.dtype = case["K"], case["dtype"]
    return wl


def _inputs(wl, seed):
    """Replicas, weights and a velocity as after some steps of training."""
    dev = torch.device("cuda")
    reps, w, v = gen.device_inputs(wl, seed, dev)
    g = torch.Generator(device=dev)
    g.manual_seed(seed + 2)
    for s in wl.segments:
        v[s.offset:s.offset + s.length] = torch.randn(s.length, generator=g, device=dev) * 1e-4
    return reps, w, v


def prepare(case, seed):
    wl = _workload(case)
    reps, w, v = _inputs(wl, seed)
    op = case["op"]
    s = {"op": op, "reps": reps, "w": w, "v": v, "args": (wl.lr, MU, wl.wd, wl.batch),
         "plan": fc.Plan(wl.table(), case["K"], case["dtype"], case["order"])}
    if op in ("step_out", "composed", "reduce"):
        s["out"] = torch.zeros_like(w)
    if op in ("step_bcast", "composed"):
        s["copies"] = torch.zeros((case["K"], gen.default_stride(wl)), dtype=torch.float32, device=w.device)
    return s


def run(state):
    s, plan, op = state, state["plan"], state["op"]
    if op == "reduce":
        plan.tree_reduce(s["reps"], s["out"])
        return {"sum": s["out"]}
    if op == "step":
        plan.step(s["reps"], s["w"], s["v"], *s["args"])
        return {"w": s["w"], "v": s["v"]}
    if op == "step_out":
        plan.step(s["reps"], s["w"], s["v"], *s["args"], out=s["out"])
        return {"w": s["w"], "v": s["v"], "sum": s["out"]}
    if op == "step_bcast":
        plan.step(s["reps"], s["w"], s["v"], *s["args"], bcast=s["copies"])
        return {"w": s["w"], "v": s["v"], "copies": s["copies"]}
    if op == "noalloc":
        plan.step_noalloc(s["reps"], s["w"], s["v"], *s["args"])
        return {"w": s["w"], "v": s["v"]}
    plan.tree_reduce(s["reps"], s["out"])
    plan.sgd_step(s["w"], s["v"], s["out"], *s["args"])
    plan.broadcast(s["w"], s["copies"])
    return {"w": s["w"], "v": s["v"], "sum": s["out"], "copies": s["copies"]}


def work(case):
    n = _workload(case).n_params
    update = 0 if case["op"] == "reduce" else 8
    return {"bytes": n * _elem_bytes(case), "flops": n * (case["K"] - 1 + update)}


def tolerance(case):
    # the summation order and the rounding of every operation are part of the
    # interface, so every correct implementation gives the same bits
    return "exact"


def exact(case, seed):
    wl = _workload(case)
    reps, w, v = _inputs(wl, seed)
    f32 = lambda x: float(np.float32(x))  # noqa: E731
    w, v = w.double(), v.double()
    total = torch.zeros_like(w)
    part = max(1, (1 << 28) // case["K"])  # elements summed at a time
    for s in wl.segments:
        for a in range(s.offset, s.offset + s.length, part):
            b = min(a + part, s.offset + s.length)
            total[a:b] = reps[:, a:b].double().sum(0)
    del reps
    if case["op"] == "reduce":
        return {"sum": total}
    for s in wl.segments:
        sl = slice(s.offset, s.offset + s.length)
        d = total[sl] / wl.batch + f32(wl.wd) * s.decay_mult * w[sl]
        v[sl] = f32(MU) * v[sl] + f32(wl.lr) * s.lr_mult * d
        w[sl] -= v[sl]
    got = {"w": w, "v": v}
    if case["op"] in ("step_out", "composed"):
        got["sum"] = total
    if case["op"] in ("step_bcast", "composed"):
        copies = torch.zeros((case["K"], gen.default_stride(wl)), dtype=torch.float64, device=w.device)
        for s in wl.segments:
            copies[:, s.offset:s.offset + s.length] = w[s.offset:s.offset + s.length]
        got["copies"] = copies
    return got
