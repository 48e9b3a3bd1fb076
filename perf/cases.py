"""What the speed of this library is measured on: the serving stream under its policies, the single steps (segment, exit head,
compaction) a program with a driver of its own calls, int8 and bf16, from one request to ten thousand.

A case is a dict of plain values, `prepare` makes what a program holds before the call (the engine with its tables, the
inputs on the GPU), `run` is one pass through the public calls, `work` says what the pass cannot do without.

Kinds of cases
  stream    Engine.serve_stream on n requests that are all queued at the start, so that the time is the path's and not the
            arrival rate's: admission, segments, exit heads, compaction and refill under one of the three policies
  exits     every segment and every exit head on one whole batch: what a program does that sets exit thresholds or measures
            the accuracy of each exit
  boundary  one exit boundary on a batch of activations: exit head, compaction of the survivors, refill of the freed slots
"""
import json
import math
import os

import numpy as np
import torch

import paper_2209_13443_amd as ee
import workloads as W

_CALIB = os.path.join(os.path.dirname(os.path.abspath(W.__file__)), "calib")
_STREAM_NETS = ("tiny_i8", "resnet18_i8", "mobilenetv2_i8", "resnet50_i8", "resnet50_eq_i8", "inception_i8", "resnet50_bf16")
_STEP_NETS = _STREAM_NETS + ("tiny_bf16",)


def _stream(name, net, n, b_max, refill, lanes=1, tuned=True):
    return dict(name=name, kind="stream", net=net, n=n, b_max=b_max, refill=refill, lanes=lanes, tuned=tuned)


def listed():
    return [
        # a lone user's requests, served one after the other: the SERIAL baseline, launches and latency are everything
        _stream("serial_resnet50_i8", "resnet50_i8", 8, 1, 0),
        # a small model on small images in few slots, Algorithm 1 as printed apart from the smallest catch-up batch
        _stream("alg1_tiny_i8", "tiny_i8", 64, 8, 1),
        # model-level batching: batches without refill, the batch shrinks from exit to exit
        _stream("static_resnet18_i8", "resnet18_i8", 1024, 32, 0),
        # the mobile network, all requests queued, stage pools
        _stream("pools_mobilenetv2_i8", "mobilenetv2_i8", 4096, 64, 2, lanes=2),
        # the benchmark's own stream at capacity
        _stream("pools_resnet50_i8", "resnet50_i8", 10000, 64, 2, lanes=2),
        # the paper's Algorithm 1 on it; a number of requests that fills no last batch
        _stream("alg1_resnet50_i8", "resnet50_i8", 3001, 64, 1),
        # the large-batch bf16 stream
        _stream("pools_resnet50_bf16", "resnet50_bf16", 8000, 256, 2, lanes=2),
        # the second network of the evaluation: rectangular kernels, concatenation
        _stream("pools_inception_i8", "inception_i8", 3000, 64, 2, lanes=2),
        # single steps on a ragged batch, by a program that never ran the tuner
        dict(name="exits_resnet50_i8", kind="exits", net="resnet50_i8", b=37, tuned=False),
        # bf16 steps on a handful of samples
        dict(name="exits_resnet50_bf16", kind="exits", net="resnet50_bf16", b=5, tuned=True),
        # the smallest call: one image through every segment and exit head
        dict(name="exits_mobilenetv2_i8", kind="exits", net="mobilenetv2_i8", b=1, tuned=True),
        # one boundary of the large-batch stream: 321 MB of activations in, the survivors and 56 newcomers out
        dict(name="boundary_resnet50_bf16", kind="boundary", net="resnet50_bf16", stage=0, b=200, b_incr=56),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    what = rng.random()
    if what < 0.6:
        refill = rng.choice((0, 1, 2, 2))
        b_max = _log_int(rng, 1, 256)
        return dict(kind="stream", net=rng.choice(_STREAM_NETS), n=_log_int(rng, 1, min(5000, 128 * b_max)), b_max=b_max, refill=refill,
                    lanes=rng.choice((1, 2)) if refill == 2 else 1, tuned=rng.random() < 0.75)
    net = rng.choice(_STEP_NETS)
    if what < 0.85:
        return dict(kind="exits", net=net, b=_log_int(rng, 1, 256), tuned=rng.random() < 0.75)
    b = _log_int(rng, 1, 200)
    return dict(kind="boundary", net=net, stage=rng.randrange(len(_record(net)["split"]) - 1), b=b, b_incr=rng.randint(0, min(56, b)))


_records, _nets, _engines = {}, {}, {}


def _record(net):
    """The network's calibration record (exit split, thresholds)."""
    if net not in _records:
        with open(os.path.join(_CALIB, net + ".json")) as f:
            _records[net] = json.load(f)
    return _records[net]


def _net(net):
    if net not in _nets:
        _nets[net] = W.load_net(net)
    return _nets[net]


def _engine(net, b_max, lanes, tuned):
    """A program loads its network and tunes it once and serves with that engine from then on: (engine, latency table)."""
    key = (net, b_max, lanes, tuned)
    if key not in _engines:
        eng = ee.Engine(_net(net), b_max)
        if lanes > 1:
            eng.set_lanes(lanes)
        if tuned:
            eng.autotune(reps=3)
        _engines[key] = (eng, eng.measure_lut(reps=1))
    return _engines[key]


def _inputs(blob, n, shape, gen, post_relu=False):
    """n samples of the given shape: uniform int8 or normal bf16 (as 16-bit patterns), the request pools' distributions."""
    if blob.dtype == W.DT_I8:
        x = torch.randint(-128, 128, (n,) + shape, dtype=torch.int8, device="cuda", generator=gen)
        return x.clamp_(min=0) if post_relu else x
    x = torch.empty((n,) + shape, dtype=torch.bfloat16, device="cuda")
    for i in range(0, n, 512):
        part = torch.randn((min(512, n - i),) + shape, device="cuda", generator=gen)
        x[i:i + 512] = part.clamp_(min=0) if post_relu else part
    return x.view(torch.int16)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    blob = _net(case["net"])
    if case["kind"] == "stream":
        eng, lut = _engine(case["net"], case["b_max"], case["lanes"], case["tuned"])
        return dict(case=case, eng=eng, lut=lut, pool=_inputs(blob, case["n"], blob.in_shape(), gen), arrivals=np.zeros(case["n"], np.int64),
                    zero_copy=int(eng.zero_copy_supported()))
    if case["kind"] == "exits":
        eng, _ = _engine(case["net"], case["b"], 1, case["tuned"])
        return dict(case=case, eng=eng, x=_inputs(blob, case["b"], blob.in_shape(), gen), shapes=[blob.stage_out_shape(s) for s in range(blob.n_stages)],
                    thr=[float(e["thr"]) for e in blob.exits])
    s, b, incr = case["stage"], case["b"], case["b_incr"]
    eng, _ = _engine(case["net"], b + incr, 1, False)
    shape, e = blob.stage_out_shape(s), _record(case["net"])["exits"][s]
    # the exit's share of the batch leaves, from slots all over it
    flags = (torch.randperm(b, device="cuda", generator=gen) < round(b * e["exited"] / e["reached"])).to(torch.uint8)
    return dict(case=case, eng=eng, act=_inputs(blob, b, shape, gen, True), flags=flags, ids=torch.randperm(b, device="cuda", generator=gen).to(torch.int32),
                new=_inputs(blob, incr, shape, gen, True) if incr else None,
                new_ids=torch.arange(b, b + incr, dtype=torch.int32, device="cuda") if incr else None, thr=float(blob.exits[s]["thr"]))


def _values(eng, t):
    return t.view(torch.bfloat16) if eng.dtype == ee.EE_BF16 else t


def run(state):
    case, eng = state["case"], state["eng"]
    if case["kind"] == "stream":
        res, stats, _ = eng.serve_stream(state["arrivals"], state["pool"], state["lut"], b_max=case["b_max"], refill=case["refill"],
                                         min_incr=max(1, case["b_max"] // 2), lanes=case["lanes"], zero_copy=state["zero_copy"])
        # latencies and the counts of runs are measurements; what a request gets is not
        return dict(exit_idx=res["exit_idx"], label=res["label"], conf=res["conf"], score=res["score"])
    if case["kind"] == "exits":
        act, out = state["x"], []
        for s, shape in enumerate(state["shapes"]):
            act = eng.stage_forward(s, act, shape)
            out.append((_values(eng, act),) + eng.exit_head(s, act, state["thr"][s]))
        return out
    label, conf, score, flag = eng.exit_head(case["stage"], state["act"], state["thr"])
    merged, ids, b_rem, b_merged = eng.compact_refill(case["stage"], state["flags"], state["act"], state["ids"], state["new"], state["new_ids"])
    return dict(label=label, conf=conf, score=score, flag=flag, merged=_values(eng, merged), ids=ids, b_rem=b_rem, b_merged=b_merged)


def work(case):
    blob = _net(case["net"])
    es, stages = blob.elem_bytes, range(blob.n_stages)
    size = lambda shape: es * int(np.prod(shape))
    macs, weights = [], []                                  # per segment with its exit head
    for s in stages:
        head = int(blob.exits[s]["c"]) * int(blob.exits[s]["n_cls"])
        m, w = head, es * head
        for op in blob.stage_ops(s):
            if int(op["kind"]) in (W.OP_CONV, W.OP_DWCONV):
                k = int(op["kh"]) * int(op["kw"]) * (int(op["c_in"]) if int(op["kind"]) == W.OP_CONV else 1)
                m += int(op["h_out"]) * int(op["w_out"]) * int(op["c_out"]) * k
                w += es * int(op["c_out"]) * k
        macs.append(m)
        weights.append(w)
    if case["kind"] == "stream":                            # a request runs the segments up to its exit
        split = _record(case["net"])["split"]
        reach = [1.0 - sum(split[:s]) for s in stages]
        return {"bytes": case["n"] * (size(blob.in_shape()) + 32) + sum(weights), "flops": 2.0 * case["n"] * sum(r * m for r, m in zip(reach, macs))}
    if case["kind"] == "exits":                             # every segment's output is handed back
        b = case["b"]
        return {"bytes": b * (size(blob.in_shape()) + sum(size(blob.stage_out_shape(s)) + 17 for s in stages)) + sum(weights), "flops": 2.0 * b * sum(macs)}
    s, b, incr = case["stage"], case["b"], case["b_incr"]
    e = _record(case["net"])["exits"][s]
    kept = b - round(b * e["exited"] / e["reached"])
    head = int(blob.exits[s]["c"]) * int(blob.exits[s]["n_cls"])
    return {"bytes": size(blob.stage_out_shape(s)) * (b + incr + kept + incr) + es * head + 18 * b, "flops": 2.0 * b * head}


def tolerance(case):
    if _net(case["net"]).dtype == W.DT_I8:
        return "exact"
    # bf16 activations are rounded after every layer and the order of a layer's sum is the kernel's; a confidence within
    # the rounding of a threshold may leave at the next exit, with that exit's label and confidence
    return {"rel": 0.02, "max": 0.9, "differ": 0.01}
