"""The work this package is used for, as timed cases.

Four kinds of call:

* ``tables``: explicit op tables already on the GPU -- random programs, or
  hand-written programs lowered by the front end -- simulated with
  dsim_simulate_tables, then the best feasible programs selected.
* ``grid``: a strategy grid of a model simulated with
  dsim_simulate_parametric, then the best feasible strategies selected.
* ``written``: a strategy grid's whole programs written as tables with
  dsim_materialize_tables, simulated and ranked.
* ``generate``: the random-program workload written on the GPU.

A pass is what a user's program does per cluster or per search: it holds its
model, its strategies or tables, and its result buffers; the device model's
rates differ from seed to seed (another calibration of the cluster).
"""
import math
import os
import random
from dataclasses import replace

import numpy as np
import torch

from paper_2111_05426_amd import dsim, frontend, programs
from paper_2111_05426_amd import workloads as W

LOG2_1E3, LOG2_1E6, LOG2_1E9, LOG2_1E12 = (math.log2(v) for v in (1e3, 1e6, 1e9, 1e12))


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _grid(name, w, kind="grid"):
    """A workload's model, grid rule and cluster as plain values."""
    m, g = w.model, w.grid
    return {"name": name, "kind": kind, "family": m.family, "mode": m.mode, "layers": m.n_layers, "heads": m.n_heads,
            "d": m.d_model, "d_ff": m.d_ff, "seq": m.seq_len, "vocab": m.vocab, "batch": m.global_batch,
            "elem": m.elem_bytes, "schedule": m.schedule, "recompute": m.recompute, "zero": m.zero,
            "overlap": m.overlap, "max_devices": g.max_devices, "k_mode": g.k_mode, "k_max": g.k_max,
            "cluster": "mi355x" if w.device.matmul else "default", "cap": w.device.mem_cap_bytes, "top": w.top_k}


def _random(name, n, ops, dev, ragged, top=1):
    return {"name": name, "kind": "tables", "programs": "random", "n": n, "ops": ops, "n_dev": dev, "ragged": ragged,
            "cluster": "default", "top": top}


def _lowered(name, n, layers, d, heads, cluster, top=1):
    return {"name": name, "kind": "tables", "programs": "lowered", "n": n, "layers": layers, "d": d, "heads": heads,
            "n_dev": 8, "cluster": cluster, "top": top}


def listed():
    return [
        # the benchmark's default step: a million random programs, HBM-resident
        _random("random_1m", 1_000_000, 2048, 8, False),
        # programs of different lengths padded to the longest, each with its
        # own resident bytes, an odd number of them
        _random("random_ragged", 40_001, 600, 5, True, top=8),
        # the smallest call of the table path: a few hundred short programs
        _random("random_small", 640, 256, 8, False),
        # hand-written GPT-2-shaped layer programs through the front end,
        # on the cluster calibrated on this GPU (MatMul regression, nodes)
        _lowered("lowered_gpt2", 400, 4, 768, 12, "mi355x"),
        # the tiny MLP's grid written out op by op and simulated as tables
        _grid("tiny_mlp_written", W.TINY_MLP, kind="written"),
        # the random workload's tables, written before they are simulated
        {"name": "generate", "kind": "generate", "n": 250_000, "ops": 512, "n_dev": 8},
        # strategy grids, from 30 candidates (latency and launches) over a few
        # hundred to the GPT-3-shaped 39,965, with its ZeRO and its calibrated
        # two-stream variant
        _grid("tiny_mlp", W.TINY_MLP),
        _grid("large_mlp", W.LARGE_MLP),
        _grid("gpt2_small_train", W.GPT2_SMALL_TRAIN),
        _grid("gpt3_175b", W.GPT3_175B),
        _grid("gpt3_175b_zero", W.GPT3_175B_ZERO),
        _grid("gpt3_175b_mi355x_overlap", W.GPT3_175B_MI355X_OVERLAP),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_model(rng, mlp):
    mode = rng.choice([W.INFER, W.TRAIN_SGD, W.TRAIN_ADAM, W.TRAIN_ADAM_MIXED, W.TRAIN_ADAM_MIXED])
    train = mode != W.INFER
    option = rng.choice(["plain", "plain", "recompute", "zero", "overlap"]) if train else "plain"
    c = {"mode": mode, "schedule": rng.choice([W.SCHED_1F1B, W.SCHED_1F1B, W.SCHED_GPIPE]),
         "recompute": int(option == "recompute"), "zero": int(option == "zero"), "overlap": int(option == "overlap"),
         "cluster": rng.choice(["default", "default", "mi355x"]), "elem": rng.choice([2, 2, 4]),
         "cap": rng.choice([0, 288_000_000_000]), "top": rng.choice([1, 1, 4, 16])}
    if mlp:
        c.update(family=W.MLP, layers=rng.randint(4, 32), heads=1, d=256 * _log_int(rng, 1, 32), seq=1, vocab=1,
                 batch=64 * _log_int(rng, 1, 128))
        c.update(d_ff=c["d"])
    else:
        heads = rng.choice([12, 16, 24, 32, 64, 96])
        d = heads * rng.choice([64, 80, 128])
        c.update(family=W.TRANSFORMER, layers=rng.randint(6, 96), heads=heads, d=d, d_ff=4 * d,
                 seq=128 * _log_int(rng, 1, 16), vocab=rng.choice([50257, 32000, 51200, 30522]),
                 batch=32 * _log_int(rng, 2, 48))
    return c


def draw(rng):
    kind = rng.choice(["tables", "tables", "tables", "grid", "grid", "grid", "grid", "written", "generate"])
    if kind == "tables":
        if rng.random() < 0.4:
            heads = rng.choice([12, 16])
            return _unnamed(_lowered("", _log_int(rng, 30, 1500), rng.choice([4, 8]), 64 * heads, heads,
                                     rng.choice(["default", "mi355x"]), top=rng.choice([1, 4])))
        dev = rng.randint(2, 8)
        ops = _log_int(rng, 60, 2048)
        n = _log_int(rng, 200, min(1_000_000, 1_500_000_000 // ops))
        return _unnamed(_random("", n, ops, dev, rng.random() < 0.5, top=rng.choice([1, 8])))
    if kind == "generate":
        ops = _log_int(rng, 60, 2048)
        return {"kind": kind, "n": _log_int(rng, 500, 128_000_000 // ops), "ops": ops, "n_dev": rng.randint(2, 8)}
    if kind == "written":
        # sizes whose flop and byte counts are exact in fp32, as tables need
        c = _draw_model(rng, True)
        c.update(kind=kind, layers=rng.choice([4, 6, 8]), d=rng.choice([64, 128, 256]), batch=rng.choice([32, 48, 64]),
                 elem=4, max_devices=4, k_mode=rng.choice([0, 1]), k_max=rng.choice([4, 8]), cap=0)
        c["d_ff"] = c["d"]
        return c
    mlp = rng.random() < 0.4
    c = _draw_model(rng, mlp)
    if mlp:
        c.update(kind=kind, max_devices=rng.choice([4, 8, 16, 32]), k_mode=rng.choice([0, 1, 2]),
                 k_max=_log_int(rng, 4, 64))
    else:
        c.update(kind=kind, max_devices=2 ** rng.randint(4, 10), k_mode=rng.choice([0, 1, 1, 2]),
                 k_max=_log_int(rng, 8, 256))
    return c


def _unnamed(c):
    return {k: v for k, v in c.items() if k != "name"}


# ---------------------------------------------------------------------------
# State
# ---------------------------------------------------------------------------
def _cluster(case, seed):
    """The case's device model with its rates as another calibration of the
    cluster would give them (within a few percent)."""
    rng = random.Random("rates %d" % seed)
    base = W.MI355X if case["cluster"] == "mi355x" else W.DeviceSpec()

    def near(v):
        return v * rng.uniform(0.95, 1.05)

    dev = replace(base, flops_per_s=near(base.flops_per_s), mem_bytes_per_s=near(base.mem_bytes_per_s),
                  link_bytes_per_s=near(base.link_bytes_per_s), link_latency_s=near(base.link_latency_s),
                  launch_s=near(base.launch_s), mem_cap_bytes=int(case.get("cap", 0)))
    if base.matmul:
        dev = replace(dev, matmul=tuple(near(v) for v in base.matmul),
                      network=(base.network[0], near(base.network[1]), near(base.network[2])))
    return replace(dev, streams=W.STREAMS_FREE) if case.get("overlap") else dev


def _model(case):
    return W.ModelSpec(case["family"], case["mode"], case["layers"], case["heads"], case["d"], case["d_ff"],
                       case["seq"], case["vocab"], case["batch"], case["elem"], case["schedule"], case["recompute"],
                       case["zero"], case["overlap"])


def _strategies(case):
    return dsim.dsim_create_grid(_model(case), W.GridSpec(case["max_devices"], 0, case["k_mode"], case["k_max"]))


def _selection(n, k):
    return {"k": k, "ws": torch.empty(max(dsim.dsim_argmin_workspace(n, k), 16), dtype=torch.uint8, device="cuda"),
            "idx": torch.empty(k, dtype=torch.int64, device="cuda"),
            "mk": torch.empty(k, dtype=torch.float64, device="cuda"),
            "found": torch.empty(1, dtype=torch.int32, device="cuda")}


_SIDE = []


def _side_stream():
    """One second stream for the whole program."""
    if not _SIDE:
        _SIDE.append(torch.cuda.Stream())
    return _SIDE[0]


def _prepare_random(case, seed):
    n, ops, nd = case["n"], case["ops"], case["n_dev"]
    tab = dsim.alloc_tables(n, ops)
    dsim.dsim_generate_random_tables(seed, n, ops, nd, tab)
    init = None
    if case["ragged"]:
        g = torch.Generator(device="cuda").manual_seed(seed)
        tab["n_ops"] = torch.randint(max(1, ops // 4), ops + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
        init = torch.randint(0, 64 << 30, (n, nd), generator=g, device="cuda", dtype=torch.int64)
    return tab, init, n


def _prepare_lowered(case, seed):
    rng = random.Random("programs %d" % seed)
    places = [(1, 1), (2, 2), (4, 2), (2, 4), (1, 4)]
    texts = []
    for i in range(case["n"]):
        tp, pp = places[i % len(places)]
        texts.append(programs.gpt2_layers(rng.randint(1, 16), 64 * rng.randint(1, 16), d=case["d"],
                                          heads=case["heads"], n_layers=case["layers"], tp=tp, pp=pp))
    p = frontend.lower_batch(texts, [{"%flat": [-1]}] * len(texts), n_dev=8,
                             threads=max(1, min(os.cpu_count() or 1, 16)))
    tab = {k: torch.from_numpy(np.ascontiguousarray(p[k]).view(np.int32 if p[k].dtype == np.uint32 else p[k].dtype))
           .cuda() for k in ("code", "flops", "bytes", "alloc", "free", "mm_k", "n_ops")}
    return tab, torch.from_numpy(p["init_live"].view(np.int64)).cuda(), case["n"]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "generate":
        return {"kind": kind, "case": case, "seed": seed, "tab": dsim.alloc_tables(case["n"], case["ops"])}
    s = {"kind": kind, "device": _cluster(case, seed)}
    if kind == "tables":
        s["tab"], s["init"], n = (_prepare_random if case["programs"] == "random" else _prepare_lowered)(case, seed)
        s["n"], s["n_dev"] = n, case["n_dev"]
        s["res"] = dsim.alloc_results(n, case["n_dev"])
        s["sel"] = _selection(n, case["top"])
        return s
    strat = _strategies(case)
    n = len(strat)
    s["model"], s["cand"] = _model(case), torch.from_numpy(strat).cuda()
    s["n"], s["sel"] = n, _selection(n, case["top"])
    if kind == "written":
        s["n_dev"] = 8 if case["overlap"] else 4
        s["max_ops"] = _written_ops(s)
        s["res"] = dsim.alloc_results(n, s["n_dev"])
    else:
        s["res"] = dsim.alloc_results(n, int(strat[:, 2].max()))
        s["ws"], s["side"] = dsim.alloc_parametric_workspace(n), _side_stream()
    return s


def _written_ops(s):
    """The grid's longest program, which the caller sizes its tables for."""
    res = dsim.alloc_results(s["n"], 4)
    dsim.dsim_simulate_parametric(s["model"], s["cand"], s["device"], res)
    return int(res["n_ops"].max().item())


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _select(s):
    r, q = s["res"], s["sel"]
    dsim.dsim_argmin(r["makespan"], r["cand_peak"], r["status"], s["device"].mem_cap_bytes, q["k"], q["ws"],
                     q["idx"], q["mk"], q["found"])
    out = {k: v for k, v in r.items() if k != "row_width"}
    out.update(idx=q["idx"], mk=q["mk"], found=q["found"])
    return out


def run(s):
    kind = s["kind"]
    if kind == "generate":
        c, t = s["case"], s["tab"]
        dsim.dsim_generate_random_tables(s["seed"], c["n"], c["ops"], c["n_dev"], t)
        return dict(t)
    if kind == "tables":
        dsim.dsim_simulate_tables(s["tab"], s["n"], s["n_dev"], s["device"], s["res"], init_live=s["init"])
        return _select(s)
    if kind == "written":
        tab, written = dsim.dsim_materialize_tables(s["model"], s["cand"], s["n_dev"], s["max_ops"])
        dsim.dsim_simulate_tables(tab, s["n"], s["n_dev"], s["device"], s["res"], init_live=tab["init_live"])
        out = _select(s)
        out.update(table_ops=tab["n_ops"], init_live=tab["init_live"], table_status=written)
        return out
    dsim.dsim_simulate_parametric(s["model"], s["cand"], s["device"], s["res"], workspace=s["ws"],
                                  side_stream=s["side"])
    return _select(s)


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how far another implementation may be off
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "generate":
        records = case["n"] * case["ops"]
        return {"bytes": 20 * records + 4 * case["n"], "flops": 2 * records}
    if kind == "tables":
        nd, n = case["n_dev"], case["n"]
        per = 4 + 36 + 16 * nd
        if case["programs"] == "random":
            records = n * case["ops"] * (0.625 if case["ragged"] else 1.0)
            width, per = 20, per + (8 * nd if case["ragged"] else 0)
        else:
            records = n * 34 * case["layers"]   # the mean record count of a lowered program, about
            width, per = 24, per + 8 * nd
        # an op's cost (two products, a sum) and its start and end
        return {"bytes": width * records + per * n, "flops": 5 * records}
    strat = _strategies(case)
    n, rw = len(strat), int(strat[:, 2].max())
    P, K = strat[:, 2].astype(np.float64), strat[:, 3].astype(np.float64)
    phases = 1 if case["mode"] == W.INFER else 2
    # a start and an end for every block of every stage and every Send
    flops = 2.0 * float(np.sum(phases * K * (2 * P - 1)))
    if kind == "written":
        # every record written and read once: at least a block's layers on
        # every device
        records = float(np.sum(strat[:, 0] * strat[:, 1] * phases * K * case["layers"] * 2))
        return {"bytes": 48 * records + n * (16 + 40 + 24 * 4), "flops": 5 * records}
    return {"bytes": n * (16 + 36 + 16 * rw), "flops": flops}


def tolerance(case):
    """Every result is bit-reproducible: the interface fixes the order of each
    fp64 operation, and everything else is whole numbers."""
    return "exact"


# ---------------------------------------------------------------------------
# The same results in plain torch
# ---------------------------------------------------------------------------
def _walk(tab, init, n, nd, dev):
    """Every program's ops in order, all programs at once (the semantics of the
    table format in include/dsim.h)."""
    u32, f64, i64 = 0xffffffff, torch.float64, torch.int64
    clk = torch.zeros((nd, n), dtype=f64, device="cuda")
    live = torch.zeros((nd, n), dtype=i64, device="cuda") if init is None else init.t().contiguous()
    peak, status = live.clone(), torch.zeros(n, dtype=torch.int32, device="cuda")
    ids = torch.arange(nd, device="cuda")[:, None]
    ops = tab["n_ops"].to(i64)
    S, mm, net = (dev.streams[0] if dev.streams else 1), dev.matmul, dev.network
    inv_f, inv_b, inv_l = 1.0 / dev.flops_per_s, 1.0 / dev.mem_bytes_per_s, 1.0 / dev.link_bytes_per_s
    for j in range(tab["code"].shape[0]):
        code = tab["code"][j].to(i64) & u32
        kind, a, b, cls = code & 255, (code >> 8) & 255, (code >> 16) & 255, code >> 24
        fl, by = tab["flops"][j].to(f64), tab["bytes"][j].to(f64)
        al, fr = tab["alloc"][j].to(i64) & u32, tab["free"][j].to(i64) & u32
        comp, send, ar = kind == 0, kind == 1, kind == 2
        on_a, on_b, in_mask = ids == a, ids == b, ((b >> ids) & 1) == 1
        mem = torch.where(comp, on_a, torch.where(send, on_a | on_b, in_mask)) & (j < ops)
        cnt = mem.sum(0).to(f64)
        lat, il = torch.full((n,), dev.link_latency_s, dtype=f64, device="cuda"), inv_l
        if net or S > 1:
            lo = torch.where(mem, ids, nd).amin(0) // S
            hi = torch.where(mem, ids, -1).amax(0) // S
            il = torch.full((n,), inv_l, dtype=f64, device="cuda")
            if net:
                cross = lo // net[0] != hi // net[0]
                lat, il = torch.where(cross, net[2], lat), torch.where(cross, 1.0 / net[1], il)
            if S > 1:
                lat, il = torch.where(lo == hi, dev.streams[2], lat), torch.where(lo == hi, 1.0 / dev.streams[1], il)
        cost = dev.launch_s + torch.maximum(fl * inv_f, by * inv_b)
        if mm:
            c = tuple(mm) + (0.0,) * (5 - len(mm))
            k = (tab["mm_k"][j].to(i64) & u32).to(f64) if tab.get("mm_k") is not None else 0.0
            lin = ((c[0] + c[1] * fl) + c[2] * by) + c[3] * k
            cost = torch.where(cls == 1, torch.clamp(lin, min=c[4]), cost)
        steps = 2.0 * (cnt - 1)
        ring = torch.where(cnt > 1, steps * lat + (steps / cnt) * (by * il), 0.0)
        chain = torch.where(cnt > 1, (cnt - 1) * lat + by * il, 0.0)
        cost = torch.where(comp, cost, torch.where(send, lat + by * il, torch.where(ar, ring, chain)))
        end = torch.where(mem, clk, 0.0).amax(0) + cost
        clk = torch.where(mem, end, clk)
        gets = torch.where(send, on_b, torch.where(kind == 3, ~on_a, on_a)) & mem & ~ar
        frees = torch.where(kind == 4, in_mask, on_a) & mem & ~ar
        live = live + torch.where(gets, al, 0)
        peak = torch.where(mem & ~ar, torch.maximum(peak, live), peak)
        under = frees & (fr > live)
        status |= torch.where(under.any(0), 8, 0).to(torch.int32)
        live = torch.where(under, 0, live - torch.where(frees, fr, 0))
    mk, cp = clk.amax(0), peak.amax(0)
    if dev.mem_cap_bytes:
        status |= torch.where(cp > dev.mem_cap_bytes, 32, 0).to(torch.int32)
    return {"makespan": mk, "finish": clk.t().contiguous(), "peak": peak.t().contiguous(), "cand_peak": cp,
            "n_ops": ops, "walked_ops": ops, "status": status}


def _splitmix(seed, n):
    def shr(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)

    def wrap(v):
        return v - (1 << 64) if v >= 1 << 63 else v

    z = n * wrap(0x9E3779B97F4A7C15) + seed
    z = (z ^ shr(z, 30)) * wrap(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * wrap(0x94D049BB133111EB)
    return z ^ shr(z, 31)


def _log_uniform(r, lo, hi):
    u = ((r >> 11) & ((1 << 53) - 1)).to(torch.float64) * 2.0 ** -53
    return torch.exp2(lo + u * (hi - lo))


def exact(case, seed):
    if case["kind"] == "generate":
        # flops and bytes depend on their draws alone; the codes and buffer
        # sizes are whole numbers
        n, ops = case["n"], case["ops"]
        flops = torch.empty((ops, n), dtype=torch.float64, device="cuda")
        bytes_ = torch.empty_like(flops)
        c = torch.arange(n, dtype=torch.int64, device="cuda") << 32
        for j in range(ops):
            at = c + (j * 32 + 1)
            kind = (((_splitmix(seed, at) >> 32) & 0xffffffff) * 10) >> 32
            flops[j] = torch.where(kind < 7, _log_uniform(_splitmix(seed, at + 3), LOG2_1E6, LOG2_1E12), 0.0)
            message = torch.floor(_log_uniform(_splitmix(seed, at + 7), LOG2_1E3, LOG2_1E9).to(torch.float32).double())
            bytes_[j] = torch.where((kind == 7) | (kind == 8), message,
                                    _log_uniform(_splitmix(seed, at + 4), LOG2_1E3, LOG2_1E9))
        return {"flops": flops, "bytes": bytes_, "code": None, "alloc": None, "free": None, "n_ops": None}
    if case["kind"] != "tables":
        # a strategy's program takes up to 10^8 ops to walk in plain Python;
        # the results are compared bit for bit instead
        return None
    s = prepare(case, seed)
    out = _walk(s["tab"], s["init"], s["n"], s["n_dev"], s["device"])
    rank, at = torch.where(out["status"] == 0, out["makespan"], math.inf).sort(stable=True)
    k = case["top"]
    ok = rank[:k] < math.inf
    idx = torch.full((k,), -1, dtype=torch.int64, device="cuda")
    mk = torch.full((k,), math.inf, dtype=torch.float64, device="cuda")
    m = ok.numel()
    idx[:m], mk[:m] = torch.where(ok, at[:k], -1), rank[:k]
    out.update(idx=idx, mk=mk, found=ok.sum().to(torch.int32).reshape(1))
    return out
