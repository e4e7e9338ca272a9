"""GPU parity of the table materialiser: each strategy's whole distributed
program (every op of every device) written as explicit op tables by
dsim_materialize_tables and simulated by dsim_simulate_tables, against the
oracle's full-program simulation (times within 1e-12 relative and expected
bit-identical; op counts, peaks and status exact) and against the
parametric path on the same strategies."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2111_05426_amd.workloads import (DeviceSpec, INFER, SCHED_GPIPE, TINY_MLP, TRAIN_ADAM, TRAIN_ADAM_MIXED,
                                            TRAIN_SGD,
                                            mlp, transformer)

pytestmark = pytest.mark.gpu
REL = 1e-12
ST_BAD_STRATEGY, ST_NOT_TABLE = 16, 64


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_05426_amd import dsim
    dsim.lib()
    return torch


def materialize_and_simulate(torch, model, strat, dev, n_dev, max_ops):
    from paper_2111_05426_amd import dsim
    cand = torch.from_numpy(np.ascontiguousarray(strat, np.int32)).cuda()
    t, mst = dsim.dsim_materialize_tables(model, cand, n_dev, max_ops)
    r = dsim.alloc_results(len(strat), n_dev)
    dsim.dsim_simulate_tables(t, len(strat), n_dev, dev, r, init_live=t["init_live"])
    torch.cuda.synchronize()
    out = {k: v.cpu().numpy() for k, v in r.items() if k != "row_width"}
    out["mat_status"] = mst.cpu().numpy()
    out["table_ops"] = t["n_ops"].cpu().numpy().astype(np.int64)
    out["init_live"] = t["init_live"].cpu().numpy()
    out["gpu"] = r
    return out


def check_against_oracle(g, o, strat, n_dev):
    ok = o["status"] == 0
    assert np.array_equal(g["mat_status"][ok], np.zeros(ok.sum(), np.int32))
    assert np.array_equal(g["status"][ok], np.zeros(ok.sum(), np.int32))
    assert np.array_equal(g["table_ops"][ok], o["n_ops"][ok].astype(np.int64))
    np.testing.assert_allclose(g["makespan"][ok], o["makespan"][ok], rtol=REL, atol=0)
    assert np.array_equal(g["makespan"][ok], o["makespan"][ok])
    assert np.array_equal(g["cand_peak"][ok].view(np.uint64), o["cand_peak"][ok])
    for i in np.nonzero(ok)[0]:
        D, H, P, K = (int(v) for v in strat[i])
        dh = D * H
        fin, pk = g["finish"][i], g["peak"][i].view(np.uint64)
        for p in range(P):
            # every replica of a stage ends at the stage's time with its peak
            assert np.all(fin[p * dh:(p + 1) * dh] == o["finish"][i, p]), (strat[i], p)
            assert np.all(pk[p * dh:(p + 1) * dh] == o["peak"][i, p]), (strat[i], p)
        assert np.all(fin[P * dh:] == 0.0) and np.all(pk[P * dh:] == 0)


def all_strats(D, H, P, K, n_dev):
    return np.array([(d, h, p, k) for d in D for h in H for p in P for k in K if d * h * p <= n_dev], np.int32)


def test_tiny_mlp_grid_as_tables(torch_gpu, orc):
    """The tiny MLP grid (30 strategies on <= 4 devices) as explicit tables of
    a few hundred ops each."""
    from paper_2111_05426_amd import dsim
    w = TINY_MLP
    strat = dsim.dsim_create_grid(w.model, w.grid)
    assert len(strat) == 30
    o = orc.run_strategies(w.model, strat, w.device, slice=False, row_width=int(strat[:, 2].max()), threads=8)
    assert np.all(o["status"] == 0)
    max_ops = int(o["n_ops"].max())
    assert 100 <= max_ops <= 2000
    g = materialize_and_simulate(torch_gpu, w.model, strat, w.device, 4, max_ops)
    check_against_oracle(g, o, strat, 4)
    # the same programs through the transform-driven kernel
    rp = dsim.alloc_results(len(strat), int(strat[:, 2].max()))
    dsim.dsim_simulate_parametric(w.model, torch_gpu.from_numpy(strat).cuda(), w.device, rp)
    torch_gpu.cuda.synchronize()
    assert np.array_equal(rp["makespan"].cpu().numpy(), g["makespan"])
    assert np.array_equal(rp["n_ops"].cpu().numpy().astype(np.int64), g["table_ops"])
    # selection over the table results
    idx, mk, found = dsim.select_topk(g["gpu"]["makespan"], g["gpu"]["cand_peak"], g["gpu"]["status"],
                                      w.device.mem_cap_bytes, 3)
    ri, rm, rf = orc.topk(o["makespan"], o["cand_peak"], o["status"], w.device.mem_cap_bytes, 3)
    torch_gpu.cuda.synchronize()
    assert int(found.item()) == rf and np.array_equal(idx.cpu().numpy(), ri)


CASES = [
    ("mlp_sgd", mlp(4, 64, 48, 4, TRAIN_SGD), all_strats([1, 2], [1, 2], [1, 2, 4], [1, 2, 3, 5], 8)),
    ("mlp_adam_uneven", mlp(6, 64, 40, 2, TRAIN_ADAM), all_strats([1, 2], [1, 2], [1, 2, 3], [1, 3, 7], 8)),
    ("mlp_infer", mlp(5, 64, 30, 4, INFER), all_strats([1, 2, 3], [1, 2], [1, 2], [1, 2, 4], 8)),
    ("tf_train", transformer(4, 32, 4, 8, 101, 12, 2, TRAIN_ADAM), all_strats([1, 2], [1, 2, 4], [1, 2], [1, 2, 5], 8)),
    ("tf_mixed", transformer(3, 32, 4, 8, 64, 8, 2, TRAIN_ADAM_MIXED), all_strats([1, 2], [1, 2], [1, 3], [1, 4], 8)),
    ("tf_infer", transformer(4, 48, 6, 16, 97, 9, 2, INFER), all_strats([1, 3], [1, 2], [1, 2, 4], [1, 3], 8)),
    ("mlp_gpipe", mlp(6, 64, 40, 2, TRAIN_ADAM, schedule=SCHED_GPIPE), all_strats([1, 2], [1, 2], [1, 2, 3], [1, 3, 7], 8)),
    ("tf_gpipe", transformer(4, 32, 4, 8, 101, 12, 2, TRAIN_ADAM, schedule=SCHED_GPIPE),
     all_strats([1, 2], [1, 2, 4], [1, 2], [1, 2, 5], 8)),
    ("mlp_recompute", mlp(8, 64, 40, 2, TRAIN_ADAM, recompute=1), all_strats([1, 2], [1, 2], [1, 2, 3], [1, 3, 7], 8)),
    ("tf_recompute", transformer(4, 32, 4, 8, 101, 12, 2, TRAIN_ADAM_MIXED, recompute=1),
     all_strats([1, 2], [1, 2, 4], [1, 2], [1, 2, 5], 8)),
    ("tf_gpipe_recompute", transformer(5, 32, 4, 8, 101, 12, 2, TRAIN_ADAM, schedule=SCHED_GPIPE, recompute=1),
     all_strats([1, 2], [1, 2], [1, 2, 3], [1, 3], 8)),
]
# empirical MatMul cost: matrix multiplications are class-1 records, their
# reduction lengths in the materialised mm_k array
MM = (6.1e-6, 2.3e-14, 7.7e-13, 3.1e-9, 2.2e-5)


ZERO_CASES = [
    ("mlp_zero", mlp(4, 64, 48, 4, TRAIN_ADAM, zero=1), all_strats([2, 3, 4, 8], [1, 2], [1, 2], [1, 2, 3], 8)),
    ("mlp_zero_sgd_rc", mlp(6, 32, 48, 2, TRAIN_SGD, recompute=1, zero=1),
     all_strats([2, 4], [1, 2], [1, 3], [1, 2, 5], 8)),
    ("tf_zero", transformer(4, 32, 4, 8, 101, 12, 2, TRAIN_ADAM, zero=1), all_strats([2, 3, 4], [1, 2], [1, 2], [1, 2, 3], 8)),
    ("tf_zero_mixed_gpipe", transformer(3, 32, 4, 8, 64, 8, 2, TRAIN_ADAM_MIXED, schedule=SCHED_GPIPE, zero=1),
     all_strats([2, 4], [1, 2], [1, 2, 3], [1, 2], 8)),
    ("tf_zero_rc", transformer(5, 32, 4, 8, 101, 12, 2, TRAIN_ADAM, recompute=1, zero=1),
     all_strats([2, 3], [1, 2], [1, 2], [1, 3], 8)),
]


@pytest.mark.parametrize("case", ZERO_CASES, ids=[c[0] for c in ZERO_CASES])
def test_zero_programs_as_tables(torch_gpu, orc, case):
    """ZeRO programs hold broadcast and reduce records; their data replicas
    own different parameter groups, so finish times, peaks and resident
    bytes are compared device by device with the oracle's full program."""
    name, model, strat = case
    dev = DeviceSpec(mem_cap_bytes=10 ** 6)
    o = orc.run_strategies(model, strat, dev, slice=False, row_width=int(strat[:, 2].max()), threads=8)
    assert np.all(o["status"] == 0)
    g = materialize_and_simulate(torch_gpu, model, strat, dev, 8, int(o["n_ops"].max()))
    assert np.all(g["mat_status"] == 0) and np.all(g["status"] == 0)
    assert np.array_equal(g["table_ops"], o["n_ops"].astype(np.int64))
    assert np.array_equal(g["makespan"], o["makespan"])
    assert np.array_equal(g["cand_peak"].view(np.uint64), o["cand_peak"])
    differ = 0
    for i, (D, H, P, K) in enumerate(strat.tolist()):
        r = orc.sim_strategy(model, D, H, P, K, dev)
        n = D * H * P
        assert np.array_equal(g["finish"][i, :n], r["dev_finish"]), (name, strat[i].tolist())
        assert np.array_equal(g["peak"][i, :n].view(np.uint64), r["dev_peak"]), (name, strat[i].tolist())
        assert np.array_equal(g["init_live"][i, :n].view(np.uint64), r["dev_resident"]), (name, strat[i].tolist())
        differ += len(set(r["dev_peak"][:D * H].tolist())) > 1
    assert differ > 0   # the replicas really differ somewhere


@pytest.mark.parametrize("mm", ["roofline", "matmul", "network"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_small_programs_as_tables(torch_gpu, orc, case, mm):
    name, model, strat = case
    dev = DeviceSpec(mem_cap_bytes=10 ** 6, matmul=MM if mm == "matmul" else None,
                     network=(2, 4.7e9, 1.9e-5) if mm == "network" else None)
    o = orc.run_strategies(model, strat, dev, slice=False, row_width=int(strat[:, 2].max()), threads=8)
    assert np.any(o["status"] == 0)
    g = materialize_and_simulate(torch_gpu, model, strat, dev, 8, int(o["n_ops"].max()))
    check_against_oracle(g, o, strat, 8)
    # invalid strategies are flagged by the materialiser itself (node
    # placement is a precondition of the transform-driven simulation only:
    # tables carry device ids and simulate any placement)
    if mm == "network":
        o = orc.run_strategies(model, strat, replace(dev, network=None), slice=False,
                               row_width=int(strat[:, 2].max()), threads=8)
    bad = o["status"] & ST_BAD_STRATEGY != 0
    assert np.all(g["mat_status"][bad] == ST_BAD_STRATEGY) and np.all(g["table_ops"][bad] == 0)


OV_CASES = [
    ("mlp_ov", mlp(4, 64, 48, 4, TRAIN_ADAM, overlap=1), all_strats([1, 2, 4], [1, 2], [1, 2], [1, 2, 3], 4)),
    ("mlp_ov_gpipe_rc", mlp(6, 32, 48, 2, TRAIN_SGD, schedule=SCHED_GPIPE, recompute=1, overlap=1),
     all_strats([1, 2], [1, 2], [1, 3], [1, 2, 5], 4)),
    ("tf_ov", transformer(4, 32, 4, 8, 101, 12, 2, TRAIN_ADAM_MIXED, overlap=1),
     all_strats([1, 2, 3, 4], [1, 2], [1, 2], [1, 2, 3], 4)),
    ("tf_ov_rc", transformer(5, 32, 4, 8, 101, 12, 2, TRAIN_ADAM, recompute=1, overlap=1),
     all_strats([1, 2], [1, 2], [1, 2], [1, 3], 4)),
    ("tf_ov_infer", transformer(4, 48, 6, 16, 97, 9, 2, INFER, overlap=1), all_strats([1, 3], [1, 2], [1, 2], [1, 3], 4)),
]


@pytest.mark.parametrize("net", [False, True, "overflow"])
@pytest.mark.parametrize("case", OV_CASES, ids=[c[0] for c in OV_CASES])
def test_overlap_programs_as_tables(torch_gpu, orc, case, net):
    """Overlapped programs put two streams on every GPU (devices 2g and
    2g + 1, hand-overs as Sends between them): device by device against the
    oracle's full program, and per stage against the transform-driven
    kernel."""
    from paper_2111_05426_amd import dsim
    name, model, strat = case
    dev = DeviceSpec(streams=(2, 5.3e11, 1.7e-6), network=(1, 4.7e9, 1.9e-5) if net else None)
    if net == "overflow":   # every tier so slow that some clocks overflow to +inf
        dev = DeviceSpec(1e-301, 1e-301, 2e-303, 1e-6, 0.0, 0, streams=(2, 2e-303, 0.0), network=(1, 3e-303, 1.9e-5))
    P = int(strat[:, 2].max())
    o = orc.run_strategies(model, strat, dev, slice=False, row_width=P, threads=8)
    assert np.all(o["status"] == 0)
    g = materialize_and_simulate(torch_gpu, model, strat, dev, 8, int(o["n_ops"].max()))
    assert np.all(g["mat_status"] == 0) and np.all(g["status"] == 0)
    assert np.array_equal(g["table_ops"], o["n_ops"].astype(np.int64))
    assert np.array_equal(g["makespan"], o["makespan"])
    assert np.array_equal(g["cand_peak"].view(np.uint64), o["cand_peak"])
    for i, (D, H, Pi, K) in enumerate(strat.tolist()):
        r = orc.sim_strategy(model, D, H, Pi, K, dev)
        n = 2 * D * H * Pi
        assert np.array_equal(g["finish"][i, :n], r["dev_finish"]), (name, strat[i].tolist())
        assert np.array_equal(g["peak"][i, :n].view(np.uint64), r["dev_peak"]), (name, strat[i].tolist())
        assert np.array_equal(g["init_live"][i, :n].view(np.uint64), r["dev_resident"]), (name, strat[i].tolist())
        assert not g["peak"][i, 1:n:2].any()   # communication streams hold nothing
    rp = dsim.alloc_results(len(strat), P)
    dsim.dsim_simulate_parametric(model, torch_gpu.from_numpy(strat).cuda(), dev, rp)
    torch_gpu.cuda.synchronize()
    assert np.array_equal(rp["makespan"].cpu().numpy(), g["makespan"])
    assert np.array_equal(rp["finish"].cpu().numpy(), o["finish"])
    assert np.array_equal(rp["n_ops"].cpu().numpy().astype(np.int64), g["table_ops"])


def test_materialize_errors(torch_gpu, orc):
    m = mlp(4, 64, 48, 4, TRAIN_SGD)
    dev = DeviceSpec()
    strat = np.array([(2, 2, 4, 1),     # 16 devices > n_dev = 8
                      (1, 1, 2, 2),     # fine, but more ops than max_ops below
                      (1, 1, 1, 1)], np.int32)
    o = orc.run_strategies(m, strat[1:], dev, slice=False, row_width=2, threads=1)
    small = int(o["n_ops"][1])              # enough for (1,1,1,1) only
    assert int(o["n_ops"][0]) > small
    g = materialize_and_simulate(torch_gpu, m, strat, dev, 8, small)
    assert list(g["mat_status"]) == [ST_BAD_STRATEGY, ST_NOT_TABLE, 0]
    assert list(g["table_ops"]) == [0, 0, small]
    assert g["makespan"][2] == o["makespan"][1]
    # a FLOP count that needs more than 24 significant bits
    odd = mlp(2, 4097, 8, 4, INFER)
    g = materialize_and_simulate(torch_gpu, odd, np.array([(1, 1, 1, 1)], np.int32), dev, 8, 64)
    assert list(g["mat_status"]) == [ST_NOT_TABLE] and g["table_ops"][0] == 0


# A wavefront lists a schedule's blocks and Sends and writes 64 of them at a
# time: programs of fewer and of many more than 64, one and eight stages, and
# tables too short for them.
@pytest.mark.parametrize("option", ["plain", "gpipe", "recompute", "zero", "overlap"])
@pytest.mark.parametrize("family", ["mlp", "tf"])
def test_long_schedules(torch_gpu, orc, family, option):
    kw = {"gpipe": dict(schedule=SCHED_GPIPE), "plain": {}}.get(option, {option: 1})
    model = mlp(8, 64, 96, 2, TRAIN_ADAM, **kw) if family == "mlp" else transformer(8, 32, 4, 8, 64, 96, 2, TRAIN_ADAM, **kw)
    n_dev = 8
    strat = all_strats([1, 2], [1, 2], [1, 2, 4, 8], [1, 2, 31, 32, 48], 4 if option == "overlap" else 8)
    dev = DeviceSpec(streams=(2, float("inf"), 0.0)) if option == "overlap" else DeviceSpec()
    o = orc.run_strategies(model, strat, dev, slice=False, row_width=8, threads=8)
    ok = o["status"] == 0
    assert np.any(ok)
    strat, o = strat[ok], {k: v[ok] for k, v in o.items()}
    max_ops = int(o["n_ops"].max())
    g = materialize_and_simulate(torch_gpu, model, strat, dev, n_dev, max_ops)
    assert np.array_equal(g["mat_status"], np.zeros(len(strat), np.int32))
    assert np.array_equal(g["table_ops"], o["n_ops"].astype(np.int64))
    assert np.array_equal(g["makespan"], o["makespan"])
    assert np.array_equal(g["cand_peak"].view(np.uint64), o["cand_peak"])
    # one record too few for the longest program: that one does not fit, the others do
    g = materialize_and_simulate(torch_gpu, model, strat, dev, n_dev, max_ops - 1)
    assert np.array_equal(g["mat_status"] == ST_NOT_TABLE, o["n_ops"] == max_ops)


# Many short programs are written by eight lanes each (tables of at most 512
# rows for more than 8,192 candidates), the others by a wavefront each, with
# neighbours kept on one XCD: the same words as a small call writes, which the
# tests above compare with the oracle.
@pytest.mark.parametrize("max_ops", [511, 512, 513])
@pytest.mark.parametrize("option", ["plain", "gpipe", "recompute", "zero", "overlap", "infer"])
@pytest.mark.parametrize("family", ["mlp", "tf"])
def test_many_programs(torch_gpu, family, option, max_ops):
    from paper_2111_05426_amd import dsim
    torch = torch_gpu
    kw = {"gpipe": dict(schedule=SCHED_GPIPE), "plain": {}, "infer": {}}.get(option, {option: 1})
    mode = INFER if option == "infer" else TRAIN_ADAM
    model = mlp(8, 64, 96, 2, mode, **kw) if family == "mlp" else transformer(4, 32, 4, 8, 64, 96, 2, mode, **kw)
    n_dev = 8
    # programs that fit, that do not, and strategies with too many devices,
    # stages or microbatches
    strat = np.array([(d, h, p, k) for d in (1, 2, 3, 5, 8) for h in (1, 2, 4) for p in (1, 2, 4, 8)
                      for k in (1, 2, 5, 12, 97)], np.int32)

    def tables(rows):
        t, status = dsim.dsim_materialize_tables(model, torch.from_numpy(np.ascontiguousarray(rows)).cuda(), n_dev, max_ops)
        torch.cuda.synchronize()
        return t, status

    t0, st0 = tables(strat)
    seen = set(st0.cpu().numpy().tolist())
    assert {0, ST_BAD_STRATEGY} <= seen and (ST_NOT_TABLE in seen or option == "infer")
    at = np.random.default_rng(7).permutation(np.arange(8193 + 70) % len(strat))
    at[1000:1100] = at[1000]            # equal neighbours too
    for n in (8193, len(at)):
        pick = torch.from_numpy(at[:n]).cuda()
        t, st = tables(strat[at[:n]])
        assert torch.equal(st, st0[pick])
        assert torch.equal(t["n_ops"], t0["n_ops"][pick]) and torch.equal(t["init_live"], t0["init_live"][pick])
        live = torch.arange(max_ops, device="cuda")[:, None] < t["n_ops"][None, :]
        for k in ("code", "flops", "bytes", "alloc", "free", "mm_k"):
            a, b = t[k].view(torch.int32), t0[k].view(torch.int32)[:, pick]
            assert torch.equal(torch.where(live, a, 0), torch.where(live, b, 0)), k
