"""Ranges of a call's size in which it must not fall behind: each test compares
two times of the same library on the same card, with a wide margin on either
side (the figures in the docstrings are an MI355X's)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2111_05426_amd import dsim
    dsim.lib()
    return torch


def call_us(torch, call, reps=20, runs=7):
    """The least mean time of a call among `reps` in a row."""
    call()
    best = np.inf
    for _ in range(runs):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / reps)
    return best


def selection(torch, n, k):
    from paper_2111_05426_amd import dsim
    g = torch.Generator(device="cuda").manual_seed(n)
    mk = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    pk = torch.zeros(n, dtype=torch.int64, device="cuda")
    st = torch.zeros(n, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(dsim.dsim_argmin_workspace(n, k), 16), dtype=torch.uint8, device="cuda")
    idx = torch.empty(k, dtype=torch.int64, device="cuda")
    out = torch.empty(k, dtype=torch.float64, device="cuda")
    found = torch.empty(1, dtype=torch.int32, device="cuda")
    return lambda: dsim.dsim_argmin(mk, pk, st, 0, k, ws, idx, out, found)


def test_selection_around_one_block(torch_gpu):
    """1,024 keys cost about what 1,025 do (15 us; counted in one block they
    took 43)."""
    small, more = (call_us(torch_gpu, selection(torch_gpu, n, 4)) for n in (1024, 1025))
    print("top-4 of 1,024: %.1f us, of 1,025: %.1f us" % (small, more))
    assert small < 1.8 * more


def test_selection_of_many_keys(torch_gpu):
    """Sixteen times the keys cost far less than sixteen times as much (52 and
    291 us; 1,352 with at most 512 blocks of 256 threads)."""
    few, many = (call_us(torch_gpu, selection(torch_gpu, n, 16), 5) for n in (1_000_000, 16_000_000))
    print("top-16 of a million: %.1f us, of 16 million: %.1f us" % (few, many))
    assert many < 12 * few


@pytest.mark.parametrize("name", ["equal", "grid"])
def test_materialize_many_programs(torch_gpu, name):
    """64,000 programs are written in a small multiple of the time of filling
    their words: equal ones of 108 records 6 times (139 us; 29 times with a
    wavefront each), a grid of 465 records on average 18 times (1.8 ms; 39
    times with neighbours on different XCDs)."""
    from paper_2111_05426_amd import dsim
    from paper_2111_05426_amd.workloads import GridSpec, TRAIN_SGD, mlp
    torch = torch_gpu
    n, model = 64_000, mlp(4, 256, 512, 4, TRAIN_SGD)
    grid = dsim.dsim_create_grid(model, GridSpec(8, 0, 1, 8))
    strat = grid[np.arange(n) % len(grid)] if name == "grid" else np.tile(np.array([[2, 1, 1, 2]], np.int32), (n, 1))
    cand = torch.from_numpy(np.ascontiguousarray(strat)).cuda()
    rows = 1720 if name == "grid" else 110
    t, status = dsim.dsim_materialize_tables(model, cand, 8, rows)
    assert not status.any()
    words = 6 * int(t["n_ops"].long().sum().item())
    del t
    fill = torch.empty(words, dtype=torch.int32, device="cuda")
    base = call_us(torch, lambda: fill.fill_(1), 10)
    took = call_us(torch, lambda: dsim.dsim_materialize_tables(model, cand, 8, rows), 3, 5)
    print("%s: %d words, filled in %.1f us, written in %.1f us" % (name, words, base, took))
    assert took < (28 if name == "grid" else 14) * base


@pytest.mark.parametrize("family,k_max", [("mlp", 4), ("mlp", 64), ("tf", 4), ("tf", 64)])
def test_many_strategies_of_few_stages(torch_gpu, family, k_max):
    """100,000 strategies of one stage take far less than as many of sixteen
    (up to 4 microbatches: MLP 50 us, transformer 63; up to 64: 93 and 138; with
    sixteen lanes each 389, 480, 583 and 687, as long as of sixteen stages)."""
    from paper_2111_05426_amd import dsim
    from paper_2111_05426_amd.workloads import DeviceSpec, TRAIN_ADAM, TRAIN_ADAM_MIXED, mlp, transformer
    torch = torch_gpu
    model = mlp(16, 1024, 8192, 2, TRAIN_ADAM) if family == "mlp" else transformer(24, 1024, 16, 1024, 50257, 4096, 2, TRAIN_ADAM_MIXED)
    n, took = 100_000, {}
    for P in (1, 16):
        grid = np.array([(D, H, P, K) for K in range(1, k_max + 1) for H in (1, 2) for D in (1, 2, 4, 8, 16, 32, 64)
                         if P == 1 or H == 1 or family == "tf"], np.int32)
        cand = torch.from_numpy(np.ascontiguousarray(grid[(np.arange(n) * len(grid)) // n])).cuda()
        r, ws = dsim.alloc_results(n, P), dsim.alloc_parametric_workspace(n)
        took[P] = call_us(torch, lambda: dsim.dsim_simulate_parametric(model, cand, DeviceSpec(), r, workspace=ws), 5, 5)
        assert not (r["status"] != 0).any()
    print("%s, K <= %d: one stage %.1f us, sixteen %.1f us" % (family, k_max, took[1], took[16]))
    assert took[1] < 0.5 * took[16]
