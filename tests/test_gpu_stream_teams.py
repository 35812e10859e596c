"""Few instances on long rows: the compute units that the batch leaves idle help with the items of an
instance, a tile of its band at a time.  Sizes around a tile, more tiles than helpers and the
reverse, items by the team and passes by the owner alone in turn, instances that dismiss their helpers.
Bit-exact against the oracle, several calls in a row (the second finds what the first left behind)."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import assert_same, binding  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


def _batch(seed, batch, n, draw_w, caps, mode=W.MODE_SEQUENTIAL):
    r = np.random.Generator(np.random.PCG64(seed))
    w = np.asarray(draw_w(r, (batch, n)), np.int32)
    v = r.integers(0, 5000, size=(batch, n)).astype(np.int32)       # some items of no value
    kb = W._sequential(f"teams_{seed}", w, v, np.tile(np.array([caps], np.int32), (batch, 1)))
    kb.mode = mode
    return kb


def _run(binding, oracle, kb, max_capacity, calls=2):
    import torch
    print(f"case {kb.name} batch={kb.batch} n={kb.item_stride} max_capacity={max_capacity}", flush=True)
    ref = oracle.solve_batch(kb, nthreads=16, cap_limit=max_capacity)
    with binding.DeftKnapsack(max_batch=kb.batch, max_items=kb.item_stride, max_knapsacks=kb.knap_stride,
                              max_capacity=max_capacity) as h:
        db = h.upload(kb)
        for _ in range(calls):
            out = h.solve_batch(db)
            torch.cuda.synchronize()
            assert_same(kb, out, ref)


@pytest.mark.parametrize("cap", [131071, 131072, 139263, 139264, 139265, 163840])
@pytest.mark.parametrize("batch", [1, 7, 8, 100, 128, 129])
def test_tiles_and_helpers(binding, oracle, cap, batch):
    """Heavy items (each its own job) and mixed ones, from 255 helpers an instance to none."""
    heavy = lambda r, s: r.integers(36000, 90000, size=s)  # noqa: E731
    mixed = lambda r, s: np.where(r.random(s) < 0.2, r.integers(36000, 60000, size=s), r.integers(1, 12000, size=s))  # noqa: E731
    _run(binding, oracle, _batch(51000 + cap + batch, batch, 9, heavy, [cap, cap // 3]), cap)
    _run(binding, oracle, _batch(52000 + cap + batch, min(batch, 8), 18, mixed, [cap // 2, cap]), cap)


@pytest.mark.parametrize("cap,n", [(139999, 20), (139999, 21), (260095, 40), (260096, 40), (262143, 40), (262144, 40)])
def test_which_rows_get_helpers(binding, oracle, cap, n):
    """Both sides of 7000 cells per item and of 262144 cells."""
    _run(binding, oracle, _batch(53500 + cap + n, 3, n, lambda r, s: r.integers(1, 4 * cap // n, size=s), [cap, cap * 2 // 5]), cap)


@pytest.mark.parametrize("batch,cap", [(1, 2200000), (1, 2097151), (1, 2097152), (5, 600000), (16, 400000)])
def test_long_rows(binding, oracle, batch, cap):
    """More tiles than helpers; every width of band on the way; light items that passes serve."""
    for seed, share, n in ((1, 0.5, 14), (2, 0.9, 30)):
        _run(binding, oracle, _batch(53000 + batch + seed, batch, n, lambda r, s: r.integers(1, int(2 * cap / share / n), size=s).clip(1, cap),
                                     [cap, cap * 2 // 5]), cap)


def test_capacity_sweeps(binding, oracle):
    for seed, w_hi in ((1, 20000), (2, 150000)):
        _run(binding, oracle, _batch(54000 + seed, 3, 20, lambda r, s: r.integers(1, w_hi, size=s), [100000, 300000, 299999, 150000, 1],
                                     W.MODE_CAPACITY_SWEEP), 300000)


def test_instances_that_need_no_team(binding, oracle):
    """Faulty ones, settled ones, short windows on a handle for long ones, no items at all."""
    kb = _batch(55000, 8, 20, lambda r, s: r.integers(1, 60000, size=s), [200000, 90000])
    kb.weights[1, 3] = 0
    kb.capacities[2, 0] = 200001
    kb.weights[3] = 100
    kb.capacities[4] = [30000, 131071]
    kb.n_items[5] = 0
    kb.n_knapsacks[6] = 0
    _run(binding, oracle, kb, 200000, calls=3)


def test_replays_of_a_captured_call(binding, oracle):
    """The team's words are cleared by the call itself, so a replay finds them as the first run did."""
    import torch
    kb = _batch(56000, 2, 16, lambda r, s: r.integers(1, 60000, size=s), [150000, 70000])
    ref = oracle.solve_batch(kb, nthreads=16, cap_limit=150000)
    with binding.DeftKnapsack(max_batch=2, max_items=16, max_knapsacks=2, max_capacity=150000) as h:
        db = h.upload(kb)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            out = h.solve_batch(db, stream)
            stream.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                out = h.solve_batch(db, stream)
        for _ in range(3):
            out.total_value.zero_()
            out.assignment.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert_same(kb, out, ref)


def test_two_teams_on_two_streams_at_once(binding, oracle):
    import torch
    kbs = [_batch(57000 + i, 2, 16, lambda r, s: r.integers(1, 60000, size=s), [150000, 70000]) for i in range(2)]
    refs = [oracle.solve_batch(kb, nthreads=16, cap_limit=150000) for kb in kbs]
    streams = [torch.cuda.Stream() for _ in kbs]
    handles = [binding.DeftKnapsack(max_batch=2, max_items=16, max_knapsacks=2, max_capacity=150000) for _ in kbs]
    dbs = [h.upload(kb) for h, kb in zip(handles, kbs)]
    torch.cuda.synchronize()
    for _ in range(3):
        outs = [h.solve_batch(db, st) for h, db, st in zip(handles, dbs, streams)]
    torch.cuda.synchronize()
    for kb, out, ref in zip(kbs, outs, refs):
        assert_same(kb, out, ref)
    for h in handles:
        h.close()
