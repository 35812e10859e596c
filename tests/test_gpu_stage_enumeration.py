"""Stages settled by enumeration of the selections that can be optimal: one wavefront ahead of rows in global
memory, the set-up wavefront of the LDS-row kernels, and the stages these reduce.  Lists around the pool's 64 items, values
that tie (the smallest mask has to come out), items of no value, a few items that hold most of the weight, values and
weights of very different sizes, windows that hold all but a little, lists that run over.  Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


def _batch(seed, batch, n, cap, kind, m=3):
    r = np.random.Generator(np.random.PCG64(seed))
    mean = 2.0 * cap / n
    w = np.maximum(1, np.rint(r.lognormal(0.0, 0.9, size=(batch, n)) * mean / 1.5)).astype(np.int64)
    v = np.rint(w * r.uniform(1.0, 4.0, size=w.shape)).astype(np.int64)
    if kind == "free":
        v = r.integers(0, 1001, size=w.shape)                   # some items of no value
    elif kind == "alike":                                        # few kinds of items: many selections are as good
        at = r.integers(0, 4, size=w.shape)
        w, v = np.maximum(1, (mean * np.array([0.5, 0.9, 1.1, 1.4])))[at].astype(np.int64), np.array([3, 5, 6, 8])[at]
    elif kind == "rates":                                        # two rates of value, many weights
        v = w * r.integers(1, 3, size=w.shape)
    elif kind == "heavy":                                        # three items hold 85 % of the weight
        w[:, :3] = np.rint(1.9 * cap * 0.28 * r.uniform(0.9, 1.1, size=(batch, min(3, n)))) if n >= 3 else w[:, :3]
        v = np.rint(w * r.uniform(1.0, 4.0, size=w.shape)).astype(np.int64)
    elif kind == "great":                                        # values far above the weights
        v = r.integers(1, (1 << 30) // n, size=w.shape)
    elif kind == "light":                                        # and far below
        v = r.integers(1, 4, size=w.shape)
    w = np.minimum(w, cap + 3)                                   # (some fit no window)
    caps = np.maximum(1, np.rint(cap * r.uniform(0.2, 1.0, size=(batch, m)))).astype(np.int64)
    caps[0] = np.minimum(cap, w[0].sum() - 1)                    # all but one unit, all, one unit too many
    if batch > 2:
        caps[1], caps[2] = np.minimum(cap, w[1].sum()), np.minimum(cap, w[2].sum() + 1)
    kb = W._sequential(f"enumeration_{kind}_{n}_{cap}", w.astype(np.int32), v.astype(np.int32), caps.astype(np.int32))
    kb.fill_order = np.argsort(r.random((batch, m)), axis=1).astype(np.int32)
    return kb


KINDS = ["priority", "free", "alike", "rates", "heavy", "great", "light"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [1, 7, 24, 63, 64, 65, 130, 300])
def test_ahead_of_rows_in_global_memory(binding, oracle, kind, n):
    run(binding, oracle, _batch(71000 + n, 6, n, 45000, kind), max_capacity=45000)


def test_more_instances_than_compute_units(binding, oracle):
    """Shorter lists, two instances on a compute unit."""
    run(binding, oracle, _batch(72000, 300, 40, 41000, "priority", m=2), max_capacity=41000)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,cap", [(600, 1000), (130, 4000), (64, 8100), (65, 10200), (200, 13000), (60, 19900), (40, 26600), (300, 38900)])
def test_every_variant_of_rows_in_lds(binding, oracle, kind, n, cap):
    """Items times capacity on both sides of where it is tried; stages settled, reduced and left alone."""
    run(binding, oracle, _batch(73000 + cap, 6, n, cap, kind), max_capacity=cap)


@pytest.mark.parametrize("kind", ["priority", "alike", "free"])
def test_without_a_handle(binding, oracle, kind):
    import torch
    from tests.test_gpu_parity import assert_same
    kb = _batch(74000, 4, 150, 9000, kind)
    ref = oracle.solve_batch(kb, nthreads=16, cap_limit=9000)
    out = binding.solve_batch_static(binding.DeviceBatch(kb, torch.device("cuda", 0)), 9000)
    torch.cuda.synchronize()
    assert_same(kb, out, ref)


def test_faults_beside_good_instances(binding, oracle):
    kb = _batch(75000, 8, 50, 45000, "priority")
    kb.weights[1, 3] = 0
    kb.values[2, 4] = -1
    kb.capacities[3, 0] = 45001
    kb.n_items[4] = 0
    kb.n_knapsacks[5] = 0
    kb.values[6] = 2 ** 30
    kb.fill_order[7] = 0
    run(binding, oracle, kb, max_capacity=45000)


def _stages(items, caps, name):
    w, v = np.array(items, dtype=np.int64).T
    return W._sequential(name, w[None], v[None], [caps])


def _both_entry_points(binding, oracle, kb, max_capacity):
    import torch
    from tests.test_gpu_parity import assert_same
    ref = run(binding, oracle, kb, max_capacity=max_capacity)
    out = binding.solve_batch_static(binding.DeviceBatch(kb, torch.device("cuda", 0)), max_capacity)
    torch.cuda.synchronize()
    assert_same(kb, out, ref)


GREATEST = 2 ** 31 - 1


@pytest.mark.parametrize("weight", [GREATEST, GREATEST - 1, 2 ** 30, 2 ** 30 + 1, 14001, 20001])
def test_items_heavier_than_every_window(binding, oracle, weight):
    """They are never open, whatever they are worth: their weights do not add up in 32 bits, and they set no price."""
    first = [(500, 0)] * 96 + [(10, 10), (700, 300)] + [(weight, 5)] * 3
    second = [(1000, 0)] * 60 + [(weight, 9)] * 3
    _both_entry_points(binding, oracle, _stages(first, [14000], "worthless_and_too_heavy"), 14000)
    _both_entry_points(binding, oracle, _stages(second, [20000], "nothing_to_take"), 20000)
    r = np.random.Generator(np.random.PCG64(76000))
    for count in (1, 2, 4, 33):
        kb = _batch(76000 + count, 6, 150, 13000, "priority")
        for b in range(6):
            at = r.choice(150, size=count, replace=False)
            kb.weights[b, at], kb.values[b, at] = weight, r.integers(1, 1 << 22, size=count)
        _both_entry_points(binding, oracle, kb, 20000)


@pytest.mark.parametrize("kind", ["priority", "free"])
def test_windows_that_some_items_do_not_fit(binding, oracle, kind):
    """Windows from the largest to the smallest, the last ones smaller than many of the items still open."""
    kb = _batch(77000, 12, 150, 13000, kind, m=6)
    kb.capacities[:] = np.array([13000, 6000, 900, 250, 60, 15])
    kb.fill_order = None
    _both_entry_points(binding, oracle, kb, 13000)
    kb.values[:, 10:] = 0                     # what is worth something fits, or nearly, beside what is not
    _both_entry_points(binding, oracle, kb, 13000)


def test_a_stage_reduced_to_nothing_before_one_that_is_swept(binding, oracle):
    """What the first stage takes in any case is not part of the second one's answer."""
    light, close = [(10, 10000)] * 40, [(w, w - 1 - (7 * i) % 60) for i, w in enumerate(range(311, 371))]
    for caps in ([700, 340], [700, 340, 340], [700, 340, 700]):
        _both_entry_points(binding, oracle, _stages(light + close, caps, f"reduced_{len(caps)}"), 7000)
    kb = _batch(78000, 300, 100, 7000, "rates", m=4)
    _both_entry_points(binding, oracle, kb, 7000)


def _milliseconds(binding, kb, cap):
    import torch
    with binding.DeftKnapsack(max_batch=kb.batch, max_items=kb.item_stride, max_knapsacks=kb.knap_stride, max_capacity=cap, device=0) as h:
        db = h.upload(kb)
        h.solve_batch(db)
        h.set_profiling(True)
        best = np.inf
        for _ in range(3):
            h.solve_batch(db)
            torch.cuda.synchronize()
            best = min(best, h.get_profile().total_ms)
        return best


@pytest.mark.parametrize("kind", ["alike", "light", "near", "rates"])
@pytest.mark.parametrize("n,cap", [(20, 45000), (60, 60000), (100, 100000)])
def test_an_attempt_that_leads_nowhere_ends_early(binding, oracle, kind, n, cap):
    """Many selections as good as the best: bit-exact, and at most a small multiple of the time that the sweep of such a
    batch takes (values equal to weights are swept at once), where going through them took up to 75 times as long."""
    kb = _batch(79000 + n, 64, n, cap, "rates" if kind == "near" else kind, m=2)
    if kind == "near":
        kb.values[:] = kb.weights + np.random.Generator(np.random.PCG64(n)).integers(0, 3, size=kb.weights.shape)
    run(binding, oracle, kb.slice(0, 8), max_capacity=cap)
    swept = _batch(79000 + n, 64, n, cap, "priority", m=2)
    swept.values[:] = swept.weights
    took, sweep = _milliseconds(binding, kb, cap), _milliseconds(binding, swept, cap)
    print(f"{took:.3f} ms, sweep {sweep:.3f} ms", flush=True)
    assert took < 4 * sweep + 0.2


def _counted(binding, oracle, kb, cap):
    """Bit-exact against the oracle, and what the sweeps went through by the library's own counts, as a share of what they
    would without enumeration (rows in LDS), or in row cells (rows in global memory)."""
    import torch
    from tests.test_gpu_parity import assert_same
    ref = oracle.solve_batch(kb, nthreads=16, cap_limit=cap)
    with binding.DeftKnapsack(max_batch=kb.batch, max_items=kb.item_stride, max_knapsacks=kb.knap_stride, max_capacity=cap, device=0) as h:
        db = h.upload(kb)
        h.set_profiling(True)
        out = h.solve_batch(db)
        torch.cuda.synchronize()
        prof = h.get_profile()
        assert_same(kb, out, ref)
        return int(prof.streamed_row_cells) if h.info().seq_path == 3 else int(prof.swept_cell_updates) / int(ref.touched_cells.sum())


def _near(seed, n, cap):
    kb = _batch(seed, 6, n, cap, "rates")
    kb.values[:] = kb.weights + np.random.Generator(np.random.PCG64(n)).integers(0, 3, size=kb.weights.shape)
    return kb


@pytest.mark.parametrize("kind,n,cap,low,high", [
    ("priority", 200, 13000, 0.0, 0.02), ("free", 300, 38900, 0.0, 0.02), ("great", 200, 13000, 0.0, 0.02),  # settled
    ("light", 200, 13000, 0.05, 0.5), ("light", 300, 38900, 0.05, 0.5),                                      # reduced
    ("heavy", 200, 13000, 0.4, 1.0),                                                                         # not tried
    ("near", 200, 13000, 0.6, 1.0), ("rates", 300, 38900, 0.6, 1.0)])                                        # given up
def test_stages_are_settled_reduced_or_left(binding, oracle, kind, n, cap, low, high):
    kb = _near(90003, n, cap) if kind == "near" else _batch(90002, 6, n, cap, kind)
    assert low <= _counted(binding, oracle, kb, cap) <= high


def test_a_stage_is_reduced_to_nothing(binding, oracle):
    items = [(10, 10000)] * 40 + [(w, w - 1 - (7 * i) % 60) for i, w in enumerate(range(311, 371))]
    assert _counted(binding, oracle, _stages(items, [700], "nothing_left"), 7000) == 0
    assert 0 < _counted(binding, oracle, _stages(items, [700, 340], "nothing_left_then_swept"), 7000) < 0.02


@pytest.mark.parametrize("kind,settled", [("priority", True), ("great", True), ("heavy", True), ("alike", False), ("light", False), ("near", False)])
def test_long_rows_are_settled_or_streamed(binding, oracle, kind, settled):
    kb = _near(90003, 148, 45000) if kind == "near" else _batch(90001, 6, 148, 45000, kind)
    assert (_counted(binding, oracle, kb, 45000) == 0) == settled
