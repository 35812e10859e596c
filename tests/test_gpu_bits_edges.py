"""The bit-set kernels where they can go wrong: list lengths around a block of four items, a
register of 64 and the plane counts' limits; capacities around a register slot; runs of taken items
longer than a wavefront; batches that fill workgroups of several instances unevenly.  Bit-exact
against the oracle."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu

FLAG = 2   # DEFT_FLAG_SUBSET_SUM


def _sequential(seed, batch, n, w_hi, caps):
    r = np.random.Generator(np.random.PCG64(seed))
    w = r.integers(1, w_hi + 1, size=(batch, n)).astype(np.int32)
    cap = np.tile(np.array([caps], np.int32), (batch, 1))
    kb = W._sequential(f"edges_{seed}", w, w.copy(), cap)
    return kb


@pytest.mark.parametrize("n", [1, 3, 4, 5, 6, 7, 8, 9, 63, 64, 65, 66, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024])
def test_list_lengths(binding, oracle, n):
    """Two windows whose capacity the list reaches early, late or not at all."""
    for seed, share in ((1, 2), (2, 1)):
        cap = min(8000, max(3, 30 * n // share))
        run(binding, oracle, _sequential(31000 + 10 * n + seed, 9, n, 60, [cap, max(1, cap // 3)]), flags=FLAG)


@pytest.mark.parametrize("cap", [1, 31, 32, 33, 2046, 2047, 2048, 2049, 4095, 4096, 6143, 6144, 14335, 14336, 20479, 20480])
def test_capacities_around_a_slot(binding, oracle, cap):
    """Light items, items of a word and of a slot, items as heavy as the window."""
    for seed, w_hi in ((1, max(1, cap // 20)), (2, cap)):
        run(binding, oracle, _sequential(32000 + 10 * cap + seed, 7, 70, w_hi, [cap, max(1, cap - 1)]), flags=FLAG)


def test_items_of_whole_words_and_slots(binding, oracle):
    """Shifts of 32 k and 2048 k cells and their neighbours."""
    w = np.array([[32, 64, 2048, 31, 33, 2047, 2049, 4096, 1, 96, 1024, 6144, 63, 65, 2016, 2080]], np.int32)
    for cap in (2048, 6000, 9999, 14335):
        kb = W._sequential(f"whole_words_{cap}", np.tile(w, (3, 1)), np.tile(w, (3, 1)), [[cap, cap // 2]] * 3)
        run(binding, oracle, kb, flags=FLAG)


def test_long_runs_of_taken_items(binding, oracle):
    """Equal weights: the walk takes every item of the front, in runs beyond 64 lanes; one light
    item in between breaks a run."""
    w = np.full((4, 400), 25, np.int32)
    w[1, 200] = 3
    w[2, ::97] = 7
    w[3, 5] = 1
    kb = W._sequential("runs", w, w.copy(), [[5000, 4000]] * 4)
    run(binding, oracle, kb, flags=FLAG)
    kb = W._sequential("runs_short_of_the_capacity", w, w.copy(), [[5024, 4011]] * 4)
    run(binding, oracle, kb, flags=FLAG)


@pytest.mark.parametrize("batch", [1, 257, 2049, 4099])
def test_uneven_workgroups(binding, oracle, batch):
    kb = W.random_sequential(33000 + batch, batch=batch, n_max=30, m_max=3, w_hi=60, v_hi=9, cap_hi=700, ties=True)
    run(binding, oracle, kb, flags=FLAG)
    kc = W.random_capacity_sweep(33500 + batch, batch=min(batch, 300), n_max=90, m_max=5, w_hi=60, v_hi=9, cap_hi=2500, ties=True)
    run(binding, oracle, kc, flags=FLAG)


@pytest.mark.parametrize("mode", ["sequential", "algorithm1", "capacities"])
def test_short_lists_on_a_handle_for_long_ones(binding, oracle, mode):
    """The kernel goes by the call's lists: the same outputs, and about as fast, as on a handle for lists no longer (with
    the kernels of the longer lists 1.13 to 1.41 times as long)."""
    import torch
    r = np.random.Generator(np.random.PCG64(34000))
    B, n, cap = 8192, 80, 12000
    x = r.lognormal(0.0, 1.0, size=(B, n))
    w = np.maximum(1, np.rint(x * (2.2 * cap / x.sum(axis=1, keepdims=True)))).astype(np.int32)
    full = lambda v: np.full(B, v, np.int32)  # noqa: E731
    kb = W._sequential("short_lists", w, w.copy(), np.tile(np.array([[cap, cap * 4 // 10] * 2], np.int32), (B, 1)))
    if mode == "algorithm1":
        kb = W.KnapsackBatch(name=mode, mode=W.MODE_RECURSIVE, batch=B, item_stride=n, knap_stride=2, n_items=full(n),
                             n_knapsacks=full(1), weights=w, values=w.copy(), capacities=kb.capacities[:, :2].copy(),
                             fill_order=None, drop_time=(w // 3).astype(np.int32))
    if mode == "capacities":
        caps = np.rint(cap / 1.35 * (1 + 0.05 * np.tile(np.arange(8), (B, 1)))).astype(np.int32)
        kb = W.KnapsackBatch(name=mode, mode=W.MODE_CAPACITY_SWEEP, batch=B, item_stride=n, knap_stride=8, n_items=full(n),
                             n_knapsacks=full(8), weights=w, values=w.copy(), capacities=caps, fill_order=None, drop_time=None)
    took, outs = [], []
    for max_items in (n, 314, 700):
        with binding.DeftKnapsack(max_batch=B, max_items=max_items, max_knapsacks=8, max_capacity=cap, flags=FLAG) as h:
            db = h.upload(kb)
            best = np.inf
            for _ in range(12):
                h.set_profiling(True)
                o = h.solve_batch(db)
                torch.cuda.synchronize()
                best = min(best, h.get_profile().sweep_ms)
            took.append(best)
            outs.append([getattr(o, k).cpu().numpy().copy() for k in ("status", "total_value", "knap_value", "knap_load", "assignment")])
    print(f"{mode}: {took} ms", flush=True)
    for got in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(got, outs[0]))
    run(binding, oracle, kb.slice(0, 64), max_capacity=cap, max_items=314, flags=FLAG)
    assert max(took[1:]) < 1.08 * took[0]
