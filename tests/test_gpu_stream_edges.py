"""The streamed sweep (rows in global memory) where it can go wrong: weights around its block sizes and
around what its rings can hold, list lengths around the items of a pass, windows that nearly hold
everything or nearly nothing, capacity sweeps beyond the list's weight.  Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


def _batch(seed, batch, n, draw_w, caps, mode=W.MODE_SEQUENTIAL, v_hi=5000):
    r = np.random.Generator(np.random.PCG64(seed))
    w = np.asarray(draw_w(r, (batch, n)), np.int32)
    v = r.integers(0, v_hi, size=(batch, n)).astype(np.int32)       # some items of no value
    cap = np.tile(np.array([caps], np.int32), (batch, 1))
    kb = W._sequential(f"stream_{seed}", w, v, cap)
    kb.mode = mode
    return kb


@pytest.mark.parametrize("n", [1, 2, 6, 7, 8, 9, 14, 15, 16, 23])
def test_list_lengths(binding, oracle, n):
    for seed, w_hi in ((1, 9000), (2, 80000 // n + 2)):
        kb = _batch(41000 + 10 * n + seed, 5, n, lambda r, s: r.integers(1, w_hi, size=s), [45000, 20000])
        run(binding, oracle, kb, max_capacity=45000)


@pytest.mark.parametrize("weight", [1, 511, 512, 1023, 1024, 1025, 1535, 1536, 2560, 3583, 7680, 15000, 33000, 35000, 36352, 36353, 37000, 40000])
def test_weights_around_the_blocks_and_the_rings(binding, oracle, weight):
    """One weight throughout, then mixed with light and heavy neighbours (passes of every length)."""
    run(binding, oracle, _batch(42000 + weight, 3, 12, lambda r, s: np.full(s, weight), [52000, 30000]), max_capacity=52000)
    run(binding, oracle, _batch(43000 + weight, 5, 30, lambda r, s: np.where(r.random(s) < 0.3, weight, r.integers(1, 6000, size=s)),
                                [61000, 40000]), max_capacity=61000)


@pytest.mark.parametrize("share", [0.02, 0.3, 0.9, 0.99, 1.0, 1.2])
def test_bands_of_every_width(binding, oracle, share):
    """The window as a share of the list's weight: the band of cells that matter is narrow where it
    holds almost nothing or almost everything."""
    weight = 60000 / share
    kb = _batch(44000 + int(100 * share), 6, 60, lambda r, s: r.integers(1, int(2 * weight / 60), size=s), [60000, 25000])
    run(binding, oracle, kb, max_capacity=60000)


def test_capacity_sweeps(binding, oracle):
    caps = [100, 39000, 52000, 4000, 70000, 69999, 1]
    for seed, w_hi in ((1, 2000), (2, 9000), (3, 30000)):
        kb = _batch(45000 + seed, 5, 25, lambda r, s: r.integers(1, w_hi, size=s), caps, W.MODE_CAPACITY_SWEEP)
        run(binding, oracle, kb, max_capacity=70000)


@pytest.mark.parametrize("n", [1, 6, 7, 12, 40])
@pytest.mark.parametrize("over", [-1, 0, 1, 5000])
def test_capacity_sweeps_whose_every_capacity_is_near_or_beyond_the_weight(binding, oracle, n, over):
    """The least capacity one short of the list's weight, the weight itself, and beyond: from the
    weight on there is no row to sweep, and no row cell is counted."""
    import torch
    weight = 50000 // n * n
    kb = _batch(46000 + n, 4, n, lambda r, s: np.full(s, weight // n), [weight + over + 9000, weight + over, weight + over + 1],
                W.MODE_CAPACITY_SWEEP)
    kb.weights[:, 0] += 2 * (n > 1)
    kb.weights[:, -1] -= 2 * (n > 1)
    run(binding, oracle, kb, max_capacity=70000)
    with binding.DeftKnapsack(max_batch=kb.batch, max_items=kb.item_stride, max_knapsacks=kb.knap_stride, max_capacity=70000) as h:
        db = h.upload(kb)
        h.set_profiling(True)
        h.solve_batch(db)
        torch.cuda.synchronize()
        cells = int(h.get_profile().streamed_row_cells)
    assert cells == 0 if over >= 0 else 0 < cells <= 4 * n * 2 * (weight + 1), cells
