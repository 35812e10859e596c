"""Stages of subset-sum problems by what they leave out, where that can go wrong: lists around a chunk of 64 and the
plane counts, excesses around 63, 512 and 2047, prefixes that reach the capacity only after several more items or not
at all, runs too short in the items' order, items of one or two weights, items heavier than all before them.  All modes,
bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import binding, run  # noqa: F401  (binding is a fixture)
from tests.test_gpu_schedule import assert_same, simulate

pytestmark = pytest.mark.gpu

FLAG = 2   # DEFT_FLAG_SUBSET_SUM


def _weights(r, kind, batch, n):
    if kind == "lognormal":
        return np.maximum(1, np.rint(r.lognormal(3.5, 1.2, size=(batch, n))))
    if kind == "light":
        return r.integers(1, 9, size=(batch, n))
    if kind == "heavy":       # few light items: the 64 lowest sums show nothing
        return r.integers(100, 900, size=(batch, n))
    if kind == "thirds":      # nothing but multiples of three, and here and there an item that is not
        return 3 * r.integers(1, 60, size=(batch, n)) + (r.random((batch, n)) < 0.02)
    if kind == "two":         # two weights
        return np.where(r.random((batch, n)) < 0.5, 14, 35)
    if kind == "late_light":  # light items behind heavy ones: runs that begin late
        w = np.sort(r.lognormal(4.0, 1.3, size=(batch, n)), axis=1)[:, ::-1] + 1
        return np.where(r.random((batch, n)) < 0.1, r.permuted(w, axis=1), w)
    # jumps: light lists that an item of many times their weight takes past the capacity
    w = r.integers(1, 70, size=(batch, n))
    return np.where(r.random((batch, n)) < 0.03, r.integers(500, 6000, size=(batch, n)), w)


KINDS = ("lognormal", "light", "heavy", "thirds", "two", "late_light", "jumps")


@pytest.mark.parametrize("n", [65, 127, 128, 129, 300, 512, 513, 700])
@pytest.mark.parametrize("kind", KINDS)
def test_windows_in_turn(binding, oracle, kind, n):
    r = np.random.Generator(np.random.PCG64(51000 + n + 1000 * KINDS.index(kind)))
    w = _weights(r, kind, 40, n).astype(np.int64)
    caps = (w.sum(axis=1, keepdims=True) * r.uniform(0.03, 0.6, size=(40, 3))).astype(np.int64).clip(1, 65535)
    kb = W._sequential(f"excess_{kind}_{n}", w, w.copy(), caps)
    run(binding, oracle, kb, flags=FLAG)


@pytest.mark.parametrize("kind", KINDS)
def test_levels_capacities_and_queues(binding, oracle, kind):
    import dataclasses
    r = np.random.Generator(np.random.PCG64(52000 + KINDS.index(kind)))
    w = np.minimum(_weights(r, kind, 24, 150), 3000).astype(np.int32)
    total = w.sum(axis=1, keepdims=True)
    base = W.random_recursive(52100, batch=24, n_max=150, w_hi=5, v_hi=5, cap_hi=9, t_hi=3, ties=True)
    caps = (total * r.uniform(0.2, 0.7, size=(24, 1))).astype(np.int32).clip(1, 65535)
    kb = dataclasses.replace(base, item_stride=150, weights=w, values=w.copy(), n_items=np.full(24, 150, np.int32),
                             capacities=np.concatenate([caps, 0 * caps], axis=1).astype(np.int32), knap_stride=2,
                             n_knapsacks=np.ones(24, np.int32), drop_time=r.integers(0, 40, size=(24, 150)).astype(np.int32))
    run(binding, oracle, kb, flags=FLAG)
    base = W.random_capacity_sweep(52200, batch=24, n_max=150, m_max=9, w_hi=5, v_hi=5, cap_hi=9, ties=True)
    caps = (total * r.uniform(0.02, 0.9, size=(24, 9))).astype(np.int32).clip(0, 65535)
    kb = dataclasses.replace(base, item_stride=150, weights=w, values=w.copy(), n_items=np.full(24, 150, np.int32),
                             capacities=caps, knap_stride=9, n_knapsacks=r.integers(1, 10, size=24).astype(np.int32))
    run(binding, oracle, kb, flags=FLAG)
    back = (total[:, 0] * r.uniform(0.3, 0.8, size=24)).astype(np.int32).clip(1, 65535)
    sb = W.ScheduleBatch(name=kind, batch=24, n_buckets=150, iterations=7, comm_time=w,
                         drop_time=r.integers(0, 40, size=(24, 150)).astype(np.int32),
                         forward_time=(back * 0.45).astype(np.int32), backward_time=back)
    cap = int(back.max())
    assert_same(simulate(binding, sb, cap), oracle.simulate_batch(sb, cap_limit=cap, nthreads=16))


@pytest.mark.parametrize("excess", [1, 31, 62, 63, 64, 65, 95, 96, 127, 128, 511, 512, 2047, 2048, 2100])
def test_excesses_by_construction(binding, oracle, excess):
    """A list that one item takes `excess` past the capacity, light items of weights from 1, 2, 3, 5 or 33 on before it."""
    r = np.random.Generator(np.random.PCG64(53000 + excess))
    w, caps = [], []
    for least in (1, 2, 3, 5, 33):
        for _ in range(6):
            x = r.integers(least, max(least + 40, excess // 12), size=100)
            x[80] = excess + int(r.integers(1, 50))
            w.append(x)
            caps.append([int(x[:81].sum()) - excess, 900])
    w = np.array(w, np.int32)
    run(binding, oracle, W._sequential(f"by_construction_{excess}", w, w.copy(), np.array(caps, np.int32)), flags=FLAG)
