"""Handles without flags: instances whose values equal their weights go to the bit-set kernels, the
others to rows of values, in one call.  Both kinds side by side, faulty instances among them, in every
mode that asks, on both sides of the batch and size at which a call asks at all (fewer than 1024
instances with items times capacity below 2^17 go to the rows at once).  Bit-exact against
the oracle."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import assert_same, binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


def _mix(kb, seed, equal):
    """`equal` of the instances get values equal to weights, one item of some others almost does."""
    r = np.random.Generator(np.random.PCG64(seed))
    kb.values = np.ascontiguousarray(kb.values)
    for b in np.flatnonzero(r.random(kb.batch) < equal):
        kb.values[b] = kb.weights[b]
    for b in range(0, kb.batch, 5):     # a single value that differs, anywhere in the list (also first and last)
        kb.values[b] = kb.weights[b]
        n = int(kb.n_items[b])
        if n:
            kb.values[b, (0, n - 1, n // 2)[b // 5 % 3]] += 1 + b % 3
    return kb


@pytest.mark.parametrize("equal", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("batch,n_max,cap_hi", [
    (63, 60, 900), (64, 60, 900), (5, 120, 3000), (67, 60, 4000),   # two calls that do not ask, two that do
    (301, 70, 9000), (130, 600, 13000), (40, 90, 38000),            # one record width after the other
])
def test_sequential(binding, oracle, batch, n_max, cap_hi, equal):
    kb = W.random_sequential(41000 + cap_hi + batch, batch=batch, n_max=n_max, m_max=4, w_hi=max(9, cap_hi // 12), v_hi=50,
                             cap_hi=cap_hi)
    kb = _mix(kb, 1, equal)
    kb.weights[1, 0] = 0                # faults of every kind are reported by whichever kernel meets them
    kb.capacities[2, 0] = cap_hi + 7
    kb.n_items[3] = -1
    run(binding, oracle, kb, max_capacity=cap_hi)


@pytest.mark.parametrize("batch,cap_hi", [(70, 900), (66, 8000), (20, 13000)])
def test_other_modes(binding, oracle, batch, cap_hi):
    for equal in (0.5, 1.0):
        kr = W.random_recursive(42000 + cap_hi, batch=batch, n_max=140, w_hi=max(9, cap_hi // 30), v_hi=60, cap_hi=cap_hi,
                                t_hi=max(1, cap_hi // 200))
        run(binding, oracle, _mix(kr, 2, equal), max_capacity=cap_hi)
        kc = W.random_capacity_sweep(43000 + cap_hi, batch=batch, n_max=140, m_max=31, w_hi=max(9, cap_hi // 30), v_hi=60,
                                     cap_hi=cap_hi)
        run(binding, oracle, _mix(kc, 3, equal), max_capacity=cap_hi)


@pytest.mark.parametrize("mode", [W.MODE_SEQUENTIAL, W.MODE_RECURSIVE, W.MODE_CAPACITY_SWEEP])
@pytest.mark.parametrize("batch,n,cap,asks", [
    (1023, 64, 2047, False), (1024, 64, 2047, True),    # the batch
    (3, 64, 2047, False), (3, 64, 2048, True), (3, 65, 2017, True),   # items times capacity: 131008, 131072, 131105
])
def test_where_a_call_asks(binding, oracle, mode, batch, n, cap, asks):
    """Both sides of the rule; a call that asks is two launches, one that does not is one."""
    import torch
    if mode == W.MODE_SEQUENTIAL:
        kb = W.random_sequential(44000 + batch + cap, batch=batch, n_max=n, m_max=2, w_hi=120, v_hi=50, cap_hi=cap)
    elif mode == W.MODE_RECURSIVE:
        kb = W.random_recursive(44000 + batch + cap, batch=batch, n_max=n, w_hi=120, v_hi=50, cap_hi=cap, t_hi=9)
    else:
        kb = W.random_capacity_sweep(44000 + batch + cap, batch=batch, n_max=n, m_max=4, w_hi=120, v_hi=50, cap_hi=cap)
    kb = _mix(kb, 4, 0.5)
    assert kb.item_stride == n
    ref = oracle.solve_batch(kb, nthreads=16, cap_limit=cap)
    with binding.DeftKnapsack(max_batch=batch, max_items=n, max_knapsacks=max(2, kb.knap_stride), max_capacity=cap) as h:
        db = h.upload(kb)
        h.set_profiling(True)
        out = h.solve_batch(db)
        torch.cuda.synchronize()
        launches = int(h.get_profile().sweep_launches)
        assert_same(kb, out, ref)
    assert launches == (2 if asks else 1)
