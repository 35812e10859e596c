"""The LDS-row kernels on values that are weights, through the two ways that still lead there: the entry
point without a handle, on every compiled variant, and calls too short to look at the values.  Sweeps
that end at the reached capacity, write-back of the variant's highest slots (both add-TID bases), the walk
from the last swept item.  Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import assert_same, binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_capacity,n_max,w_hi,batch", [
    (1023, 160, 30, 64), (4095, 600, 30, 20), (8191, 1160, 30, 12), (10239, 1450, 30, 5), (13311, 1890, 30, 5),
    (19967, 2830, 30, 5), (26623, 3000, 39, 4), (38911, 3000, 57, 2),
])
def test_every_variant_without_a_handle(binding, oracle, max_capacity, n_max, w_hi, batch):
    import torch
    kb = W.filling_rows(45000 + max_capacity, batch=batch, n_max=n_max, m_max=3, w_hi=w_hi, cap_lo=max_capacity * 55 // 100,
                        cap_hi=max_capacity)
    assert np.array_equal(kb.values, kb.weights)
    print(f"case {kb.name} batch={kb.batch} n<={n_max} max_capacity={max_capacity}", flush=True)
    ref = oracle.solve_batch(kb, nthreads=16, cap_limit=max_capacity)
    out = binding.solve_batch_static(binding.DeviceBatch(kb, torch.device("cuda", 0)), max_capacity)
    torch.cuda.synchronize()
    assert_same(kb, out, ref)


@pytest.mark.parametrize("n_max,cap_hi", [(120, 1023), (31, 4095), (15, 8191), (9, 13311), (6, 19967), (3, 38911)])
def test_calls_too_short_to_look(binding, oracle, n_max, cap_hi):
    for batch in (1, 60):
        ks = W.random_sequential(46000 + cap_hi, batch=batch, n_max=n_max, m_max=3, w_hi=max(9, 2 * cap_hi // n_max), v_hi=9,
                                 cap_hi=cap_hi, ties=True)
        run(binding, oracle, ks, max_capacity=cap_hi)
        kr = W.random_recursive(47000 + cap_hi, batch=batch, n_max=n_max, w_hi=max(9, 2 * cap_hi // n_max), v_hi=9, cap_hi=cap_hi,
                                t_hi=max(1, cap_hi // 100), ties=True)
        run(binding, oracle, kr, max_capacity=cap_hi)
        kc = W.random_capacity_sweep(48000 + cap_hi, batch=batch, n_max=n_max, m_max=7, w_hi=max(9, 2 * cap_hi // n_max), v_hi=9,
                                     cap_hi=cap_hi, ties=True)
        run(binding, oracle, kc, max_capacity=cap_hi)
