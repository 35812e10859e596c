"""Stages that are settled before the wavefronts of an instance meet at a barrier: their answers come after the outputs
are cleared, whichever wavefront prepares the stages (it differs by instance), however many windows and items there are."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,n", [(1000, 130), (4000, 700), (8100, 300), (10200, 1500), (13000, 600), (19900, 900), (26600, 1100), (38900, 1100)])
def test_answers_of_settled_stages_stay(binding, oracle, cap, n):
    r = np.random.Generator(np.random.PCG64(91000 + cap))
    batch, m = 24, 64
    w = r.integers(1, 4, size=(batch, n))
    v = r.integers(0, 1001, size=(batch, n))
    w[:, 5:] = cap + 1                      # six items at most fit: all together, or by their subsets
    at = r.integers(0, n, size=batch)
    w[np.arange(batch), at] = 2
    caps = r.integers(1, 3, size=(batch, m))
    caps[:, -1] = cap
    caps[1::2] = cap
    kb = W._sequential(f"settled_{cap}_{n}", w, v, caps)
    kb.fill_order = np.tile(np.arange(m)[::-1], (batch, 1)).astype(np.int32)
    kb.fill_order[::3] = np.argsort(r.random((len(kb.fill_order[::3]), m)), axis=1)
    for _ in range(3):
        run(binding, oracle, kb, max_capacity=cap)
