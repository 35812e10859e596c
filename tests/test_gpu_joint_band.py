"""GPU parity of the two-link solve where the band of rows that is computed begins, ends or is
empty: capacities around the weight of all items on link 0, around one item's, zero; single
items; items of no value; items heavier than the LDS ring or than the capacity."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,w_hi,c1_max,c2_hi", [(1, 9, 12, 40), (7, 12, 90, 256), (33, 40, 700, 300), (24, 200, 900, 512),
                                                 (64, 64, 512, 512), (90, 5, 300, 70)])
def test_edges_of_the_band(binding, oracle, n, w_hi, c1_max, c2_hi):
    kb = W.random_joint(7100 + n, batch=40, n_max=n, w_hi=w_hi, v_hi=3, c1_hi=c1_max, c2_hi=c2_hi, ragged=n > 1)
    for b in range(kb.batch):   # around the sum of all weights, of all but the last, of the first, of the last
        w = kb.weights[b, 0, :max(1, int(kb.n_items[b]))].astype(np.int64)
        at = (w.sum(), w[:-1].sum(), w[0], w[-1], w[1:].sum())[b % 5] + (b // 5) % 3 - 1
        if b < 30:
            kb.capacities[b, 0] = min(max(int(at), 0), c1_max)
    kb.weights[::7, 0, n // 2] = c1_max + 5
    kb.weights[3, 0, 0] = 2 ** 31 - 1   # no sum of weights may wrap
    print(f"case {kb.name}", flush=True)
    run(binding, oracle, kb)
