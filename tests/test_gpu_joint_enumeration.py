"""The two-link solve by enumeration of the selections that can be optimal, and what it leaves to the table sweep:
lists around the fewest and the most items it takes, values that tie (the smallest choice number has to come out),
items of no value, items that fit one link or none, links that hold everything, lists that run over, capacities
around the greatest it takes.  Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2503_16815_amd import workloads as W
from tests.test_gpu_parity import binding, run  # noqa: F401  (binding is a fixture)

pytestmark = pytest.mark.gpu


def _batch(seed, batch, n, w_hi, c1, c2, kind="free"):
    r = np.random.Generator(np.random.PCG64(seed))
    kb = W.random_joint(seed, batch=batch, n_max=n, w_hi=w_hi, v_hi=1000, c1_hi=c1, c2_hi=c2, ragged=False)
    if kind == "alike":          # few kinds of items: many selections are as good
        at = r.integers(0, 5, size=(batch, n))
        kb.weights[:, 0], kb.weights[:, 1] = 1 + np.array([1, 3, 4, 6, 7])[at], 2 + np.array([5, 9, 12, 14, 25])[at]
        kb.values[:] = np.array([7, 11, 15, 22, 30])[at]
    elif kind == "ratio":        # link 1 takes three times link 0's time throughout: moving items costs nothing
        kb.weights[:, 1] = np.minimum(3 * kb.weights[:, 0].astype(np.int64), 2 ** 31 - 1)
    elif kind == "time":         # values are the times on link 0
        kb.values[:] = kb.weights[:, 0]
    elif kind == "great":
        kb.values[:] = r.integers(1, (1 << 30) // n, size=kb.values.shape)
    elif kind == "nothing":      # half of the items are worth nothing, some fit no link
        kb.values[:, ::2] = 0
        kb.weights[:, :, 3::7] = 2 ** 31 - 1
    kb.capacities[:, 0] = r.integers(max(1, c1 // 2), c1 + 1, size=batch)
    kb.capacities[:, 1] = r.integers(max(1, c2 // 2), c2 + 1, size=batch)
    kb.capacities[0] = (c1, c2)
    return kb


KINDS = ["free", "alike", "ratio", "time", "great", "nothing"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,w_hi,c1,c2", [(15, 20, 60, 90), (16, 20, 60, 90), (33, 30, 200, 150), (64, 40, 300, 400), (65, 12, 120, 500),
                                          (150, 30, 180, 170)])
def test_kinds_of_lists(binding, oracle, kind, n, w_hi, c1, c2):
    run(binding, oracle, _batch(81000 + n, 6, n, w_hi, c1, c2, kind))


@pytest.mark.parametrize("c1,c2", [(768, 40), (769, 40), (40, 768), (40, 769), (1, 300), (300, 1), (127, 63), (128, 64), (129, 65)])
def test_capacities_around_the_cells_and_the_limit(binding, oracle, c1, c2):
    run(binding, oracle, _batch(82000 + c1 + c2, 4, 40, max(4, min(c1, c2) // 4), c1, c2))


@pytest.mark.parametrize("n", [1023, 1024, 1025])
def test_as_many_items_as_threads(binding, oracle, n):
    run(binding, oracle, _batch(83000 + n, 2, n, 9, 70, 60))


def test_links_that_hold_everything(binding, oracle):
    """All items of value fit link 0; fit both links together; all but one do."""
    kb = _batch(84000, 9, 30, 12, 400, 700)
    total = kb.weights[:, 0].sum(axis=1)
    kb.capacities[:, 0] = np.minimum(400, np.array([total[b] + (0, -1, -40)[b % 3] for b in range(9)]))
    run(binding, oracle, kb)


def test_faults_beside_good_instances(binding, oracle):
    kb = _batch(85000, 6, 24, 30, 150, 150)
    kb.weights[1, 1, 3] = 0
    kb.values[2, 4] = -1
    kb.capacities[3, 1] = -1
    kb.n_items[4] = 0
    run(binding, oracle, kb)


def _one_link(items, c, link, order=None):
    """Items (weight, value) that fit `link` alone, capacity c there; in the order given or as listed."""
    w, v = np.array(items, dtype=np.int64).T
    if order is not None:
        w, v = w[order], v[order]
    weights = np.full((1, 2, len(w)), 50, dtype=np.int64)
    weights[0, link] = w
    caps = [[c, 1]] if link == 0 else [[1, c]]
    return W.KnapsackBatch(name=f"one_link_{len(w)}_{c}_{link}", mode=W.MODE_JOINT2, batch=1, item_stride=len(w), knap_stride=2,
                           n_items=np.array([len(w)], np.int32), n_knapsacks=np.array([2], np.int32),
                           weights=weights.astype(np.int32), values=v[None].astype(np.int32),
                           capacities=np.array(caps, np.int32))


@pytest.mark.parametrize("link", [0, 1])
def test_more_items_as_close_to_the_price_than_are_listed(binding, oracle, link):
    """The best selection met first leaves more than 64 items to decide, none of them twice: the listed 64 are not all."""
    first = [(5, 500)] * 10 + [(4, 570)] * 70 + [(3, 475)]
    second = [(2, v) for v in range(251, 284)] + [(2, v) for v in range(117, 150)] + [(2, 200), (1, 5)]
    r = np.random.Generator(np.random.PCG64(86000))
    for items, c in ((first, 310), (second, 67)):
        run(binding, oracle, _one_link(items, c, link))
        for _ in range(3):
            run(binding, oracle, _one_link(items, c, link, r.permutation(len(items))))


@pytest.mark.parametrize("link", [0, 1])
@pytest.mark.parametrize("either", [29, 30, 31, 32, 33, 34, 40])
def test_as_many_items_to_decide_as_are_listed(binding, oracle, link, either):
    """2 x either + 2 items around the listed 64, with distinct losses and with ties (the highest index gives way)."""
    items = [(2, 251 + i) for i in range(either)] + [(2, 149 - i) for i in range(either)] + [(2, 200), (1, 5)]
    ties = [(2, 251 + i // 4) for i in range(either)] + [(2, 149 - i // 4) for i in range(either)] + [(2, 200), (1, 5)]
    for x in (items, ties):
        run(binding, oracle, _one_link(x, 2 * either + 1, link))
        run(binding, oracle, _one_link(x, 2 * either + 1, link, np.arange(len(x))[::-1]))


@pytest.mark.parametrize("n", [65, 66, 80, 130, 300])
def test_many_items_that_fit_one_link_only(binding, oracle, n):
    kb = _batch(87000 + n, 8, n, 6, 200, 150)
    kb.values[:] = 100 * kb.weights[:, 0] + np.random.Generator(np.random.PCG64(n)).integers(-60, 61, size=kb.values.shape)
    kb.weights[:4, 1] = 151
    kb.values[4:] = np.maximum(1, kb.values[4:])
    kb.weights[4:, 1], kb.weights[4:, 0] = np.minimum(kb.weights[4:, 0], 150), 201
    kb.values[:] = np.maximum(kb.values, 1)
    run(binding, oracle, kb)


def _profiled(binding, oracle, batches, c1, c2):
    """The batches one after the other on one handle, each against the oracle; the cells that the table sweep answered and ms."""
    import torch
    from tests.test_gpu_parity import assert_same
    got = []
    with binding.DeftKnapsack(max_batch=max(kb.batch for kb in batches), max_items=max(kb.item_stride for kb in batches),
                              max_knapsacks=2, max_c1=c1, max_c2=c2, device=0) as h:
        for kb in batches:
            ref = oracle.solve_batch(kb, nthreads=16, c1_limit=c1, c2_limit=c2)
            db = h.upload(kb)
            best = np.inf
            for _ in range(3):
                h.set_profiling(True)
                out = h.solve_batch(db)
                torch.cuda.synchronize()
                prof = h.get_profile()
                assert_same(kb, out, ref)
                best = min(best, prof.total_ms)
            got.append((int(prof.swept_cell_updates), best))
    return got


def test_what_is_settled_and_what_is_left_to_the_table(binding, oracle):
    """By the library's own count: unrelated values on links that hold a part are settled; where moving an item costs nothing
    there is too much to look through; lists below the fewest are swept; all fits link 0.  One handle, calls in turn."""
    settled = _batch(88000, 12, 49, 34, 339, 54, "free")
    settled.weights[:, 1] = settled.weights[:, 0] * np.random.Generator(np.random.PCG64(88)).integers(3, 7, size=(12, 49))
    settled.capacities[:] = (339, 54)
    left = _batch(88001, 5, 64, 64, 400, 400, "ratio")
    left.capacities[:] = (400, 400)
    few = _batch(88002, 7, 15, 40, 90, 120, "free")
    few.capacities[:] = (90, 120)
    fits = _batch(88003, 9, 30, 5, 300, 300, "free")
    fits.capacities[:] = (300, 300)
    cells = [c for c, _ in _profiled(binding, oracle, [settled, left, settled, few, fits, left, fits], 400, 400)]
    all_left, all_few = 5 * 64 * 401 * 401, 7 * 15 * 91 * 121
    assert cells[1:2] + cells[3:] == [all_left, all_few, 0, all_left, 0]
    assert max(cells[0], cells[2]) <= 49 * 340 * 55, "one instance may run late (attempts are bounded by time)"


@pytest.mark.parametrize("batch", [8, 64])
@pytest.mark.parametrize("n,w_hi", [(24, 100), (40, 70), (64, 64)])
def test_attempts_do_not_hold_up_the_sweep(binding, oracle, batch, n, w_hi):
    """Instances that are hardly ever settled (moving an item costs nothing): bit-exact, and about as fast as with
    a link one unit beyond what enumeration takes, which is swept at once (behind all attempts: 1.4 to 2.3 times as long)."""
    kb = _batch(89000 + n, batch, n, w_hi, 769, 700, "ratio")
    kb.capacities[:] = (769, 700)
    tried = kb.slice(0, batch)
    tried.capacities = np.full_like(kb.capacities, 700)
    tried.capacities[:, 0] = 768
    (_, sweep), (_, took) = _profiled(binding, oracle, [kb, tried], 769, 700)
    print(f"{took:.3f} ms, sweep {sweep:.3f} ms", flush=True)
    assert took < 1.25 * sweep + 0.05


def _time_on_link0(seed, batch, n, w_hi, c1, c2):
    """Values that are the times on link 0, link 1 three to six times as slow."""
    r = np.random.Generator(np.random.PCG64(seed + 1))
    kb = _batch(seed, batch, n, w_hi, c1, c2, "time")
    kb.weights[:, 1] = kb.weights[:, 0] * r.integers(3, 7, size=(batch, n))
    kb.capacities[:] = (c1, c2)
    return kb


@pytest.mark.parametrize("w_hi,c1,c2,batch,limit", [(35, 668, 63, 256, 1.5), (35, 103, 316, 32, 1.4)])
def test_attempts_in_parts_end_in_time(binding, oracle, w_hi, c1, c2, batch, limit):
    """Lists that run over of instances that are hardly ever settled: an attempt keeps to its time also while a list is
    made in parts that no pair suits.  ms as measured: 1.05 and 0.92; without a look at the clock there 10.0 and 5.3."""
    (left, took), = _profiled(binding, oracle, [_time_on_link0(90000 + c1, batch, 39, w_hi, c1, c2)], c1, c2)
    print(f"{c1} x {c2}, {batch}: {took:.3f} ms, left {left}", flush=True)
    assert left > 0 and took < limit


def test_parts_are_for_lists_that_they_can_settle(binding, oracle):
    """Many departures within one unit of value: an attempt whose lists run over gives up once other groups do not help.  Against the
    same items on links of which one is beyond what enumeration takes, so that they are swept at once (0.69 of that time; with
    parts until the attempt's time is up 0.87)."""
    n, w_hi, c1, c2 = 39, 35, 103, 316
    kb = _time_on_link0(90000 + c1, 32, n, w_hi, c1, c2)
    swept = kb.slice(0, 32)
    swept.capacities = np.full_like(kb.capacities, c1)
    swept.capacities[:, 1] = 769
    (_, sweep), (left, took) = _profiled(binding, oracle, [swept, kb], c1, 769)
    print(f"{n} {c1} x {c2}: {took:.3f} ms, sweep {sweep:.3f} ms, left {left}", flush=True)
    assert left > 0 and took < 0.78 * sweep


@pytest.mark.parametrize("seed,v_hi", [(102, 1000), (103, 1000), (106, 1000), (108, 1000), (109, 60), (110, 25)])
def test_lists_that_run_over_are_made_in_parts(binding, oracle, seed, v_hi):
    """64 items on links of 512: of 256 such instances some have more combinations than a list holds, in one or more of the
    groups; with few values many selections are as good, in several parts."""
    r = np.random.Generator(np.random.PCG64(seed))
    w0 = r.integers(1, 65, size=(256, 64))
    w1 = w0 * r.integers(3, 7, size=w0.shape)
    kb = W.hetero_joint(batch=256, n=64, c1=512, c2=512)
    kb.weights[:] = np.stack([w0, w1], axis=1)
    kb.values[:] = r.integers(1, v_hi + 1, size=w0.shape)
    run(binding, oracle, kb)


def test_parts_settle_what_lists_that_run_over_left(binding, oracle):
    """One instance of each of these inputs has lists that run over: made in parts they settle it (without parts one a call
    is left to its table).  An attempt that runs late may leave one."""
    batches = []
    for seed in (102, 103, 106, 108):
        r = np.random.Generator(np.random.PCG64(seed))
        w0 = r.integers(1, 65, size=(256, 64))
        kb = W.hetero_joint(batch=256, n=64, c1=512, c2=512)
        kb.weights[:] = np.stack([w0, w0 * r.integers(3, 7, size=w0.shape)], axis=1)
        kb.values[:] = r.integers(1, 1001, size=w0.shape)
        batches.append(kb)
    left = [cells // (64 * 513 * 513) for cells, _ in _profiled(binding, oracle, batches, 512, 512)]
    print(f"left: {left}", flush=True)
    assert sum(left) <= 1
