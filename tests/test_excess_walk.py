"""The claim the stages of subset-sum problems by what they leave out rest on, checked on the CPU against the oracle's DP
and walk, over Python integers as bit sets; no GPU.  Where C is reachable with items 0 .. p and not with fewer, the
selection is items 0 .. p less those that, going down from p, can still be left out of the excess (their weight less
C): an item is left out exactly when what then remains of the excess is a sum of the items before it.  The run that
stands in for sums beyond 63 only ever shows sums that are reachable."""
import numpy as np

from tests.test_oracle_pins import make_seq


def sums_before(weights):
    sets = [1]
    for w in weights:
        sets.append(sets[-1] | (sets[-1] << w))
    return sets


def by_excess(weights, cap):
    """The selection, or None where the capacity is not reachable."""
    offered = [i for i, w in enumerate(weights) if w <= cap]
    w = [weights[i] for i in offered]
    if sum(w) <= cap:
        return offered
    sets, upto = sums_before(w), 0
    for p, x in enumerate(w):
        upto += x
        excess = upto - cap
        if excess < 0 or not (sets[p] >> excess) & 1:
            continue
        taken = [p]
        for i in range(p - 1, -1, -1):
            rest = excess - w[i]
            if excess > 0 and rest >= 0 and (sets[i] >> rest) & 1:
                excess = rest
            else:
                taken.append(i)
        assert excess == 0
        return sorted(offered[i] for i in taken)
    return None


def test_selection_by_excess_is_the_dp_walk(oracle):
    r = np.random.default_rng(41001)
    seen = 0
    for _ in range(400):
        n = int(r.integers(2, 40))
        w = r.integers(1, int(r.integers(2, 60)), size=n)
        if r.random() < 0.3:
            w[r.random(n) < 0.2] *= 9
        w = w.tolist()
        cap = int(r.integers(1, max(2, int(sum(w) * r.uniform(0.1, 1.1)))))
        taken = by_excess(w, cap)
        if taken is None:
            continue
        seen += 1
        ref = oracle.solve_batch(make_seq([w], [w], [[cap]]))
        assert taken == np.flatnonzero(ref.assignment[0] == 0).tolist()
    assert seen > 300


def test_a_run_shows_reachable_sums_only():
    """All sums lo .. hi of some items, and items up to hi - lo + 1 in any order, lightest first: all of lo .. hi + their weight."""
    r = np.random.default_rng(41002)
    grown = 0
    for _ in range(800):
        light = r.integers(1, 64, size=int(r.integers(5, 30))).tolist()
        bits = sums_before(light)[-1]
        if (bits >> 32) & 0xffffffff != 0xffffffff:
            continue
        more = sorted(r.integers(1, 400, size=20).tolist())
        length = 32
        for w in more:
            if w <= length:
                length += w
                bits |= bits << w
        grown += length > 64
        want = ((1 << length) - 1) << 32
        assert bits & want == want
    assert grown > 100
