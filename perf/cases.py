"""Performance cases: the solver calls a user of the library makes, over the range of sizes,
modes, value kinds and handle kinds it is used with.

A case is a dict of plain values; `prepare` builds the candidate schedules, the handle and the
device buffers a user's program holds before the call, `run` is one call through the public
binding and returns every output of it.  All outputs are whole numbers and have to be the same,
bit for bit, whatever the implementation ("exact").

Bucket times are lognormal (Table I of the paper gives the totals and the windows), in 10 us or
1 us units; `value` says what an item is worth: its own time (the paper's objective), a priority
times its time, or something unrelated to it.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2503_16815_amd import binding, workloads as W

DEVICE = 0


def _seq(name, batch, n, k, total, back, fwd, value="time", sigma=1.2, heavy=0, ragged=False, flags=0):
    return dict(name=name, mode="sequential", batch=batch, n=n, k=k, total=total, back=back, fwd=fwd, value=value,
                sigma=sigma, heavy=heavy, ragged=ragged, flags=flags)


def listed():
    return [
        # one small scheduling decision asked for on its own: latency of a single call
        _seq("one_small", 1, 32, 1, 3200, 1000, 500, value="free", sigma=0.6),
        # a mixed bag of candidates, values unrelated to times, ragged lists, fill order given
        _seq("mixed_bag", 777, 203, 3, 21000, 7001, 3500, value="free", sigma=0.9, ragged=True),
        # GPT-2 windows in 10 us units with priorities: rows at the border of what a compute unit's LDS holds
        _seq("gpt2_10us", 256, 148, 1, 54640, 38100, 16900, value="priority", sigma=0.8),
        # the ResNet-101 candidate set, every k = 1..4 in one call, on a plain handle (bench.py's headline)
        _seq("resnet101_sweep", 4096, 314, 4, 24200, 11800, 5900),
        # the same on a handle that promises a subset-sum problem
        _seq("resnet101_subset", 4096, 314, 4, 24200, 11800, 5900, flags=2),
        # the VGG-19 candidate set (three buckets hold 85 % of the time) on a values-are-weights handle
        _seq("vgg19_sweep", 16384, 38, 4, 25800, 9300, 3700, sigma=1.0, heavy=3, flags=1),
        # Algorithm 1 on ResNet-101 backward stages, plain handle
        dict(name="backward_stages", mode="algorithm1", batch=1024, n=314, total=24200, back=11800, sigma=1.2, flags=0),
        # the Preserver's retries: one list at the window and ten inflated capacities
        dict(name="inflation", mode="capacities", batch=1024, n=314, k=11, total=24200, back=11800, sigma=1.2, flags=1),
        # the task queues simulated over eight iterations
        dict(name="task_queues", mode="queues", batch=1024, n=314, iterations=8, total=24200, back=11800, fwd=5900,
             sigma=1.2, flags=2),
        # GPT-2 windows in 1 us units with priorities: rows in HBM, a full batch and a handful of candidates
        _seq("gpt2_1us", 256, 148, 1, 546400, 381000, 169000, value="priority", sigma=0.8),
        _seq("gpt2_1us_few", 9, 148, 1, 546400, 381000, 169000, value="priority", sigma=0.8),
        # the two-link joint problem
        dict(name="two_link", mode="two_link", batch=256, n=64, c1=512, c2=512, w_hi=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    mode = rng.choice(("sequential", "sequential", "sequential", "long_rows", "algorithm1", "capacities", "queues", "two_link"))
    if mode == "sequential":
        value = rng.choice(("time", "time", "priority", "free"))
        n, back = _log(rng, 9, 700), _log(rng, 600, 24000)
        most = 1.6e10 if value == "time" else 4e9      # cells: about the listed sweeps'
        batch = min(_log(rng, 1, 6000), max(1, int(most / (n * back))))
        return dict(mode=mode, batch=batch, n=n, k=rng.randint(1, 4), total=int(back * rng.uniform(1.1, 2.8)) + n, back=back,
                    fwd=max(1, int(back * rng.uniform(0.3, 0.6))), value=value, sigma=round(rng.uniform(0.5, 1.3), 2),
                    heavy=rng.choice((0, 0, 3)), ragged=rng.random() < 0.4, flags=rng.choice((0, 1, 2)) if value == "time" else 0)
    if mode == "long_rows":
        back = _log(rng, 45000, 381000)
        n, batch = rng.randint(20, 148), _log(rng, 1, 256)
        if batch < 128:   # few candidates: as many cells as a good dozen of the listed shape
            batch = min(batch, max(1, int(8e8 / (n * back))))
        return dict(mode="sequential", batch=batch, n=n, k=1, total=int(back * rng.uniform(1.2, 2.0)), back=back,
                    fwd=int(back * rng.uniform(0.3, 0.5)), value=rng.choice(("priority", "priority", "free")),
                    sigma=round(rng.uniform(0.5, 1.2), 2), heavy=0, ragged=rng.random() < 0.3, flags=0)
    if mode == "two_link":
        return dict(mode=mode, batch=_log(rng, 1, 256), n=rng.randint(5, 64), c1=rng.randint(40, 512), c2=rng.randint(40, 512),
                    w_hi=rng.randint(12, 64))
    n, back = _log(rng, 20, 400), _log(rng, 900, 12000)
    case = dict(mode=mode, batch=_log(rng, 1, 1024), n=n, total=int(back * rng.uniform(1.3, 2.4)) + n, back=back,
                sigma=round(rng.uniform(0.6, 1.3), 2), flags=rng.choice((0, 1, 2)))
    if mode == "capacities":
        case["k"] = rng.randint(2, 11)
    if mode == "queues":
        case["fwd"] = int(back * rng.uniform(0.3, 0.6))
        case["iterations"] = rng.randint(2, 8)
    return case


def _times(r, batch, n, total, sigma, heavy=0):
    """Bucket times >= 1 summing to about `total` per candidate; `heavy` of them hold 85 % of it."""
    x = r.lognormal(0.0, sigma, size=(batch, n))
    if heavy and n > heavy:
        x /= x.sum(axis=1, keepdims=True)
        x *= 0.15
        at = r.random((batch, n)).argsort(axis=1)[:, :heavy]
        np.put_along_axis(x, at, 0.85 / heavy * r.uniform(0.9, 1.1, size=(batch, heavy)), axis=1)
    return np.maximum(1, np.rint(x * (total / x.sum(axis=1, keepdims=True)))).astype(np.int32)


def _values(r, kind, w):
    if kind == "time":
        return w.copy()
    if kind == "priority":
        return np.rint(w * r.uniform(1.0, 4.0, size=w.shape)).astype(np.int32)
    return r.integers(1, 1001, size=w.shape).astype(np.int32)


def _batch(mode, w, v, caps, n_items, n_knap, order=None, drop=None):
    i32 = lambda a: None if a is None else np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    return W.KnapsackBatch(name="case", mode=mode, batch=w.shape[0], item_stride=w.shape[-1], knap_stride=caps.shape[1],
                           n_items=i32(n_items), n_knapsacks=i32(n_knap), weights=i32(w), values=i32(v), capacities=i32(caps),
                           fill_order=i32(order), drop_time=i32(drop))


def prepare(case, seed):
    r = np.random.Generator(np.random.PCG64(seed))
    mode, B, n = case["mode"], case["batch"], case["n"]
    if mode == "two_link":
        w1 = r.integers(1, case["w_hi"] + 1, size=(B, n))
        w = np.stack([w1, w1 * r.integers(3, 7, size=(B, n))], axis=1)
        caps = np.tile(np.array([[case["c1"], case["c2"]]]), (B, 1))
        kb = _batch(W.MODE_JOINT2, w, _values(r, "free", w1), caps, np.full(B, n), np.full(B, 2))
        h = binding.DeftKnapsack(max_batch=B, max_items=n, max_knapsacks=2, max_c1=case["c1"], max_c2=case["c2"], device=DEVICE)
        return dict(h=h, db=h.upload(kb))
    w = _times(r, B, n, case["total"], case["sigma"], case.get("heavy", 0))
    window = lambda mean: np.rint(mean * r.uniform(0.9, 1.1, size=B)).astype(np.int64)  # noqa: E731
    back = window(case["back"])
    if mode == "queues":
        fwd = window(case["fwd"])
        drop = np.rint(w / w.sum(axis=1, keepdims=True) * back[:, None])
        sb = W.ScheduleBatch(name="case", batch=B, n_buckets=n, iterations=case["iterations"], comm_time=w,
                             drop_time=drop.astype(np.int32), forward_time=fwd.astype(np.int32),
                             backward_time=back.astype(np.int32))
        h = binding.DeftKnapsack(max_batch=B, max_items=n, max_knapsacks=2, max_capacity=int(max(back.max(), fwd.max())),
                                 flags=case["flags"], device=DEVICE)
        return dict(h=h, ds=binding.DeviceSchedules(sb, h.device))
    if mode == "algorithm1":
        caps = np.stack([back, np.zeros_like(back)], axis=1)
        drop = np.rint(w / w.sum(axis=1, keepdims=True) * back[:, None])
        kb = _batch(W.MODE_RECURSIVE, w, w, caps, np.full(B, n), np.full(B, 1), drop=drop)
    elif mode == "capacities":
        caps = np.rint(back[:, None] * (1.0 + 0.05 * np.arange(case["k"])[None, :]))
        kb = _batch(W.MODE_CAPACITY_SWEEP, w, w, caps, np.full(B, n), np.full(B, case["k"]))
    else:
        m = 2 * case["k"]
        caps = np.tile(np.stack([back, window(case["fwd"])], axis=1), (1, case["k"]))
        if case["ragged"]:   # lists and window counts of their own, windows in a given order
            n_items, n_knap = r.integers(n // 2, n + 1, size=B), r.integers(1, m + 1, size=B)
            order = np.where(np.arange(m)[None, :] < n_knap[:, None], r.random((B, m)), 2.0 + np.arange(m)[None, :]).argsort(axis=1)
        else:                # the sweep over k: the longest schedules first
            n_items, n_knap, order = np.full(B, n), 2 * (case["k"] - np.arange(B) * case["k"] // B), None
        kb = _batch(W.MODE_SEQUENTIAL, w, _values(r, case["value"], w), caps, n_items, n_knap, order)
    h = binding.DeftKnapsack(max_batch=B, max_items=n, max_knapsacks=kb.knap_stride, max_capacity=int(kb.capacities.max()),
                             flags=case["flags"], device=DEVICE)
    return dict(h=h, db=h.upload(kb))


def run(state):
    if "ds" in state:
        o = binding.simulate_schedule(state["h"], state["ds"])
        return [o.stage_case, o.stage_count, o.stage_time, o.update_k, o.tail, o.status]
    o = state["h"].solve_batch(state["db"])
    return [o.total_value, o.knap_value, o.knap_load, o.assignment, o.status]


def work(case):
    """Every input read once, every output written once; two operations (add, maximum) per item
    and capacity of the first window, or per 32 capacities where a value is its weight and a
    capacity needs one bit (an item is a shift and an or of the reachable sums)."""
    mode, B, n = case["mode"], case["batch"], case["n"]
    if mode == "two_link":
        return dict(bytes=4.0 * B * (3 * n + 4 + n + 7), flops=4.0 * B * n * (case["c1"] + 1) * (case["c2"] + 1))
    if mode == "queues":
        it = case["iterations"]
        return dict(bytes=4.0 * B * (2 * n + 2 + 7 * it + 3), flops=2.0 / 32 * B * it * n * (case["back"] + case["fwd"]))
    m = 2 * case["k"] if mode == "sequential" else case.get("k", 2)
    inputs = (3 if mode == "algorithm1" else 2) * n + 2 + m + (m if case.get("ragged") else 0)
    ops = 2.0 if case.get("value", "time") != "time" else 2.0 / 32
    return dict(bytes=4.0 * B * (inputs + n + 2 * m + 3), flops=ops * B * n * case["back"])


def tolerance(case):
    return "exact"
