"""The scan's steps at the sizes where they can go wrong: one replica, as many replicas as lanes, batches from 2 to 64, more
pending batches than a step has slots for, groups of more than 64 queries that leave together, free times at the clock's
horizon, a window cut short by the end of the input.  Every per-query latency is compared with the CPU oracle; the
kernel logic also runs under the CPU emulation with its consistency checks on."""
import numpy as np
import pytest

import emu_lib
from oracle import oracle
from paper_1812_01776_amd import estimator as binding
from paper_1812_01776_amd import workloads

# (replicas, largest batch, offered load, quantum of all times in us)
SIZES = [(1, 2, 0.9, 1), (1, 64, 1.1, 1), (2, 3, 0.95, 1), (3, 64, 0.8, 10), (5, 4, 1.0, 1), (16, 64, 0.9, 100), (17, 5, 0.97, 1),
         (31, 8, 0.7, 10), (33, 2, 1.02, 1), (63, 2, 0.9, 1), (64, 2, 0.95, 100), (64, 8, 0.85, 1), (64, 64, 0.9, 1000)]


def _queue_case(seed, R, B, load, quantum, n, burst=1, start=0):
    """A two-stage chain, then a fork and join whose branches are taken by some; every stage has R replicas and batches up to B."""
    rng = np.random.default_rng(7000 + seed)
    parents = [[], [0], [1], [1], [2, 3]]
    S = len(parents)
    lat = np.zeros((S, 1, B), np.uint32)
    for s in range(S):
        a, c = rng.integers(300, 3000), rng.integers(20, 300)
        lat[s, 0] = np.maximum((a + c * np.arange(1, B + 1)) // quantum * quantum, quantum)
    gap = float(lat[:, 0, B - 1].max()) / (R * B) / load
    gaps = np.rint(rng.gamma(0.5, 2.0 * gap, size=n)).astype(np.int64)
    if burst > 1:
        gaps = np.where(np.arange(n) % burst == 0, gaps * burst, 0)
    arr = np.cumsum(gaps // quantum * quantum)
    if start:  # queueing runs into the horizon
        arr = arr + (2**32 - 2 - int(arr[-1]) - int(lat.max(axis=2).sum()) - 2 * int(lat.max()))
    mask = np.full(n, 0b10011, np.uint32)
    mask |= (rng.random(n) < 0.7).astype(np.uint32) << 2
    mask |= (rng.random(n) < 0.6).astype(np.uint32) << 3
    cost = np.full((S, 1), 3, np.uint64)
    one = np.ones((1, S), np.int64)
    return workloads.Workload("queue%d" % seed, parents, lat, cost, arr.astype(np.uint32), mask, (one * 0).astype(np.uint8),
                              (one * B).astype(np.uint8), (one * R).astype(np.uint16), int(lat.max()) * 2)


def _compare(w, est):
    cfg = binding.pack_configs(w.cfg_hw, w.cfg_batch, w.cfg_replicas)
    ref = oracle.run(w.parents, w.lat_us, w.cost_uusd_hr, w.arrival_us, w.visit_mask, w.cfg_hw, w.cfg_batch,
                     w.cfg_replicas, w.slo_us, want_latencies=True)
    assert np.array_equal(est.run_latencies(w.arrival_us, w.visit_mask, cfg).astype(np.uint64), ref["latency"])
    got = est.run(w.arrival_us, w.visit_mask, cfg, w.slo_us)
    assert np.array_equal(got["p99_us"].astype(np.uint64), ref["p99_us"])
    assert np.array_equal(got["miss_count"].astype(np.uint64), ref["miss_count"])


def _cases(i, n):
    R, B, load, quantum = SIZES[i]
    yield _queue_case(i, R, B, load, quantum, n)
    yield _queue_case(100 + i, R, B, load, quantum, n, burst=130)         # groups of 130 cut into batches that tie
    yield _queue_case(200 + i, R, B, 1.3 * load, quantum, n + 1, start=1)


def _horizon_case(i, n):
    """Queues that run into the horizon at every size: four times the load, and a trace that ends as close to the horizon as is
    accepted."""
    R, B, load, quantum = SIZES[i]
    w = _queue_case(300 + i, R, B, 4.0 * load, quantum, n)
    w.slo_us = 1
    w.arrival_us = (w.arrival_us.astype(np.int64) + (2**32 - 3 - int(w.arrival_us[-1]) - int(w.lat_us.max(axis=(1, 2)).sum()))).astype(np.uint32)
    ref = oracle.run(w.parents, w.lat_us, w.cost_uusd_hr, w.arrival_us, w.visit_mask, w.cfg_hw, w.cfg_batch,
                     w.cfg_replicas, w.slo_us, want_latencies=True)
    clamped = int((ref["latency"][0] + w.arrival_us.astype(np.uint64) == 2**32 - 1).sum())
    assert 0 < clamped < n
    return w


@pytest.mark.parametrize("i", range(len(SIZES)))
def test_queues_at_the_horizon_emulated(i):
    w = _horizon_case(i, 8000 if SIZES[i][0] * SIZES[i][1] == 4096 else 1500)
    _compare(w, emu_lib.make(w))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [8000, 20001])
@pytest.mark.parametrize("i", range(len(SIZES)))
def test_queues_at_the_horizon_gpu(i, n):
    w = _horizon_case(i, n)
    est = binding.Estimator(w.parents, w.lat_us, w.cost_uusd_hr)
    _compare(w, est)
    est.close()


@pytest.mark.parametrize("i", range(len(SIZES)))
def test_steps_at_the_edges_emulated(i):
    for w in _cases(i, 421):
        _compare(w, emu_lib.make(w))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 63, 64, 65, 5000])
@pytest.mark.parametrize("i", range(len(SIZES)))
def test_steps_at_the_edges_gpu(i, n):
    for w in _cases(i, n):
        est = binding.Estimator(w.parents, w.lat_us, w.cost_uusd_hr)
        _compare(w, est)
        est.close()


# ---- workgroups that share candidates: one candidate alone, fewer candidates than workgroups, more candidates than wavefronts,
#      a last workgroup with fewer candidates than the others
def _counted(C, S, n, seed):
    rng = np.random.default_rng(9000 + seed)
    w = workloads.random_case(50 + S, S=S, n=n, C=1, dag="random", max_b=8, max_r=4)
    w.cfg_hw = rng.integers(0, 2, size=(C, S)).astype(np.uint8)
    w.cfg_batch = rng.integers(1, 9, size=(C, S)).astype(np.uint8)
    w.cfg_replicas = rng.integers(1, 5, size=(C, S)).astype(np.uint16)
    return w


@pytest.mark.parametrize("C", [1, 2, 3, 7, 17])
def test_candidate_counts_emulated(C):
    w = _counted(C, 4, 90, C)
    _compare(w, emu_lib.make(w))


@pytest.mark.gpu
@pytest.mark.parametrize("S", [2, 9])
@pytest.mark.parametrize("C", [1, 255, 513, 1537, 6145])
def test_candidate_counts_gpu(C, S):
    w = _counted(C, S, 130, C)
    est = binding.Estimator(w.parents, w.lat_us, w.cost_uusd_hr)
    _compare(w, est)
    est.close()


def _join_case(k, n, start):
    """A fork of k branches, each taken by some queries, joined again: every query is fed by one to k streams, and what a
    round of the join passes on is sometimes more and sometimes less than a wavefront has lanes."""
    rng = np.random.default_rng(8000 + 10 * k + n)
    parents = [[]] + [[0]] * k + [list(range(1, k + 1))]
    S = k + 2
    lat = np.zeros((S, 1, 8), np.uint32)
    for s in range(S):
        lat[s, 0] = rng.integers(300, 3000) + rng.integers(20, 300) * np.arange(1, 9)
    arr = np.cumsum(np.rint(rng.gamma(0.5, 400.0, size=n)).astype(np.int64))
    if start:  # queueing runs into the horizon
        arr = arr + (2**32 - 2 - int(arr[-1]) - int(lat.max(axis=2).sum()) - 5000)
    mask = np.full(n, 1 | 1 << (k + 1), np.uint32)
    for b in range(1, k + 1):
        mask |= (rng.random(n) < (0.9 if b == 1 else 0.4)).astype(np.uint32) << b
    one = np.ones((1, S), np.int64)
    batch = rng.integers(1, 9, size=(1, S))
    return workloads.Workload("join%d" % k, parents, lat, np.full((S, 1), 3, np.uint64), arr.astype(np.uint32), mask, (one * 0).astype(np.uint8),
                              batch.astype(np.uint8), (one * 3).astype(np.uint16), 5000)


@pytest.mark.parametrize("k", [2, 3, 4, 7])
def test_joins_emulated(k):
    for n, start in ((1, 0), (63, 0), (65, 1), (900, 0)):
        w = _join_case(k, n, start)
        _compare(w, emu_lib.make(w))


@pytest.mark.gpu
@pytest.mark.parametrize("start", [0, 1])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 6000])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 7])
def test_joins_gpu(k, n, start):
    w = _join_case(k, n, start)
    est = binding.Estimator(w.parents, w.lat_us, w.cost_uusd_hr)
    _compare(w, est)
    est.close()
