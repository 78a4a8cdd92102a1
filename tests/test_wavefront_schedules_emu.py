"""The driver of the simulation kernel under other schedules than one operation after the other.

In the CPU emulation the wavefronts of a launch are alive together.  With EST_EMU_SCHEDULE set a turn lasts a random number of
primitives, so operations of one candidate run inside one another, read cursors their neighbours publish on the way, and a
wavefront can sleep between any two primitives while the others finish whole candidates.
"""
import numpy as np
import pytest

import emu_lib
from oracle import oracle
from paper_1812_01776_amd import estimator as binding
from paper_1812_01776_amd import workloads
from test_shared_prefix import _check as check_shared


def _check(w, est=None):
    est = est or emu_lib.make(w)
    cfg = binding.pack_configs(w.cfg_hw, w.cfg_batch, w.cfg_replicas)
    ref = oracle.run(w.parents, w.lat_us, w.cost_uusd_hr, w.arrival_us, w.visit_mask, w.cfg_hw, w.cfg_batch, w.cfg_replicas, w.slo_us,
                     want_latencies=True)
    got = est.run(w.arrival_us, w.visit_mask, cfg, w.slo_us)
    assert np.array_equal(got["p99_us"].astype(np.uint64), ref["p99_us"])
    assert np.array_equal(got["miss_count"].astype(np.uint64), ref["miss_count"])
    lat = est.run_latencies(w.arrival_us, w.visit_mask, cfg)
    assert np.array_equal(lat.astype(np.uint64), ref["latency"])
    return est


@pytest.mark.parametrize("waves", [1, 4, 12])
@pytest.mark.parametrize("seed", range(4))
def test_operations_inside_one_another_match_oracle(seed, waves, monkeypatch):
    # (a pipeline of more than eight operations takes workgroups of up to twelve wavefronts)
    monkeypatch.setenv("EST_EMU_SCHEDULE", str(seed))
    monkeypatch.setenv("EST_EMU_WAVES", str(waves))
    _check(workloads.random_case(seed + 40, S=8, n=250, C=2 + 3 * (seed % 2), max_b=8, max_r=4, tie_heavy=seed % 3 == 0))


@pytest.mark.parametrize("seed", range(4))
def test_long_queues_inside_one_another_match_oracle(seed, monkeypatch):
    monkeypatch.setenv("EST_EMU_SCHEDULE", str(seed))
    w = [workloads.backlog_case, workloads.provisioned_case][seed % 2](seed)
    _check(w.subset(n_queries=min(w.n_queries, 600)))


@pytest.mark.parametrize("seed", range(4))
def test_shared_stages_inside_one_another_match_oracle(seed, monkeypatch):
    monkeypatch.setenv("EST_EMU_SCHEDULE", str(seed))
    monkeypatch.setenv("EST_EMU_WAVES", "12")
    w, bases, base_of = workloads.neighbourhood_case(seed, S=7)
    check_shared(emu_lib.make(w), w, bases, base_of, "cpu")


@pytest.mark.parametrize("schedule", [None, 2, 4, 7])
def test_a_wavefront_without_work_waits_as_long_as_anything_moves(schedule, monkeypatch):
    # one stage: two operations, so that at least two of the four wavefronts have nothing to do until the trace ends
    monkeypatch.setenv("EST_EMU_STILL_LIMIT", "64")
    if schedule is not None:
        monkeypatch.setenv("EST_EMU_SCHEDULE", str(schedule))
    _check(workloads.random_case(2, S=1, n=1500, C=1))


@pytest.mark.parametrize("schedule", [None, 8])
def test_a_candidate_that_cannot_end_ends_the_call(schedule, monkeypatch):
    monkeypatch.setenv("EST_EMU_STILL_LIMIT", "64")
    monkeypatch.setenv("EST_EMU_HOLD_LOCK", "1")
    if schedule is not None:
        monkeypatch.setenv("EST_EMU_SCHEDULE", str(schedule))
    with pytest.raises(binding.EstimatorError) as ei:
        _check(workloads.random_case(2, S=3, n=100, C=2))
    assert ei.value.code == binding.EST_EINTERNAL


@pytest.mark.parametrize("waves,schedule", [(4, 14), (4, 29), (2, 29), (4, 30), (2, 31)])
def test_a_helper_may_finish_a_candidate_before_its_starter_goes_on(waves, schedule, monkeypatch):
    # candidates of one query and one stage: a helper that took the slot for the previous candidate's can run both operations of
    # the next one while the wavefront that started it sleeps
    monkeypatch.setenv("EST_EMU_SCHEDULE", str(schedule))
    monkeypatch.setenv("EST_WAVES_PER_CANDIDATE", str(waves))
    w = workloads.random_case(3, S=1, n=1, C=200)
    _check(w)
