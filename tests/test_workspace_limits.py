"""Scratch of the caller's own that holds barely one candidate, or fewer than there are: what fits is run, with the oracle's results.

The streams between operations get shorter rings where that makes a call fit, down to what each ring needs: a whole group of
batches that complete together, or a merge's windows.
"""
import types

import numpy as np
import pytest

import emu_lib
from oracle import oracle
from paper_1812_01776_amd import estimator as binding
from paper_1812_01776_amd import workloads


def _tensors(w, device):
    import torch
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a).view(dt).reshape(-1).copy()).to(device)
    return t(w.arrival_us, np.int32), t(w.visit_mask, np.int32), t(binding.pack_configs(w.cfg_hw, w.cfg_batch, w.cfg_replicas), np.uint8)


def _run(est, w, tensors, nbytes, device):
    """The results in a workspace of that many bytes, or None when the call refuses it."""
    import torch
    raw = torch.empty(nbytes + 256, dtype=torch.uint8, device=device)
    ws = raw[-raw.data_ptr() % 256:][:nbytes]
    stream = None if device != "cpu" else types.SimpleNamespace(cuda_stream=0)  # the emulation's "device" memory is host memory
    try:
        r = est.run_dev(*tensors, w.n_configs, w.slo_us, workspace_t=ws, stream=stream)
    except binding.EstimatorError as e:
        assert e.code == binding.EST_ENOMEM
        return None
    return {k: v.cpu().numpy() for k, v in r.items()}


def _smallest(est, w, tensors, device):
    """The smallest accepted workspace, to half a per cent."""
    lo, hi = 1024, 2048
    while _run(est, w, tensors, hi, device) is None:
        assert hi < 1 << 24
        lo, hi = hi, 2 * hi
    while hi - lo > max(64, hi // 200):
        mid = (lo + hi) // 128 * 64
        if _run(est, w, tensors, mid, device) is None:
            lo = mid
        else:
            hi = mid
    return hi


def _same(got, ref):
    assert np.array_equal(got["p99_us"].view(np.uint32).astype(np.uint64), ref["p99_us"])
    assert np.array_equal(got["miss_count"].view(np.uint32).astype(np.uint64), ref["miss_count"])
    assert np.array_equal(got["cost_uusd_hr"].view(np.uint64), ref["cost_uusd_hr"])


def _at_the_limit(w, est, device):
    tensors = _tensors(w, device)
    ref = oracle.run(w.parents, w.lat_us, w.cost_uusd_hr, w.arrival_us, w.visit_mask, w.cfg_hw, w.cfg_batch, w.cfg_replicas, w.slo_us)
    least = _smallest(est, w, tensors, device)
    for nbytes in (least, least + least // 2, 3 * least):
        _same(_run(est, w, tensors, nbytes, device), ref)
    assert est.workspace_bytes(w.n_queries, 1) >= least
    return least


def _uniform(parents, replicas, batch, n=20, C=6):
    S = len(parents)
    w = workloads.random_case(1, S=S, n=n, C=C, max_b=64)
    w.parents = parents
    w.visit_mask = np.full(n, 2**S - 1, np.uint32)
    w.cfg_batch = np.full((C, S), batch, np.uint8)
    w.cfg_replicas = np.full((C, S), replicas, np.uint16)
    return w


# What a call of 6 candidates and 20 queries needed when rings of 1,024 elements and more were the shortest, in bytes
FORMER_NEED = [([[], [0]], 1, 1, 21_990), ([[], [0]], 4, 8, 22_246), ([[], [0]], 16, 64, 46_821), ([[], [0]], 64, 64, 170_717),
               ([[], [0], [0], [0], [1, 2, 3]], 1, 1, 55_780), ([[], [0], [0], [0], [1, 2, 3]], 4, 8, 56_548),
               ([[], [0], [0], [0], [1, 2, 3]], 16, 64, 126_176), ([[], [0], [0], [0], [1, 2, 3]], 64, 64, 485_578)]


@pytest.mark.production_rings
@pytest.mark.parametrize("parents,replicas,batch,former", FORMER_NEED)
def test_what_held_one_candidate_still_does_emulated(parents, replicas, batch, former):
    w = _uniform(parents, replicas, batch)
    assert _at_the_limit(w, emu_lib.make(w), "cpu") <= former


@pytest.mark.production_rings
@pytest.mark.parametrize("schedule", [None, 1])
@pytest.mark.parametrize("seed", range(4))
def test_tight_rings_match_oracle_emulated(seed, schedule, monkeypatch):
    # traces many times the rings' length: forks, joins, filters and completions that tie, full batch groups included
    if schedule is not None:
        monkeypatch.setenv("EST_EMU_SCHEDULE", str(seed))
    w = workloads.random_case(seed + 60, n=500, C=2, max_b=[4, 16, 64][seed % 3], max_r=[2, 16][seed % 2], tie_heavy=seed % 2 == 0,
                              small_times=seed == 3)
    _at_the_limit(w, emu_lib.make(w), "cpu")


def _many(C):
    w = workloads.random_case(7, S=4, n=300, C=C, dag="linear")
    w.cfg_replicas = np.maximum(w.cfg_replicas, 2)
    return w


@pytest.mark.production_rings
def test_rings_get_shorter_where_that_holds_more_candidates_emulated():
    w = _many(8)
    est = emu_lib.make(w)
    tensors = _tensors(w, "cpu")
    _run(est, w, tensors, 1 << 24, "cpu")
    assert est.stats()["n_slots"] == 8
    per_long = est.stats()["workspace_bytes"] // 8
    assert per_long > 4 * 8192 * 8  # four rings of 8,192 elements
    _run(est, w, tensors, 4 * per_long, "cpu")
    assert est.stats()["n_slots"] == 8 and est.stats()["workspace_bytes"] < 4 * per_long


@pytest.mark.gpu
@pytest.mark.production_rings
@pytest.mark.parametrize("parents,replicas,batch,former", FORMER_NEED)
def test_what_held_one_candidate_still_does(parents, replicas, batch, former):
    w = _uniform(parents, replicas, batch)
    assert _at_the_limit(w, binding.Estimator(w.parents, w.lat_us, w.cost_uusd_hr), "cuda") <= former


@pytest.mark.gpu
@pytest.mark.production_rings
@pytest.mark.parametrize("seed", range(12))
def test_tight_rings_match_oracle(seed):
    w = workloads.random_case(seed + 60, n=4000, C=5, max_b=[4, 16, 64][seed % 3], max_r=[2, 16][seed % 2], tie_heavy=seed % 2 == 0,
                              small_times=seed % 5 == 0)
    _at_the_limit(w, binding.Estimator(w.parents, w.lat_us, w.cost_uusd_hr), "cuda")
