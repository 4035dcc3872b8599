"""GPU tests of the batched forms: every windowed-kernel shape and launch form
against the oracle, plans (hipGraph capture of the whole forward) against the
eager calls, replay determinism with other work in between and with inputs
changed in place, and the autotuner's cache."""
import json
import os

import numpy as np
import pytest

from gpu_util import (OnDevice, assert_F_close, assert_mean_flux_root, assert_subset_flux,
                      assert_tau_close, gpu_normalise, gpu_tau, A_REL)
from oracle import oracle as O
from paper_1105_4747_amd import lyaf as L
from synth import fields

pytestmark = pytest.mark.gpu


def oracle_tau(w):
    return O.tau(w.delta, w.vpec, w.dv, w.T0, w.gamma, offsets=w.offsets, tau_ref=w.tau_ref,
                 delta_pivot=w.delta_pivot)


def ragged_mix(seed=41, S=24):
    """Ragged batch: short skewers (full-sum path and halo-duplicated staging),
    long ones, dv from 1 to 4 km/s."""
    return fields.ragged_workload("mix", S, 40, 3000, 1.0, 4.0, 1e4, 2.5e4, 1.1, 1.6, 1.0, 0.8,
                                  6.0, seed=seed)


@pytest.mark.parametrize("shape", range(L.NUM_SHAPES))
@pytest.mark.parametrize("persistent", [False, True])
def test_every_shape_and_launch_form(shape, persistent):
    from paper_1105_4747_amd import lyaf as L
    fl = L.FLAG_SHAPE(shape) | (L.FLAG_PERSISTENT if persistent else 0)
    for w in (fields.config1().subset(range(16)), ragged_mix()):
        print(f"case: {w.name} shape={shape} persistent={persistent}", flush=True)
        got = gpu_tau(w, flags=fl).cpu().numpy()
        assert_tau_close(got, oracle_tau(w), f"{w.name} shape {shape}")


def _plan(w, d, autotune=False, graph=True):
    import torch
    from paper_1105_4747_amd import lyaf as L
    ts = torch.empty(w.n_pix, device="cuda:0", dtype=torch.float32)
    F = torch.empty_like(ts)
    A = torch.empty((), device="cuda:0", dtype=torch.float64)
    p = L.Plan(d.delta, d.vpec, d.dv, d.T0, d.gamma, d.offsets, w.target_F, ts, F, A,
               tau_ref=w.tau_ref, delta_pivot=w.delta_pivot, window_k=w.window_k,
               autotune=autotune, graph=graph)
    return p, ts, F, A


def _eager(w, d):
    raw = gpu_tau(w, d=d)
    return gpu_normalise(raw, w.target_F)


@pytest.mark.parametrize("graph", [True, False])
def test_plan_replays_match_eager_bitwise(graph):
    import torch
    w = ragged_mix(seed=43)
    d = OnDevice(w)
    p, ts, F, A = _plan(w, d, graph=graph)
    print(f"case: plan graph={graph} {p.describe()}", flush=True)
    e_ts, e_F, e_A = _eager(w, d)
    for rep in range(3):
        # other work on the stream between replays
        junk = torch.randn(1 << 20, device="cuda:0").sum()
        ts.fill_(float("nan"))
        p.execute()
        torch.cuda.synchronize()
        assert torch.equal(ts, e_ts) and torch.equal(F, e_F) and torch.equal(A, e_A), rep
        del junk
    # new field contents at the same addresses
    d.delta.mul_(1.3)
    d.vpec.add_(5.0)
    p.execute()
    torch.cuda.synchronize()
    w2 = fields.Workload(w.name, d.delta.cpu().numpy(), d.vpec.cpu().numpy(), w.offsets, w.dv,
                         w.T0, w.gamma, w.target_F, w.window_k)
    e_ts, e_F, e_A = _eager(w2, OnDevice(w2))
    assert torch.equal(ts, e_ts) and torch.equal(F, e_F) and torch.equal(A, e_A)
    assert p.status() == 0
    raw_ref = oracle_tau(w2)
    A_g = float(A.cpu())
    assert_tau_close(ts.cpu().numpy() / A_g, raw_ref, "plan raw tau")
    _, F_ref, _ = O.normalise(raw_ref, w2.target_F)
    assert_F_close(F.cpu().numpy(), F_ref, "plan F")
    p.close()


def test_autotune_times_every_candidate_and_caches(tmp_path, monkeypatch):
    monkeypatch.setenv("LYAF_TUNE_CACHE", str(tmp_path / "tune.txt"))
    w = ragged_mix(seed=45)
    d = OnDevice(w)
    p, ts, F, A = _plan(w, d, autotune=True)
    info = p.describe()
    print(f"case: autotune {info}", flush=True)
    assert info["tuned"] and not info["from_cache"] and info["graph"]
    assert len(info["timings_us"]) == 2 * L.NUM_SHAPES
    lines = open(tmp_path / "tune.txt").read().split("\n")
    assert lines[0].startswith(info["key"] + " ")
    raw_ref = oracle_tau(w)
    A_g = float(A.cpu())
    assert_tau_close(ts.cpu().numpy() / A_g, raw_ref, "tuned raw tau")
    p.close()
    p2, ts2, F2, A2 = _plan(w, d, autotune=True)
    info2 = p2.describe()
    assert info2["from_cache"] and info2["key"] == info["key"]
    assert (info2["streams"], info2["targets_per_lane"], info2["tile"]) == \
        (info["streams"], info["targets_per_lane"], info["tile"])
    p2.close()


def test_tune_cache_rejects_entries_of_another_device_or_shape(tmp_path, monkeypatch):
    """A cached choice is reused only under its exact key (device name,
    compute-unit count, batch-shape buckets, window): entries written for
    another device, for another batch shape, or naming a shape the library
    does not have are ignored, and the plan tunes afresh."""
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LYAF_TUNE_CACHE", str(cache))
    w = ragged_mix(seed=47)
    d = OnDevice(w)
    p, *_ = _plan(w, d, autotune=True)
    key = p.describe()["key"]
    p.close()
    fields_ = key.split("|")
    assert fields_[0] == "v3" and fields_[1].startswith("gfx")
    other_dev = "|".join([fields_[0], "gfx000", *fields_[2:]])
    other_cus = "|".join([fields_[0], fields_[1], "cu1", *fields_[3:]])
    other_shape = "|".join([*fields_[:3], "S2^30", *fields_[4:]])
    cache.write_text(f"{other_dev} 1 0 1.0\n{other_cus} 1 0 1.0\n{other_shape} 1 0 1.0\n"
                     f"{key} {L.NUM_SHAPES} 0 1.0\n{key} -1 0 1.0\n{key} 0 2 1.0\n")
    p2, ts, F, A = _plan(w, d, autotune=True)
    info = p2.describe()
    print(f"case: stale tune cache {info}", flush=True)
    assert info["key"] == key and not info["from_cache"], "a stale or malformed entry was used"
    assert len(info["timings_us"]) == 2 * L.NUM_SHAPES
    assert_tau_close(ts.cpu().numpy() / float(A.cpu()), oracle_tau(w), "re-tuned raw tau")
    p2.close()
    # the re-tuned entry was appended under the exact key and is used next time
    assert cache.read_text().strip().split("\n")[-1].startswith(key + " ")
    p3, *_ = _plan(w, d, autotune=True)
    assert p3.describe()["from_cache"]
    p3.close()


def test_tune_cache_entries_saved_before_stay_in_use(tmp_path, monkeypatch):
    """A tuning file of an earlier library: its entry, under the key of the v3 shapes, is
    used, and the plan neither tunes again nor takes another shape."""
    import torch
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LYAF_TUNE_CACHE", str(cache))
    w = ragged_mix(seed=53)
    d = OnDevice(w)
    prop = torch.cuda.get_device_properties(0)
    head = (f"v3|{prop.gcnArchName.replace(':', '_')}|cu{prop.multi_processor_count}"
            f"|S2^{round(np.log2(w.n_skewers))}|N2^{round(np.log2(w.n_pix / w.n_skewers))}")
    cache.write_text("".join(f"{head}|R2^{r}|k6 3 0 1.0\n" for r in range(13)))
    p, ts, F, A = _plan(w, d, autotune=True)
    info = p.describe()
    print(f"case: saved tune entry {info['key']}", flush=True)
    assert info["from_cache"] and info["shape"] == 3 and info["persistent_grid"] == 0
    p.close()


def test_tuner_choice_follows_its_timings(tmp_path, monkeypatch):
    """The tuner keeps the fastest one-workgroup-per-item launch unless the
    persistent launch is faster by more than 2 %; every candidate is the
    median of 11 replays."""
    monkeypatch.setenv("LYAF_TUNE_CACHE", str(tmp_path / "tune.txt"))
    w = ragged_mix(seed=49)
    p, *_ = _plan(w, OnDevice(w), autotune=True)
    info = p.describe()
    p.close()
    t = info["timings_us"]
    grid = min((c for c in t if not c["persistent"]), key=lambda c: c["us"])
    pers = min((c for c in t if c["persistent"]), key=lambda c: c["us"])
    want = pers if pers["us"] < 0.98 * grid["us"] else grid
    print(f"case: tuner choice grid={grid} persistent={pers} chose shape {info['shape']} "
          f"persistent_grid {info['persistent_grid']}", flush=True)
    assert info["shape"] == want["variant"]
    assert (info["persistent_grid"] > 0) == bool(want["persistent"])


@pytest.mark.slow
def test_config3_plan_sampled():
    """20,000 ragged skewers through one tuned plan (persistent launch in a
    hipGraph); sampled skewers against the oracle; the rescaled tau must solve
    the mean-flux condition with A = 1 (a property of the GPU's own outputs),
    and F of the sampled skewers, each side normalising them on its own."""
    import torch
    w = fields.config3()
    d = OnDevice(w)
    p, ts, F, A = _plan(w, d, autotune=True)
    print(f"case: {w.name} plan {p.describe()}", flush=True)
    p.execute()
    torch.cuda.synchronize()
    A_g = float(A.cpu())
    ts_np = ts.cpu().numpy()
    # tau' is stored in float32, hence twice the A bar
    assert_mean_flux_root(ts_np, 1.0, w.target_F, "C3 plan rescaled tau", rel=2 * A_REL)
    lens = np.diff(w.offsets)
    rng = np.random.default_rng(33)
    pick = np.unique(np.concatenate([[int(np.argmin(lens)), int(np.argmax(lens))],
                                     rng.choice(w.n_skewers, 16, replace=False)]))
    sub = w.subset(pick)
    ref = oracle_tau(sub)
    sel = np.concatenate([np.arange(w.offsets[s], w.offsets[s + 1]) for s in pick])
    assert_tau_close(ts_np[sel] / A_g, ref, "C3 plan raw tau")
    assert_subset_flux(ts_np[sel] / A_g, ref, w.target_F, "C3 plan sampled F")
    p.close()
