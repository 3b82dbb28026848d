"""Host logic of the autotuner's choice (no GPU): the fastest setting wins
unless another lies within the tie margin and departs less from the
kernel's defaults (its own staging batch, heaviest-first launches)."""
from paper_2409_09295_amd import autotune as A


def _settings():
    return [(p, st, name) for name in A.SCHEDULES for p in A.CHOICES for st in A.STAGES]


def _table(kernel, times):
    t = {A._label(kernel, *c): 1.0 for c in _settings()}
    t.update({A._label(kernel, *c): v for c, v in times.items()})
    return t


def test_fastest_setting_wins_outside_the_tie_margin():
    t = _table("bwd", {(4, 1, "persistent"): 0.50, (4, 2, "heaviest_first"): 0.52})
    assert A._pick(_settings(), t, "bwd") == (4, 1, "persistent")


def test_ties_resolve_to_the_kernel_defaults():
    # within the margin: the backward's default batch at 4 pixels per lane is 2 splats
    t = _table("bwd", {(4, 1, "heaviest_first"): 0.700, (4, 2, "heaviest_first"): 0.705})
    assert A._pick(_settings(), t, "bwd") == (4, 2, "heaviest_first")
    # the forward's default at 4 pixels per lane is 1 splat; heaviest first beats persistent
    t = _table("fwd", {(4, 1, "persistent"): 0.340, (4, 1, "heaviest_first"): 0.342,
                       (4, 2, "heaviest_first"): 0.341})
    assert A._pick(_settings(), t, "fwd") == (4, 1, "heaviest_first")


def test_ties_prefer_the_faster_among_equally_default_settings():
    t = _table("fwd", {(2, 2, "heaviest_first"): 0.400, (4, 1, "heaviest_first"): 0.401})
    assert A._pick(_settings(), t, "fwd") == (2, 2, "heaviest_first")


def test_default_batches_match_the_library():
    """The tuner's notion of each kernel's default staging batch is the one
    the launch code falls back to when GS_TUNE_*_STAGE is 0."""
    import os
    import re
    csrc = os.path.join(os.path.dirname(A.__file__), "csrc")
    for kernel, src, key in (("fwd", "render_fwd.hip", "GS_TUNE_FWD_STAGE"),
                             ("bwd", "render_bwd.hip", "GS_TUNE_BWD_STAGE")):
        text = open(os.path.join(csrc, src)).read()
        m = re.search(r"stage_per_thread\(tuning\(" + key + r"\),\s*ppl == (\d) \? (\d) : (\d)\)", text)
        assert m, src
        ppl, hit, other = (int(x) for x in m.groups())
        lib = {p: hit if p == ppl else other for p in A.CHOICES}
        assert A.DEFAULT_STAGE[kernel] == lib, (kernel, A.DEFAULT_STAGE[kernel], lib)


def _tune(monkeypatch, tmp_path, times):
    """tune() on made-up times: times[(kernel, ppl)] of every stage and schedule, ppl 0
    for the launch's own choice."""
    from paper_2409_09295_amd import gs
    monkeypatch.setattr(A, "_key", lambda step: "workload")
    monkeypatch.setattr(A, "time_config",
                        lambda step, fwd, bwd, reps=3, **kw: (times["fwd", fwd], times["bwd", bwd]))
    try:
        a = A.tune(None, cache=str(tmp_path / "tune.json"))
        set_a = [gs.gs_get_tuning_setting(k) for k in range(6)]
        A.apply(0, 0)
        b = A.tune(None, cache=str(tmp_path / "tune.json"))
        set_b = [gs.gs_get_tuning_setting(k) for k in range(6)]
    finally:
        A.apply(0, 0)
    assert not a["cached"] and b["cached"] and set_a == set_b
    assert {k: v for k, v in a.items() if k != "cached"} == {k: v for k, v in b.items() if k != "cached"}
    return a, set_a


def test_the_launch_keeps_its_choice_where_no_setting_is_as_fast(monkeypatch, tmp_path):
    """Few tiles: the backward that the launch chooses is one that no setting names."""
    times = {(k, p): 0.066 + 0.01 * p for k in ("fwd", "bwd") for p in A.CHOICES}
    times.update({("fwd", 0): 0.0755, ("bwd", 0): 0.044})
    best, setting = _tune(monkeypatch, tmp_path, times)
    assert best["bwd_launch_choice"] and best["bwd_ms"] == 0.044 and setting[1] == setting[5] == 0
    assert not best["fwd_launch_choice"] and setting[0] == 1 and best["fwd_ms"] == times["fwd", 1]


def test_a_setting_is_pinned_where_it_ties_or_wins(monkeypatch, tmp_path):
    times = {(k, p): 0.7 - 0.05 * p for k in ("fwd", "bwd") for p in A.CHOICES}
    times.update({("fwd", 0): 0.495, ("bwd", 0): 0.62})
    best, setting = _tune(monkeypatch, tmp_path, times)
    assert not best["fwd_launch_choice"] and not best["bwd_launch_choice"]
    assert setting[:2] == [4, 4] and best["fwd_ppl"] == best["bwd_ppl"] == 4
