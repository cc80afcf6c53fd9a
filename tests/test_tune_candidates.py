"""The autotuner times every setting that differs in what runs, once: the start
stagger does nothing at the default geometry (seg_log2 18, block 512)."""
import itertools

import pytest

from paper_2411_01964_amd import tune


@pytest.mark.parametrize("space", [tune.SPACE, tune.BATCH_SPACE, {"seg_log2": (17, 18), "block": (512,)},
                                   {"stagger": (0, 36)}])
def test_candidates_are_the_space_without_idle_repeats(space):
    timed = list(tune.candidates(space))
    seen = {tuple(sorted(k.items())) for k in timed}
    assert len(seen) == len(timed)
    names = list(space)
    for combo in itertools.product(*(space[n] for n in names)):
        knobs = dict(zip(names, combo))
        if knobs.get("seg_log2", 18) == 18 and knobs.get("block", 512) == 512 and 72 in space.get("stagger", ()):
            knobs["stagger"] = 72
        assert tuple(sorted(knobs.items())) in seen
        seen_as = [k for k in timed if all(k[n] == knobs[n] for n in names)]
        assert len(seen_as) == 1
    idle = [k for k in timed if k.get("seg_log2") == 18 and k.get("block") == 512 and "stagger" in k]
    assert all(k["stagger"] == 72 for k in idle)


def test_a_sweep_times_each_candidate_once(monkeypatch):
    monkeypatch.setattr(tune, "apply", lambda knobs: None)
    asked = []

    def run(knobs):
        asked.append(knobs)
        return float(len(asked)), "same"
    table = tune._sweep(tune.SPACE, run, False)
    assert asked == list(tune.candidates(tune.SPACE)) and len(table) == len(asked)
    assert table[0][1] == asked[0]
