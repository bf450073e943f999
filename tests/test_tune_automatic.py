"""The tuner times the automatic plan, which alone may run windowed lanes, beside the
launch choices, and keeps it where it is the fastest."""
import json

import pytest

from paper_2101_02286_amd import cb, schemes, synth, tune

TRI = schemes.bands("tri6")


@pytest.mark.parametrize("one_partition", [False, True])
def test_automatic_plan_comes_first(one_partition):
    cands = tune.choices(TRI, 613, "fp64", strided=True, one_partition=one_partition)
    plan = cb.Plan(TRI, 613, host_only=True, **cands[0])
    assert len(plan.array(13, 1)) > 0  # windowed lanes, as without arguments
    plan.close()
    assert len(cands) > 1 and set(cands[0]) == set(cands[1])
    assert not one_partition or {c["partitions"] for c in cands} == {1}
    assert tune.choices(TRI, 613, "fp64", strided=True, max_candidates=3)[0] == dict.fromkeys(tune.AUTOMATIC, 0)


@pytest.mark.gpu
def test_tuned_ragged_lines(gpu, tmp_path):
    """Ragged strided lines run windowed lanes about twice as fast as any launch
    choice; what a cache holds from before the automatic plan was timed is not used."""
    f = synth.random_uniform((64, 613, 256), seed=1).to(gpu)
    cache = str(tmp_path / "cache" / "tune.json")
    (tmp_path / "cache").mkdir()
    old = tune._key(TRI, 613, "fp64", tuple(f.shape), 1, False)[len("v2|"):]
    json.dump({old: {"best": {"rows_per_lane": 8}, "table": []}}, open(cache, "w"))
    best, table = tune.tune(TRI, 613, f, 1, cache=cache, max_candidates=9)
    assert best == tune.AUTOMATIC and min(r["ms"] for r in table) == table[0]["ms"]
    assert len(json.load(open(cache))) == 2
    plan = tune.tuned_plan(TRI, 613, f, 1, cache=cache)
    assert len(plan.array(13, 1)) > 0
    plan.close()
