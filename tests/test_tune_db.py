"""The packaged tuning table follows from the timings kept beside it: every split, small-batch
plan and batch limit is what the tuner's rules give for them (a choice that was there
stays within tune.TIE of the best)."""
import json

import pytest

from paper_2209_01290_amd import tune


@pytest.fixture(scope="module")
def db():
    with open(tune.DEFAULT_DB) as f:
        return json.load(f)


@pytest.mark.parametrize("op", sorted(tune.OPS))
def test_choices_follow_from_timings(db, op):
    assert db["batch_words"] == list(tune.BATCH_WORDS)
    for n in range(1, 18):
        t, have = db["timings_ms"][op][str(n)], db["choices"][op][str(n)]
        assert sorted(int(c) for c in t) == tune.candidates(n)
        assert all(len(v) == len(tune.BATCH_WORDS) for v in t.values())
        assert tune._pick(t, str(have)) == str(have), (n, have, t)


@pytest.mark.parametrize("op", sorted(tune.OPS))
def test_small_plans_follow_from_timings(db, op):
    small = db["small"]
    for n in range(5, 18):
        t = small["latency_us"][op][str(n)]
        assert all(len(v) == 2 for v in t.values())           # one polynomial, eight
        have = "%d/%d" % tuple(small["choices"][op][str(n)])
        assert tune._pick(t, have) == have, (n, have, t)
        if n < tune.LIMIT_MIN_LOG2N:
            continue
        cross = {int(k.split("/")[2]): v for k, v in small["crossover_us"].items()
                 if k.startswith("%s/%d/" % (op, n))}
        limit = small["limits"][op][str(n)]
        want = tune.limit_of(cross, 1 << n, limit)
        assert want == limit or limit == tune.UNLIMITED and want == max(cross) << n, (n, limit, want)
    assert small["max_words"] == min(small["limits"]["polymul"].values())


def test_rules():
    t = {1: {"small": 1.0, "throughput": 2.0}, 2: {"small": 3.0, "throughput": 2.0}, 3: {"small": 2.0, "throughput": 3.0}}
    assert tune.limit_of(t, 8) in (8, 24) and tune.limit_of(t, 8, 1) == 8
    assert tune.limit_of({1: {"small": 3.0, "throughput": 2.0}}, 8) == 1          # never
    assert tune._pick({"a": [1.0, 2.0], "b": [1.01, 2.0]}, "b") == "b"
    assert tune._pick({"a": [1.0, 2.0], "b": [1.2, 2.0]}, "b") == "a"
