"""The tuner's search on the host: each sample count of a class is planned once,
and nothing is chosen by settings that no kernel reads."""
from paper_2609_30533_amd import autotune


def test_only_sample_counts_are_searched(monkeypatch):
    runs = []

    def score(problems, samples, lanes, budget_ms):
        runs.append(samples)
        # a later run of the same setting is a little faster, as timing noise may be
        return abs(samples - 250) - 0.1 * len(runs), len(problems)

    monkeypatch.setattr(autotune, "score", score)
    monkeypatch.setattr(autotune, "tuning_problems", lambda key, n: ["p"] * n)
    table = autotune.tune(["d2-o8", "d6-o16"], n_problems=3, log=lambda m: None)
    assert runs == list(autotune.SAMPLES) * 2
    for e in table.values():
        assert e["samples"] == 256
        assert e["lanes_bridge"] == autotune.DEFAULT["lanes_bridge"] in autotune.LANES
        assert e["lanes_extension"] == autotune.DEFAULT["lanes_extension"]
