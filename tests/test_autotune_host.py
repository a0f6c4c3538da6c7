"""The autotuner's candidates differ in what the library reads of a schedule (CPU)."""


def test_no_candidate_is_timed_twice():
    from paper_2005_13679_amd import autotune
    read = [(c["blocks_per_cu"], c["order"]) for c in autotune.CANDIDATES]
    assert len(set(read)) == len(read)
    # every key of a schedule is there, in the default and in each candidate
    assert all(set(c) == set(autotune.DEFAULT) for c in autotune.CANDIDATES)
    assert any(c == autotune.DEFAULT for c in autotune.CANDIDATES)
