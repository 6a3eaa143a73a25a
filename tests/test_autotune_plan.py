"""The tuner's candidates hold the library's own chunk plan (CPU): without it a
tuned workload could run slower than one that was not tuned."""

from paper_2410_18414_amd import autotune


def test_planned_chunk_is_a_candidate_of_every_other_knob():
    others = [k for k in autotune.KNOBS if k != "chunk"]
    all_of = {tuple(c[k] for k in others) for c in autotune.CANDIDATES}
    planned = {tuple(c[k] for k in others) for c in autotune.CANDIDATES if c["chunk"] == 0}
    assert planned == all_of and len(all_of) == 8
