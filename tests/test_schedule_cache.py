"""The autotuner's cache mirrors the schedule table: a class that went back to the
built-in rule leaves no record that would bring its old shape back."""
from paper_2510_25938_amd import lj


def merged(entry, offsets, min_class):
    b = lj.ClusterBatch(offsets, device="cpu")
    lj._merge_schedules(entry, b, {"eval": (1, 1, 0.1), "min_large": None, "min_ms": 1.0,
                                   "min_class": min_class})
    return entry


def test_class_on_the_rule_leaves_the_cache():
    entry = {"min_class": {"38": {"0": 0}, "40": {"0": 4}, "20": {"0": 2}, "100": {"0": 4, "1": 0}}}
    merged(entry, [0, 38, 76], {})  # 38 and 40 share a table key; 20 and 100 have others
    assert entry["min_class"] == {"20": {"0": 2}, "100": {"0": 4, "1": 0}}
    assert entry["eval"] == {"64": [1, 1]}


def test_tuned_classes_replace_and_absent_ones_stay():
    entry = {"min_class": {"150": {"0": 4, "1": 1, "2": 0}, "140": {"1": 0}}}
    merged(entry, [0, 150, 250], {1: 0, 2: 1})  # no class-0 cluster in the batch
    assert entry["min_class"] == {"150": {"0": 4, "1": 0, "2": 1}}


def test_first_record_and_no_minimiser():
    entry = {}
    merged(entry, [0, 13], {0: 3})
    assert entry["min_class"] == {"13": {"0": 3}} and entry["eval"] == {"16": [1, 1]}
    b = lj.ClusterBatch([0, 2000], device="cpu")  # above the minimiser's limit
    lj._merge_schedules(entry, b, {"eval": (16, 2, 0.1), "min_large": None, "min_ms": None,
                                   "min_class": {}})
    assert entry["min_class"] == {"13": {"0": 3}} and entry["eval"]["2048"] == [16, 2]
