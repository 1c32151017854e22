"""A search of a walk table (csrc/walk_common.hpp, Probe) visits eight different buckets before
it gives the key to the overflow table, whatever the table's size."""
import re

from test_probe_lanes import clang, run_model  # noqa: F401


def test_a_search_visits_different_buckets(clang, tmp_path):  # noqa: F811
    out = run_model(clang, tmp_path, "strides")
    print(out)
    counts = re.findall(r": (\d+) different", out)
    assert len(counts) == 17 and set(counts) == {"8"}
