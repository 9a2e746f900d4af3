"""The committed counter summary in the form the benchmark reads: one section per
tile, each under the fingerprint of the sources it was taken on."""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("tile", [128, 256, 512])
def test_counter_sections_are_read(tile):
    sys.path.insert(0, ROOT)
    import bench
    text = open(bench.COUNTERS_FILE).read()
    prints = re.findall(r"^kernel_sources_sha256_16 = (\w+)$", text, re.M)
    assert len(prints) == len(re.findall(r"^tile = ", text, re.M)) == 3
    assert len(set(prints)) == 1
    kv = bench.read_counters(prints[0], tile)
    assert kv is not None
    assert kv["linearisations"] > 0 and kv["fabric_read_bytes"] > kv["fabric_write_bytes"] > 0
    assert bench.read_counters("0" * 16, tile) is None
