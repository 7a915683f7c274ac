"""The recorded HBM counters hold for the sources that bench.py hashes: those of the
measured step's kernels, with every local header that they include."""
import os
import re

import bench


def test_headers_of_hashed_sources_are_hashed():
    hashed = {os.path.basename(f) for f in bench.TRAFFIC_SOURCES}
    assert {"match.hip", "tree.hip", "sort_scan.hip"} <= hashed
    for rel in bench.TRAFFIC_SOURCES:
        path = os.path.join(bench.ROOT, rel)
        with open(path) as f:
            for name in re.findall(r'#include "([^"]+)"', f.read()):
                if os.path.exists(os.path.join(os.path.dirname(path), name)):
                    assert name in hashed, (rel, name)
