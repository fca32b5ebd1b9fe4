"""The hash that ties kept traffic counters to the kernels they were taken of
covers every source that decides what those kernels do."""
import glob
import os
import re
import shutil

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1705_08266_amd", "csrc")


def _included(path, seen):
    """The local headers that a source takes in, by way of others too."""
    with open(path) as f:
        for name in re.findall(r'^#include "(dwt2_\w+\.hpp)"', f.read(), re.M):
            if name not in seen:
                seen.add(name)
                _included(os.path.join(CSRC, name), seen)
    return seen


def test_every_source_of_the_heads_and_tails_counts(tmp_path):
    names = {"dwt2_api.hip"}
    for inst in glob.glob(os.path.join(CSRC, "inst_*.hip")):
        _included(inst, names)
    assert {"dwt2_stream.hpp", "dwt2_head_tile.hpp", "dwt2_table.hpp"} < names
    for name in sorted(names):
        copy = tmp_path / name.replace(".", "_")
        shutil.copytree(CSRC, copy)
        assert bench.kernel_source_sha(str(copy)) == bench.kernel_source_sha()
        with open(copy / name, "a") as f:
            f.write("// changed\n")
        assert bench.kernel_source_sha(str(copy)) != bench.kernel_source_sha(), name
