"""bench.py books every kernel that the library launches under the stage whose function launches it."""
import os
import re

import bench

SOURCE = os.path.join(os.path.dirname(bench.__file__), "paper_2312_08053_amd", "csrc", "kimad_api.hip")
STAGES = {"run_select_passes": "profile", "launch_small_profile": "profile", "run_single_pass": "profile",
          "enqueue_allocate": "allocate", "enqueue_compress": "compress"}


def test_kernels_are_booked_where_they_are_launched():
    text = open(SOURCE).read()
    bodies = re.split(r"^(?=[A-Za-z_][\w:<>\* ]* \**\w+\()", text, flags=re.M)
    seen = {}
    for body in bodies:
        name = re.match(r"[\w:<>\* ]+? \**(\w+)\(", body)
        if not name or name[1] not in STAGES:
            continue
        for kernel in re.findall(r'KLAUNCH\([^"]*"(k_\w+)"', body):
            if kernel != "k_zero16":
                seen.setdefault(name[1], set()).add(kernel)
                assert bench.stage_of(kernel) == STAGES[name[1]], (kernel, name[1])
    assert set(seen) == set(STAGES)
    assert len(set().union(*seen.values())) >= 20
