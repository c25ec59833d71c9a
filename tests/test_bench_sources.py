"""The benchmark takes a recorded memory traffic only for the sources it was measured with: the list it hashes must hold
everything the matrix-core steppers are compiled from (the public header, mostly prose, aside)."""
import os
import re

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2203_14742_amd", "csrc")


def included(name, seen):
    if name not in seen and not name.endswith("cil.h") and os.path.exists(os.path.join(CSRC, name)):
        seen.add(name)
        for inc in re.findall(r'#include "([^"]+)"', open(os.path.join(CSRC, name)).read()):
            included(inc, seen)
    return seen


def test_traffic_is_bound_to_every_source_of_the_steppers():
    need = set()
    for f in sorted(os.listdir(CSRC)):
        if re.fullmatch(r"stepper_(mm_.*|split)\.hip", f):
            included(f, need)
    assert len(need) >= 8 and need | {"stepper.hip"} <= set(bench.STEPPER_SOURCES), sorted(need - set(bench.STEPPER_SOURCES))
    for f in bench.STEPPER_SOURCES:
        assert os.path.exists(os.path.join(CSRC, f)), f
