"""CPU: the barriers of the line kernels are reached by every wave of a block.

A block of the combined launch may have more waves than its lines need.  The
waves without work go through the same two barriers as the others, so the
barriers have to stand in the unit's own body, under no condition, and nowhere
else."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2202_09421_amd", "csrc")


def test_barriers_stand_in_the_unit_body():
    mixed = open(os.path.join(CSRC, "line4_mixed.h")).read()
    unit = open(os.path.join(CSRC, "line4_impl.h")).read()
    assert "__syncthreads" not in mixed
    assert [len(m) for m in re.findall(r"^( *)__syncthreads\(\);$", unit, re.M)] == [2, 2]
    assert unit.count("__syncthreads") == 2
