"""Register budgets that launches rely on, from the compiler's resource-usage
remarks: the segment kernels of the default launch shape and of two instances per
workgroup keep everything in registers at every degree, and the default ones up to
degree 7 in FP32 leave room for three wavefronts per SIMD (168 registers)."""
import csv
import os
import re

import pytest

from paper_2411_13507_amd import build


@pytest.fixture(scope="module")
def table():
    if not os.path.exists(build.RESOURCES):
        pytest.skip("library not built here")
    with open(build.RESOURCES) as fh:
        return {r["kernel"]: r for r in csv.DictReader(fh, delimiter="\t")}


@pytest.mark.parametrize("degree", range(3, 10))
@pytest.mark.parametrize("kernel", ["solve_kernelIfLi{}ELb0E", "solve_kernelIfLi{}ELb1E", "solve_kernelIdLi{}ELb1E",
                                    "solve_kernel_shapeILi{}ELb0ELi1ELi1E", "solve_kernel_shapeILi{}ELb1ELi1ELi1E",
                                    "solve_kernel_shapeILi{}ELb0ELi2ELi2E", "solve_kernel_shapeILi{}ELb1ELi2ELi2E"])
def test_no_scratch_at_any_degree(table, kernel, degree):
    rows = [r for k, r in table.items() if re.search(kernel.format(degree), k)]
    assert len(rows) == 1
    assert int(rows[0]["scratch"]) == 0
    if kernel.startswith("solve_kernelIf") and degree <= 7:
        assert int(rows[0]["vgpr"]) <= 168
