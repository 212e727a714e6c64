"""The level work item's groups, replayed symbolically on the CPU from the
device table the kernel receives (tests/cpp/group_plan.cpp links the
library's planner), must form exactly the product the oracle's trees define,
read every rank once and use every slot only after its value's stage."""

import os
import shutil
import subprocess
import sys

import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2109_12626_amd", "csrc")

# every remainder of groups of 7 on both layouts, then larger trees up to the
# most ranks with a group table
P_LIST = list(range(1, 140)) + [255, 256, 257, 288, 300, 511, 513, 1151, 1152,
                                1153, 2049, 4099, 65534]


@pytest.fixture(scope="module")
def replayed(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("groups") / "group_plan"
    subprocess.run([gxx, "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "cpp", "group_plan.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", str(out)],
                   check=True)
    res = subprocess.run([str(out)], input=" ".join(map(str, P_LIST)),
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[-200:]
    table = {}
    for line in res.stdout.splitlines():
        p, layout, expr = line.split(" ", 2)
        table[(int(p), layout)] = expr
    return table


def _expr(t, i):
    y = f"x{i}"
    if t.child0[i] is not None:
        y = f"({_expr(t, t.child0[i])}*{y})"
    if t.child1[i] is not None:
        y = f"({_expr(t, t.child1[i])}*{y})"
    return y


@pytest.mark.parametrize("layout", ["dual", "single"])
@pytest.mark.parametrize("p", P_LIST)
def test_groups_form_the_oracle_product(replayed, p, layout):
    sys.setrecursionlimit(10000)
    t = oracle.build_trees(p, layout=layout)
    want = _expr(t, t.roots[0])
    if len(t.roots) == 2:
        want = f"({want}*{_expr(t, t.roots[1])})"
    assert replayed[(p, layout)] == want
