"""The lattices of _pass_cases.py plan the marches they stand for (host only: the plan
is compiled by itself and asked for 256 compute units)."""
import os
import subprocess

import pytest

from _pass_cases import MARCHES
from paper_2307_11752_amd import build

SIZE = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
MAIN = r"""
#include <cstdio>
#include "handle.hpp"
int main() {
  int nx, ny, nz, s, walls;
  while (scanf("%d %d %d %d %d", &nx, &ny, &nz, &s, &walls) == 5) {
    const lbm::PopIndex L = pop_index(19, (size_t)nx * ny * nz, s);
    const PairPlan P = lbm_detail::make_pair_plan(nx, ny, nz, s, walls != 0, L, 256);
    printf("%d %d %d %d %u\n", P.use, P.geom.ZC, P.small, P.separable, L.bstride);
  }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.hip", d / "plan"
    src.write_text(MAIN)
    cmd = [build.hipcc(), f"--offload-arch={build.ARCH}", "-O1", "-std=c++17",
           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(src),
           os.path.join(build.CSRC, "pair_plan.hip"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    asked = "".join("%d %d %d %d %d\n" % (*shape, SIZE[st], walls) for shape, st, walls, *_ in MARCHES)
    r = subprocess.run([str(exe)], input=asked, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]


@pytest.mark.parametrize("k", range(len(MARCHES)))
def test_marches(plans, k):
    shape, storage, walls, planes, small, separable = MARCHES[k]
    use, zc, is_small, is_separable, bstride = plans[k]
    assert use and zc >= planes, (shape, storage, zc)
    assert (bool(is_small), bool(is_separable)) == (small, separable), (shape, storage)
    assert bstride > 0  # blocked placement


def test_both_parities_of_a_march(plans):
    # the loop takes two planes at a time and one to three follow it
    assert {p[1] % 2 for p in plans} == {0, 1}
