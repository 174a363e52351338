"""Launch shapes, which the host computes for every call: a small program over the
library's internal header prints them (no GPU call is made here)."""
import os
import shutil
import subprocess

import pytest

from paper_2111_02912_amd import _lib, build

PROG = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "kbn_internal.h"
int main(int, char **v) {
    if (!std::strcmp(v[1], "xcd")) {  // n: padded row and the subproblem of each of its workgroups
        const int64_t p = kbn_xcd_padded(std::atoll(v[2]));
        std::printf("%lld", (long long)p);
        for (int x = 0; x < p; ++x) std::printf(" %d", kbn_xcd_run_index(x, (int)p));
    }
    std::printf("\n");
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(PROG)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", build.INCLUDE, "-I",
                    build.CSRC, str(d / "rules.cpp"), _lib.LIB_PATH, "-Wl,-rpath," + os.path.dirname(_lib.LIB_PATH),
                    "-o", str(d / "rules")], check=True)

    def run(*args):
        r = subprocess.run([str(d / "rules"), *map(str, args)], capture_output=True, text=True, check=True)
        return [int(x) for x in r.stdout.split()]
    return run


@pytest.mark.parametrize("n", [1, 7, 8, 15, 63, 64, 65, 71, 72, 127, 128, 385, 1000, 4097])
def test_gather_rows_hold_every_subproblem_once(rules, n):
    """A row of workgroups covers the subproblems once each, in whole rounds of
    the eight XCDs and with no more idle workgroups than that takes."""
    padded, *index = rules("xcd", n)
    assert padded % 8 == 0 and n <= padded < n + 8
    assert sorted(index) == list(range(padded))


def test_launches_compute_no_splits():
    """The column passes' thread counts are constants of their kernels, not
    searched for again at every launch."""
    if not shutil.which("nm"):
        pytest.skip("no nm")
    names = subprocess.run(["nm", "-C", _lib.LIB_PATH], capture_output=True, text=True, check=True).stdout
    assert "k_any_cols" in names
    for f in ("col_threads(", "row_lines(", "split_cost(", "split_radices("):
        assert f not in names, f
