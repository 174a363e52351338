"""Launch shapes, which the host computes for every call: a small program over the
library's internal header prints them (no GPU call is made here)."""
import ctypes
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
    if (!std::strcmp(v[1], "xcdrow")) {  // n, row: the subproblem of each workgroup of that row
        const int64_t p = kbn_xcd_padded(std::atoll(v[2]));
        for (int x = 0; x < p; ++x) std::printf(" %d", kbn_xcd_run_index(x, (int)p, std::atoi(v[3])));
    }
    if (!std::strcmp(v[1], "gather")) {  // D J M channels weights K.. T..: staged, blocks, channels per group, groups
        KbnGeom g = {};
        g.D = std::atoi(v[2]);
        g.J = std::atoi(v[3]);
        g.ntiles = 1;
        for (int d = 0; d < g.D; ++d) {
            g.K[d] = std::atoi(v[7 + d]);
            g.T[d] = std::atoi(v[7 + g.D + d]);
            g.nt[d] = (g.K[d] + g.T[d] - 1) / g.T[d];
            g.ntiles *= g.nt[d];
        }
        const KbnGatherShape sh = kbn_gather_shape(g, std::atoll(v[4]), std::atoi(v[5]), std::atoi(v[6]));
        std::printf("%d %d %d %d", (int)sh.staged, (int)sh.blocks, sh.cg, sh.groups);
    }
    if (!std::strcmp(v[1], "most")) {  // blocks, pairs: 0 if the groups of every smaller number of pairs fit
        const int64_t b = std::atoll(v[2]), n = std::atoll(v[3]);
        int bad = 0;
        for (int staged = 0; staged < 2; ++staged)
            for (int64_t k = 1; k <= n; ++k) {
                const int64_t g = kbn_gather_groups(b, k, staged);
                bad += g < 1 || g > k || g > kbn_gather_groups_most(b, n, staged);
            }
        std::printf("%d", bad);
    }
    if (!std::strcmp(v[1], "counts"))  // sort tiles, owner tiles, M..: integers of the index pass
        for (int i = 4; v[i]; ++i)
            std::printf("%lld ", (long long)kbn_points_counts_size(std::atoll(v[i]), std::atoi(v[2]), std::atoi(v[3])));
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


@pytest.mark.parametrize("n", [1, 5, 8, 17, 64, 70, 385])
def test_gather_rows_take_turns_on_the_xcds(rules, n):
    """Eight rows (channel groups) give every XCD, the workgroup's position modulo
    eight, the same subproblems, of which the last may not exist."""
    rows = [rules("xcdrow", n, r) for r in range(8)]
    for r in rows:
        assert sorted(r) == list(range(len(r)))
    per_xcd = [sorted(s for r in rows for s in r[x::8]) for x in range(8)]
    assert all(p == per_xcd[0] for p in per_xcd)
    assert rules("xcdrow", n, 65535 * 8) == rows[0]


@pytest.mark.parametrize("nch", [1, 2, 3, 6, 7, 13, 20, 26, 27, 60, 200])
def test_direct_gather_takes_one_round_of_workgroups_or_many(rules, nch):
    """Point blocks without an LDS region: a workgroup row per channel, unless that
    is between one and four rounds of resident workgroups."""
    staged, blocks, cg, groups = rules("gather", 3, 8, 40000, nch, 1, 80, 96, 72, 8, 8, 8)
    assert not staged and blocks == 157
    if blocks * nch <= 1024:
        assert cg == 1 and groups == nch
    elif blocks * nch < 4096:
        assert cg > 1 and blocks * groups <= 1024
    else:
        assert blocks * groups > 4096 or groups == nch


@pytest.mark.parametrize("blocks", [1, 3, 8, 100, 157, 512, 1023, 1024, 1025, 3000, 8191, 8192, 20000])
@pytest.mark.parametrize("nbc", [1, 2, 7, 64, 1000, 9000])
def test_workspace_holds_the_groups_of_every_smaller_chunk(rules, blocks, nbc):
    """An omega-Jacobian keeps one partial gradient per channel group in a
    workspace sized by the largest chunk of a call."""
    assert rules("most", blocks, nbc) == [0]


# (M, image-coil pairs, weights, K, T): one wave of subproblems and many, few
# pairs and many
@pytest.mark.parametrize("M,nbc,nw,K,T", [
    (2000000, 2, 2, (512, 512), (32, 32)), (8192, 64, 2, (128, 128), (32, 32)), (3000, 400, 2, (96, 96), (32, 32)),
    (30000, 8, 2, (384, 384), (16, 16)), (32768, 256, 1, (512, 512), (32, 32)), (150000, 4, 3, (150, 180, 128), (8, 8, 8)),
    (20480, 64, 1, (400, 400), (32, 32)), (3000, 200, 1, (400,), (256,)),
])
def test_gather_groups_keep_pairs_once_the_gpu_is_filled(rules, M, nbc, nw, K, T):
    staged, blocks, cg, groups = rules("gather", len(K), 6, M, nbc * nw, nw, *K, *T)
    assert cg % nw == 0 and (groups - 1) * cg < nbc * nw <= groups * cg
    fill = -(-2048 // blocks)  # groups that fill the GPU
    assert groups <= fill or cg // nw >= 2
    if nbc >= 4 * 32:  # many pairs: several rounds of workgroups
        assert blocks * groups >= min(8192, blocks * nbc // 8)


@pytest.mark.parametrize("tiles", [(6992, 7000), (100, 100), (256, 4096), (13824, 13824), (32768, 110592)])
def test_buffers_of_more_samples_hold_fewer(rules, tiles):
    """A plan that goes back and forth between sample counts keeps the buffers of
    the larger one."""
    M = sorted({int(1.07 ** k) for k in range(30, 240)} | {152576, 160000} | {1 << k for k in range(8, 24)})
    n = rules("counts", *tiles, *M)
    assert n == sorted(n)


@pytest.mark.parametrize("tile,as_tile", [(9, 13), (10, 14), (4, 8), (7, 8), (8, 8), (16, 16)])
def test_only_matrix_core_tiles_may_be_many(tile, as_tile):
    """384^3 grids: owner tiles that no matrix-core spread takes stay below the
    rows of a grid, and those smaller than its 8 cells grow to them.  (A plan's
    bytes count its tiles; J = 4 lets a tile have 4 cells.)"""
    def footprint(t):
        o, out = _lib.KbnOpts(), ctypes.c_int64()
        o.sigma, o.J, o.spread_tile = 2.0, 4, t
        _lib.check(_lib.lib().kbn_plan_footprint(3, (ctypes.c_int64 * 3)(192, 192, 192), ctypes.byref(o), 10, 1, 1, 0,
                                                 ctypes.byref(out)), "kbn_plan_footprint")
        return out.value
    assert footprint(tile) == footprint(as_tile)


def test_launches_compute_no_splits():
    """The column passes' thread counts are constants of their kernels, not
    searched for again at every launch."""
    if not shutil.which("nm"):
        pytest.skip("no nm")
    names = subprocess.run(["nm", "-C", _lib.LIB_PATH], capture_output=True, text=True, check=True).stdout
    assert "k_any_cols" in names
    for f in ("col_threads(", "row_lines(", "split_cost(", "split_radices("):
        assert f not in names, f
