"""The workgroup-to-group map of the group kernels, on the host: every group of a
box is taken by one workgroup, and the groups of a sheet one group thick, normal
to any axis, spread over the eight XCDs (workgroups go to them in turn) and over
the four shader engines of each (its workgroups go to them in turn)."""
import os
import subprocess

import pytest

from paper_2504_00745_amd import build

MAIN = r"""
#include <cstdio>
#include "gic_device.hpp"
int main(int, char **av)
{
    const int32_t ng[3] = {atoi(av[1]), atoi(av[2]), atoi(av[3])};
    gic::DevParams P = {};
    for (int a = 0; a < 3; ++a) P.ng[a] = ng[a];
    for (unsigned b = 0; b < gic::group_grid(P); ++b) printf("%lld\n", (long long)gic::group_at(ng, b).id);
}
"""


@pytest.fixture(scope="module")
def group_map(tmp_path_factory):
    d = tmp_path_factory.mktemp("map")
    src, exe = d / "map.hip", d / "map"
    src.write_text(MAIN)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(os.path.dirname(build.HERE), "include"), "-o",
                    str(exe), str(src)], check=True, capture_output=True)
    return lambda ng: [int(s) for s in subprocess.run([str(exe), *map(str, ng)], check=True, capture_output=True,
                                                      text=True).stdout.split()]


@pytest.mark.parametrize("ng", [(1, 1, 1), (2, 2, 2), (13, 12, 14), (10, 6, 9), (7, 5, 3), (3, 8, 8), (64, 8, 64), (8, 64, 64),
                                (64, 64, 8), (16, 16, 16), (64, 12, 64), (32, 31, 30)])
def test_every_group_once_and_sheets_spread(group_map, ng):
    g = group_map(ng)
    assert sorted(v for v in g if v >= 0) == list(range(ng[0] * ng[1] * ng[2]))
    for axis in range(3):
        for at in {0, ng[axis] // 2, ng[axis] - 1}:
            xcd, engine = [0] * 8, [0] * 4
            for b, v in enumerate(g):
                if v >= 0 and (v % ng[0], v // ng[0] % ng[1], v // (ng[0] * ng[1]))[axis] == at:
                    xcd[b % 8] += 1
                    engine[b // 8 % 4] += 1
            if sum(xcd) >= 512:  # (smaller sheets fill part of the chip only)
                assert 8 * max(xcd) <= 1.7 * sum(xcd), (axis, at, xcd)
                assert 4 * max(engine) <= 1.7 * sum(engine), (axis, at, engine)
