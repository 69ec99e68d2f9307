"""What the host takes from the record of an earlier brick list (brick_fill,
fill_mode), compiled for the host: a record counts for the number of granules
that it names and for no other, and groups of bricks are taken where they are
full enough."""
import os
import subprocess

from paper_2504_00745_amd import build

MAIN = r"""
#include <cstdio>
#include "gic_launch.hpp"
using namespace gic;
int main()
{
    DevParams P = {};
    P.cell = 2.0;
    P.r_max = 1.0;  // 64 granules a brick expected
    BrickSeen seen = {100, 5000};
    BrickList B = {};
    B.seen = &seen;
    B.seen_n = 7000;  // a list of 7,000 granules followed; its record has not arrived
    for (int64_t n : {5000, 7000, 4999}) {
        const BrickFill f = brick_fill(P, n, B);
        printf("%lld %d %.17g\n", (long long)n, f.known ? 1 : 0, f.avg);
    }
    B.seen = nullptr;
    const BrickFill f = brick_fill(P, 5000, B);
    printf("0 %d %.17g\n", f.known ? 1 : 0, f.avg);
}
"""


def run(d, main, *args):
    src, exe = d / "main.hip", d / "main"
    src.write_text(main)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(os.path.dirname(build.HERE), "include"), "-o",
                    str(exe), str(src)], check=True, capture_output=True)
    out = subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True).stdout
    return [[float(w) for w in line.split()] for line in out.splitlines()]


def test_record_of_another_bed_is_not_taken(tmp_path):
    assert run(tmp_path, MAIN) == [[5000, 1, 50.0], [7000, 0, 64.0], [4999, 0, 64.0], [0, 0, 64.0]]


MODES = r"""
#include <cstdio>
#include "gic_launch.hpp"
using namespace gic;
int main()
{
    DevParams P = {};
    P.cell = 2.0;
    P.r_max = 1.0;
    BrickList B = {};
    const int32_t rec[][4] = {{20000, 1000000, 4000, 8 * 4000}, {20000, 1000000, 4000, 5 * 4000}, {20000, 1000000, 4000, 19999},
                              {20000, 1000000, 4000, 4000}, {20000, 1000000, 0, 0}, {4096, 300000, 700, 5000},
                              {4095, 300000, 700, 5000}, {20000, 1000001, 4000, 8 * 4000}, {10000, 1000000, 4000, 8 * 4000}};
    for (auto &r : rec) {
        BrickSeen seen = {r[0], r[1], r[2], r[3], 0, 0};
        B.seen = &seen;
        printf("%d\n", (int)fill_mode(P, r[1] == 1000001 ? 1000000 : r[1], B, kGroupBricks));
    }
}
"""
BLOCK, WAVE, BOTH, GROUP = range(4)


def test_groups_where_they_are_full(tmp_path):
    assert [m for m, in run(tmp_path, MODES)] == [GROUP, GROUP, WAVE, WAVE, WAVE, GROUP, WAVE, BOTH, BLOCK]


SORTS = r"""
#include <cstdio>
#include "gic_launch.hpp"
using namespace gic;
int main()
{
    BrickSeen seen = {};
    BrickList B = {};
    B.seen = &seen;
    auto form = [&](int64_t n, int64_t K, bool shuffled) { return sort_by_digits(n, K, B, sort_limit(n, shuffled)) ? 1 : 0; };
    // nothing known: from the mean of the box, and a large bed is taken to be shuffled
    printf("%d %d %d %d %d\n", form(4096, 4096, true), form(70001, 64, true), form(524288, 65536, true),
           form(524289, 1 << 20, true), form(524289, 1 << 20, false));
    // known: half of the granules in cells beyond the limit
    seen = {1000, 200000, 0, 0, 200000, 100000};
    printf("%d %d", form(200000, 64000, true), form(200001, 64000, true));
    seen.dense = 100001;
    printf(" %d %d\n", form(200000, 64000, true), form(200000, 64000, false));
    // a rollout's
    printf("%d %d\n", sort_by_digits(1048576, 1 << 20, B, sort_limit(1048576, true, true)) ? 1 : 0,
           sort_by_digits(1048577, 1 << 20, B, sort_limit(1048577, true, true)) ? 1 : 0);
    // buffers: tiles and digits
    printf("%lld %lld %lld %d %d %d %d\n", (long long)sort_tiles_max(1), (long long)sort_tiles_max(262144),
           (long long)sort_tiles_max(16777216), sort_passes(64), sort_passes(257), sort_passes(65537), sort_passes(16777217));
}
"""


def test_sorts_by_digits_where_faster(tmp_path):
    assert run(tmp_path, SORTS) == [[0, 1, 0, 1, 0], [0, 0, 1, 1], [0, 1], [1, 1024, 8192, 1, 2, 3, 4]]
