"""What the host takes from the record of an earlier brick list (brick_fill,
fill_mode), compiled for the host: a record counts for the number of granules
that it names and for no other."""
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
