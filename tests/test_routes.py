"""Which kernel takes a call (csrc/routes.h), held against measured times: for
each instrument a size at which the group kernels were measured to be the
faster ones and one at which a pixel per lane was (times in the header).  The
header needs no HIP: a small program prints its answers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0901_2702_amd", "csrc")
ANY = 2 ** 63 - 1

# (band, points, chunks, use, max_iter, faster in groups, faster in lanes)
FITS = [
    (0, 7, 1, "PLAIN", 50, 8192, 24576),
    (0, 11, 1, "PLAIN", 50, 8192, 32768),
    (0, 19, 1, "PLAIN", 50, 16384, 49152),
    (0, 29, 1, "PLAIN", 50, 24576, 57344),
    (0, 45, 1, "PLAIN", 50, 57344, 114688),
    (0, 59, 1, "PLAIN", 50, 131072, 262144),
    (0, 7, 1, "SHORT", 15, 4096, 16384),
    (0, 29, 1, "SHORT", 15, 16384, 32768),
    (0, 59, 1, "SHORT", 15, 45056, 65536),
    (0, 19, 1, "REFIT", 50, 16384, 45056),
    (0, 59, 1, "REFIT", 50, 57344, 262144),
    (1, 24, 1, "PLAIN", 50, 16384, 49152),
    (1, 32, 1, "PLAIN", 50, 24576, 49152),
    (1, 44, 1, "PLAIN", 50, 49152, 114688),
    (1, 64, 1, "PLAIN", 50, 196608, 524288),
    (1, 68, 2, "PLAIN", 50, 49152, 81920),
    (1, 92, 2, "PLAIN", 50, 98304, 393216),
    (1, 128, 2, "PLAIN", 50, 1000000, None),
    (1, 132, 3, "PLAIN", 50, 147456, 393216),
    (1, 256, 4, "PLAIN", 50, 1000000, None),
    (1, 460, 8, "PLAIN", 50, 1000000, None),
    (1, 32, 1, "SHORT", 15, 16384, 45056),
    (1, 68, 2, "SHORT", 15, 16384, 57344),
    (1, 92, 2, "SHORT", 15, 57344, 262144),
    (1, 460, 8, "SHORT", 15, 131072, None),
    (1, 44, 1, "REFIT", 50, 45056, 163840),
    (1, 68, 2, "REFIT", 50, 32768, 65536),
    (1, 460, 8, "REFIT", 50, 131072, None),
    # few trials: the set-up of a pixel counts
    (0, 59, 1, "PLAIN", 0, 256, 1024),
    (0, 59, 1, "PLAIN", 2, 1024, 16384),
    (0, 59, 1, "PLAIN", 5, 16384, 57344),
    (0, 19, 1, "PLAIN", 0, 16, 512),
    (0, 19, 1, "PLAIN", 2, 64, 2048),
    (0, 19, 1, "PLAIN", 3, 128, 2048),
    (1, 32, 1, "PLAIN", 3, 512, 2048),
    (1, 68, 2, "PLAIN", 3, 2048, 32768),
    (1, 64, 1, "PLAIN", 1, 64, 4096),
    (1, 64, 1, "PLAIN", 3, 16384, 57344),
    (1, 460, 8, "PLAIN", 0, 262144, None),
    (1, 460, 8, "PLAIN", 1, 16384, 57344),
    (1, 460, 8, "PLAIN", 2, 16384, 49152),
    (1, 460, 8, "PLAIN", 3, 24576, 49152),
]

# (band, points, chunks, with Jacobian, sizes faster in groups, sizes faster in lanes)
SYNTH = [
    (0, 7, 1, 0, (64, 1024), (4096, 16384, 131072, 1000000)),
    (0, 7, 1, 1, (64, 4096), (16384, 131072, 524288)),
    (0, 29, 1, 0, (64, 30011), (65536, 131072, 1000000)),
    (0, 29, 1, 1, (64, 16384), (45000, 131072, 524288)),
    (0, 45, 1, 1, (64, 65536), (131072,)),
    (0, 59, 1, 0, (64, 65536, 114688), (114689, 131072, 262144)),
    (0, 59, 1, 1, (64, 65536, 262144, 524288), ()),
    (1, 16, 1, 0, (64, 8192), (30011, 131072, 1000000)),
    (1, 16, 1, 1, (64, 8192), (16384, 131072, 1000000)),
    (1, 32, 1, 0, (64, 16384), (45000, 131072, 1000000)),
    (1, 44, 1, 1, (64, 16384), (45000, 131072, 1000000)),
    (1, 64, 1, 0, (64, 30011, 131072, 1000000), ()),
    (1, 64, 1, 1, (64, 30011, 131072, 1000000), ()),
    (1, 68, 2, 0, (64, 30011), (65536, 131072, 1000000)),
    (1, 68, 2, 1, (64, 16384), (30011, 65536, 1000000)),
    (1, 92, 2, 0, (64, 30011, 131072, 1000000), ()),
    (1, 92, 2, 1, (64, 16384, 131072, 1000000), (45000, 65536)),
    (1, 460, 8, 0, (64, 30011, 131072, 1000000), ()),
    (1, 460, 8, 1, (64, 30011, 65536, 262144), ()),
]


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("routes")
    src = ['#include "routes.h"', "#include <cstdio>", "using namespace vfisv;", "int main() {"]
    for band, pts, ch, use, it, _, _ in FITS:
        src.append('  printf("%%lld\\n", (long long)fit_group_max({%d, %d, %d}, FIT_%s, %d));'
                   % (band, pts, ch, use, it))
    src.append('  printf("%lld\\n", (long long)fit_group_max({false, 59, 1}, FIT_SCHEDULED, 50));')
    src.append('  printf("%lld\\n", (long long)fit_group_max({false, 117, 0}, FIT_PLAIN, 50));')
    for band, pts, ch, jac, group, lanes in SYNTH:
        for n in group + lanes:
            src.append('  printf("%%d\\n", (int)synth_by_group({%d, %d, %d}, %d, %d));'
                       % (band, pts, ch, n, jac))
    src.append('  printf("%d\\n", (int)synth_by_group({false, 117, 0}, 1, true));')
    (d / "r.cpp").write_text("\n".join(src + ["}"]))
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "r.cpp"), "-o",
                    str(d / "r")], check=True, capture_output=True)
    out = subprocess.run([str(d / "r")], check=True, capture_output=True, text=True).stdout
    return [int(x) for x in out.split()]


@pytest.mark.parametrize("i", range(len(FITS)), ids=lambda i: "-".join(map(str, FITS[i][:5])))
def test_fits_go_where_they_were_measured_faster(answers, i):
    most, group, lanes = answers[i], FITS[i][5], FITS[i][6]
    assert most >= group
    assert lanes is None or most < lanes


def test_schedules_and_instruments_without_tables_stay_with_the_lanes(answers):
    assert answers[len(FITS):len(FITS) + 2] == [0, 0] and answers[-1] == 0


def test_synthesis_goes_where_it_was_measured_faster(answers):
    got = iter(answers[len(FITS) + 2:])
    for band, pts, ch, jac, group, lanes in SYNTH:
        for n in group + lanes:
            assert next(got) == (n in group), (band, pts, ch, jac, n)
