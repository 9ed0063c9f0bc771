"""Rules of the estimate's launches (csrc/rr_estimate_rules.hpp), on the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05853_amd", "csrc")

PROGRAM = r'''
#include <cstdio>
#include <cstdlib>
#include "rr_estimate_rules.hpp"
int main(int argc, char** argv) {
    int v[7];
    for (int i = 0; i < 7 && i + 1 < argc; ++i) v[i] = atoi(argv[i + 1]);
    printf("%d\n", rr::eight_waves_pay(v[0], v[1], v[2], v[3], v[4], v[5], (unsigned)v[6]));
}
'''


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("rules")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)
    return lambda *v: bool(int(subprocess.run([str(d / "rule"), *map(str, v)], check=True, capture_output=True, text=True).stdout))


# workgroups, batch, Nb, R, heads of a workgroup, d, KB of LDS: shapes that were faster on eight waves, and slower
@pytest.mark.parametrize("shape,eight", [((256, 1, 64, 8, 2, 128, 18), True), ((128, 4, 256, 32, 1, 136, 84), True), ((282, 1, 94, 8, 2, 96, 20), True),
                                         ((500, 1, 125, 8, 2, 64, 22), True), ((512, 1, 64, 8, 2, 64, 14), True), ((480, 1, 160, 16, 1, 64, 26), True),
                                         ((312, 1, 78, 16, 1, 96, 17), True), ((336, 2, 84, 8, 1, 24, 7), True), ((500, 1, 250, 32, 1, 128, 82), True),
                                         ((500, 2, 250, 8, 2, 128, 43), False), ((500, 2, 125, 16, 1, 64, 21), False), ((381, 1, 127, 16, 1, 136, 26), False),
                                         ((508, 1, 127, 16, 1, 80, 22), False), ((416, 2, 208, 4, 1, 80, 9), False), ((494, 2, 247, 32, 1, 128, 80), False),
                                         ((436, 2, 218, 32, 1, 136, 75), False), ((513, 1, 64, 8, 2, 64, 14), False), ((200, 1, 257, 4, 1, 64, 9), False)])
def test_eight_waves_where_they_are_faster(rule, shape, eight):
    assert rule(*shape[:6], shape[6] << 10) == eight
