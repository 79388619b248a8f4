"""The ranges of columns of a wide product against trying every length, and that finding them does not grow with the width."""
import os
import subprocess

import pytest

from paper_2309_03824_amd import build

PROGRAM = r"""
#include <chrono>
#include <cstdio>
#include "wide_plan.hpp"
static int every_length(int64_t rows, int all, int64_t slots)
{
    int best = all;
    double least = 1e30;
    for (int n = 1; n <= all; ++n) {
        const int64_t workgroups = rows * ((all + n - 1) / n);
        const double cost = (double)((workgroups + slots - 1) / slots) * (n + 1.5);
        if (cost < least) { least = cost; best = n; }
    }
    return best;
}
template <class F>
static double microseconds(F f)
{
    int sum = 0;
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 2000; ++i) sum += f(1 + i % 8, 2004, 512);
    const auto t1 = std::chrono::steady_clock::now();
    volatile int keep = sum;
    (void)keep;
    return std::chrono::duration<double, std::micro>(t1 - t0).count() / 2000;
}
int main()
{
    long compared = 0;
    for (int64_t slots : {256, 512})
        for (int all = 24; all <= 2100; all += all < 130 ? 1 : 37)
            for (int64_t rows = 1; rows < 3000; rows += rows < 40 ? 1 : rows / 7) {
                ++compared;
                if (lrd::wide_chunks(rows, all, slots) != every_length(rows, all, slots)) return printf("rows %ld, %d chunks\n", (long)rows, all), 1;
            }
    printf("%ld %.3f %.3f\n", compared, microseconds(every_length), microseconds(lrd::wide_chunks));
}
"""


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    at = tmp_path_factory.mktemp("plan")
    (at / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.abspath(build.CSRC), str(at / "plan.cpp"), "-o", str(at / "plan")], check=True)
    return subprocess.run([str(at / "plan")], check=True, capture_output=True, text=True).stdout.split()


def test_the_same_ranges_as_trying_every_length(output):
    assert int(output[0]) > 10000


def test_finding_them_does_not_grow_with_the_width(output):
    every, plan = map(float, output[1:])
    assert plan * 10 < every
