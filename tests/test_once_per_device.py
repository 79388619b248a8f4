"""What a kernel needs before its first launch on a device: done on every device, from any thread, again after a failure."""
import os
import subprocess

from paper_2309_03824_amd import build

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "once_per_device.hpp"
int main()
{
    static lrd::OncePerDevice once;
    std::atomic<int> calls[80] = {};
    auto succeed = [&](int d) { return once(d, [&] { ++calls[d]; return 0; }); };
    if (once(3, [] { return 7; }) != 7) return puts("an error is handed on"), 1;
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&] { for (int i = 0; i < 10000; ++i) succeed(i % 80); });
    for (auto& t : threads) t.join();
    for (int d = 0; d < 64; ++d)
        if (calls[d] < 1 || calls[d] > 8) return printf("device %d: %d times\n", d, calls[d].load()), 1;
    for (int d = 64; d < 80; ++d)
        if (calls[d] != 1000) return printf("device %d: %d times\n", d, calls[d].load()), 1;
}
"""


def test_every_device_from_any_thread(tmp_path):
    (tmp_path / "once.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-I", os.path.abspath(build.CSRC), str(tmp_path / "once.cpp"), "-o",
                    str(tmp_path / "once")], check=True)
    res = subprocess.run([str(tmp_path / "once")], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr


def test_no_launch_keeps_a_flag_for_all_devices():
    for name in os.listdir(build.CSRC):
        if name.endswith(".hip"):
            with open(os.path.join(build.CSRC, name)) as f:
                assert "static bool" not in f.read(), name
