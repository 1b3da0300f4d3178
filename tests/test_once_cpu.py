"""Work once per device (kernel attributes): on each device, again after a failure, from any thread."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "bdc_once.h"
#include <cstdio>
#include <thread>
#include <vector>
int main() {
    bdc::OncePerDevice once;
    int calls[3] = {};
    auto on = [&](int dev, int result) { return once.run(dev, 0, [&] { ++calls[dev]; return result; }); };
    if (on(0, 7) != 7 || calls[0] != 1) return 1;              // a failure is reported
    if (on(0, 0) != 0 || calls[0] != 2) return 2;              // and not kept
    if (on(0, 7) != 0 || calls[0] != 2) return 3;              // success is
    if (on(1, 0) != 0 || calls[1] != 1) return 4;              // another device has its own
    if (on(1, 7) != 0 || on(0, 7) != 0 || calls[1] != 1) return 5;
    int far = 0;                                               // beyond what is recorded: every time
    for (int k = 0; k < 2; ++k) once.run(64, 0, [&] { ++far; return 0; });
    if (far != 2) return 6;
    bdc::OncePerDevice shared;
    std::vector<std::thread> threads;
    std::atomic<int> bad{0}, done{0};
    for (int k = 0; k < 8; ++k)
        threads.emplace_back([&] {
            for (int i = 0; i < 1000; ++i)
                if (shared.run(i % 64, 0, [&] { ++done; return 0; }) != 0) ++bad;
        });
    for (auto& t : threads) t.join();
    return bad != 0 || done < 64 || done > 8 * 64 ? 8 : 0;
}
"""


def test_once_per_device(tmp_path):
    src = tmp_path / "once.cpp"
    src.write_text(SOURCE)
    exe = str(tmp_path / "once")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_2411_00991_amd", "csrc"),
                           str(src), "-o", exe])
    assert subprocess.run([exe], timeout=60).returncode == 0
