"""The guard that raises a kernel's LDS limit before its first launch (csrc/gvq_once.h), checked on the CPU: the header is plain
C++."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1811_03617_amd", "csrc")


def test_no_thread_goes_on_before_the_step_is_done(tmp_path):
    """Eight threads at once, a step that takes a while and fails the first time: whoever is told 0 finds it done, on that device,
    and it is done once."""
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(r"""
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>
#include "gvq_once.h"
static gvq_once_per_device once;
int main()
{
    std::atomic<int> ready[3] = {}, steps[3] = {}, failed{0}, wrong{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 24; ++t)
        threads.emplace_back([&, t]() {
            const int device = t % 3;
            const int rc = once.call(device, [&]() -> int {
                const int n = steps[device]++;
                std::this_thread::sleep_for(std::chrono::milliseconds(30));
                if (n == 0) return -4;
                ready[device] = 1;
                return 0;
            });
            if (rc != 0) ++failed;
            else if (!ready[device]) ++wrong;
        });
    for (std::thread& t : threads) t.join();
    for (int d = 0; d < 3; ++d)
        if (steps[d] != 2 || once.call(d, []() { return -1; }) != 0) ++wrong;
    printf("%d wrong, %d failed\n", (int)wrong, (int)failed);
    return wrong || failed != 3;
}
""")
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
