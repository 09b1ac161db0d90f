"""The counts of resident workgroups that set the grids (cs_resident.h): one
entry per device, shared by contexts on several threads.  The header compiled
for the host, with the thread sanitizer where it runs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include "cs_resident.h"
#include <thread>
#include <vector>
#include <cstdio>
int main() {
    static cs::ResidentCache cache;
    std::atomic<int> wrong{0}, looked{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&, t] {
            for (int i = 0; i < 2000; ++i) {
                // devices of different size, two past the table, one that does not answer at first
                const int dev = (t + i) % 66;
                const bool silent = dev == 5 && i < 1000;
                const cs::Resident r = cache.get(dev, [&]() -> cs::Resident {
                    ++looked;
                    return silent ? cs::Resident{0, 256} : cs::Resident{1 + dev, 256 + dev};
                });
                if (!(r.per_cu == 1 + dev && r.cus == 256 + dev) && !(dev == 5 && r.per_cu == 0 && r.cus == 0)) ++wrong;
            }
        });
    for (auto& t : threads) t.join();
    const cs::Resident r = cache.get(5, [] { return cs::Resident{6, 261}; });
    if (r.per_cu != 6 || r.cus != 261) ++wrong;
    // kept: at most one look-up per thread for the 63 devices that answer
    int before = looked;
    for (int dev = 0; dev < 64; ++dev) cache.get(dev, [&] { ++looked; return cs::Resident{1, 1}; });
    if (looked != before) ++wrong;
    std::printf("%d\n", (int)wrong);
    return wrong != 0;
}
"""


@pytest.mark.parametrize("sanitize", [False, True])
def test_counts_are_per_device_and_thread_safe(tmp_path, sanitize):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    flags = ["-fsanitize=thread"] if sanitize else []
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", *flags,
                    "-I" + os.path.join(ROOT, "paper_2206_02937_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    if sanitize and "unexpected memory mapping" in r.stderr:
        pytest.skip("the thread sanitizer does not run on this kernel")
    assert r.returncode == 0, r.stdout + r.stderr
