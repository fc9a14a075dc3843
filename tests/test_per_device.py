"""The once-per-device set-up of the kernel launchers (csrc/per_device.h), in a small host program."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "per_device.h"

static int fail(const char* what) { std::printf("%s\n", what); return 1; }

int main() {
    cf::PerDevice once;
    int calls[65] = {};
    const int devices[] = {0, 0, 7, 0, 7, 63, 63, 64, 64, -1, -1};
    int outside = 0;
    for (int d : devices) once.run(d, [&] { if (d < 0) ++outside; else ++calls[d]; });
    if (calls[0] != 1 || calls[7] != 1 || calls[63] != 1) return fail("a device is set up once");
    if (calls[64] != 2 || outside != 2) return fail("a device without a place of its own is set up every time");

    // no thread goes on before a set-up of its device has ended
    for (int round = 0; round < 200; ++round) {
        cf::PerDevice race;
        std::atomic<int> ended[2] = {{0}, {0}}, early{0};
        std::vector<std::thread> threads;
        for (int t = 0; t < 8; ++t)
            threads.emplace_back([&, d = t & 1] {
                race.run(d, [&] { std::this_thread::yield(); ++ended[d]; });
                if (ended[d] == 0) ++early;
            });
        for (std::thread& t : threads) t.join();
        if (early != 0) return fail("a thread went on before the set-up had ended");
        race.run(0, [&] { early = 1; });
        if (early != 0) return fail("the set-up is not remembered");
    }
    return 0;
}
"""


def test_set_up_runs_once_per_device_and_before_any_thread_goes_on(tmp_path):
    src, exe = tmp_path / "p.cpp", tmp_path / "p"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I", os.path.join(ROOT, "paper_2604_25080_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
