"""A kernel's dynamic LDS limit under two threads and two devices
(csrc/lds_attr.hpp), on the CPU."""
import os
import subprocess

import paper_1501_07350_amd as offt

CSRC = os.path.join(os.path.dirname(os.path.abspath(offt.__file__)), "csrc")

# Two threads launch one kernel for the first time, with 100000 and 150000 bytes.
# The first one's call that sets the limit ends after the other's.
PROGRAM = r"""
#include <cstdio>
#include <thread>
#include "lds_attr.hpp"
using namespace offt;
int main() {
    std::atomic<uint64_t> done{0};
    std::atomic<long> limit{65536};
    std::atomic<int> entered{0}, left{0};
    auto launch = [&](size_t lds, bool slow) {
        return raise_lds_limit(done, 0, lds, 163840, [&](size_t v) {
            ++entered;
            while (entered < 2) std::this_thread::yield();   // both have found the limit too low
            if (slow) while (left < 1) std::this_thread::yield();
            limit = (long)v;
            ++left;
            return 0;
        });
    };
    int ra = -1, rb = -1;
    std::thread a([&] { ra = launch(100000, true); }), b([&] { rb = launch(150000, false); });
    a.join();
    b.join();
    // a later launch sets nothing; another device's first one does; a failure is
    // reported and tried again
    int calls = 0, fail = 1;
    auto count = [&](size_t) { ++calls; return fail; };
    const int r1 = raise_lds_limit(done, 0, 150000, 163840, count), r2 = raise_lds_limit(done, 1, 150000, 163840, count);
    fail = 0;
    const int r3 = raise_lds_limit(done, 1, 150000, 163840, count), r4 = raise_lds_limit(done, 1, 160000, 163840, count);
    const int r5 = raise_lds_limit(done, 2, 65536, 163840, count);
    printf("%d %d %ld %d%d%d%d%d %d\n", ra, rb, limit.load(), r1, r2, r3, r4, r5, calls);
}
"""


def test_two_threads_and_two_devices(tmp_path):
    src, exe = tmp_path / "lds.cpp", str(tmp_path / "lds")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=thread", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["0", "0", "163840", "01000", "2"]
