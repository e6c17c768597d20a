"""The place of a step among the scenes of a process (terrain_gate.h), on the
host alone: never more compute units taken than there are, unless one step by
itself asks for more; steps that fit run together; in order of arrival, so that
a large one is not kept out by a stream of small ones."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = r'''
#include <atomic>
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>
#include "terrain_gate.h"

int main()
{
    using namespace std::chrono_literals;
    trk::CuGate g;
    const int cap = 32, needs[8] = {1, 7, 13, 16, 25, 32, 32, 40};
    std::atomic<int> used{0}, inside{0}, bad{0}, done{0};
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; ++t)
        ts.emplace_back([&, t] {
            for (int k = 0; k < 200; ++k) {
                g.enter(needs[t], cap);
                const int u = used += needs[t], n = ++inside;
                if (u > cap && n > 1) ++bad;
                if (k % 16 == 0) std::this_thread::sleep_for(50us);
                used -= needs[t];
                --inside;
                g.leave(needs[t]);
            }
            ++done;
        });
    for (auto& t : ts) t.join();
    // two that fit are inside at once
    g.enter(16, cap);
    std::atomic<int> second{0}, large{0}, small{0};
    std::thread a([&] { g.enter(16, cap); second = 1; g.leave(16); });
    a.join();
    // a small one that comes after a large one waits behind it
    std::thread b([&] { g.enter(32, cap); large = 1; std::this_thread::sleep_for(20ms); large = 2; g.leave(32); });
    std::this_thread::sleep_for(50ms);
    std::thread c([&] { g.enter(1, cap); small = large == 2 ? 1 : 2; g.leave(1); });
    std::this_thread::sleep_for(50ms);
    const int early = large + small;
    g.leave(16);
    b.join();
    c.join();
    std::printf("%d %d %d %d %d\n", (int)bad, (int)done, (int)second, early, (int)small);
}
'''


def test_gate(tmp_path):
    src, exe = str(tmp_path / "gate.cpp"), str(tmp_path / "gate")
    with open(src, "w") as f:
        f.write(CODE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread", "-I",
                           os.path.join(ROOT, "paper_2011_00459_amd", "csrc"), src, "-o", exe])
    out = subprocess.run([exe], stdout=subprocess.PIPE, timeout=60, check=True).stdout
    assert out.split() == [b"0", b"8", b"1", b"0", b"1"]
