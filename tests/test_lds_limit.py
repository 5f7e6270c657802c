"""The table of the kernels' dynamic-LDS limits (csrc/lds_limit.hpp), compiled for the host (CPU only)."""
from test_ffn_plan import _run

LIMITS = r"""
#include "lds_limit.hpp"
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>

constexpr int kKernels = 40, kRounds = 400;

int main() {
    std::atomic<int> bad{0};
    for (int round = 0; round < kRounds; ++round) {
        moei::LdsLimits<kKernels> limits;
        std::vector<std::atomic<size_t>> limit(kKernels);
        for (auto& l : limit) l = 65536;
        std::atomic<bool> go{false};
        std::vector<std::thread> threads;
        for (int t = 0; t < 4; ++t)
            threads.emplace_back([&, t] {
                while (!go) std::this_thread::yield();
                for (int i = 0; i < kKernels; ++i) {
                    const int k = (i + t % 2) % kKernels;
                    const size_t bytes = 65536 + 1024 * (size_t)(1 + (k * 7 + t * 3) % 5);
                    if (limits.at_least(&limit[k], bytes, [&] { limit[k] = bytes; return 0; }) != 0) ++bad;
                    if (limit[k] < bytes) ++bad;  // the launch that follows needs what it asked for
                }
            });
        go = true;
        for (auto& th : threads) th.join();
    }
    if (bad) std::printf("%d launches above their kernel's limit\n", bad.load());
    // a limit that could not be raised is not taken for raised; a known one is not raised again
    moei::LdsLimits<1> one;
    int calls = 0, key = 0, other = 0;
    auto raise = [&](int rc) { return [&calls, rc] { ++calls; return rc; }; };
    bad += one.at_least(&key, 70000, raise(-4)) != -4;
    bad += one.at_least(&key, 70000, raise(0)) != 0 || calls != 2;
    bad += one.at_least(&key, 66000, raise(0)) != 0 || calls != 2;
    bad += one.at_least(&key, 70001, raise(0)) != 0 || calls != 3;
    // a kernel that the table has no room for is raised at every call
    for (int i = 0; i < 2; ++i) bad += one.at_least(&other, 70000, raise(0)) != 0 || calls != 4 + i;
    return bad != 0;
}
"""


def test_a_launch_finds_the_limit_it_asked_for(tmp_path):
    _run(tmp_path, LIMITS)
