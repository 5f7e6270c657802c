"""The plan of the streaming FFN's workgroups (csrc/ffn_plan.hpp), compiled for the host (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RULE = r"""
#include "ffn_plan.hpp"
#include <cstdio>
#include <thread>
#include <vector>

// the rule, written out: of the counts min .. max the one with the fewest rounds * wavefronts, the largest of these
static int expected(int units, int blocks, int max, int min) {
    int best = max;
    long long best_slots = -1;
    for (int m = max; m >= min; --m) {
        const long long w = (long long)blocks * m, slots = (units + w - 1) / w * w;
        if (best_slots < 0 || slots < best_slots) {
            best_slots = slots;
            best = m;
        }
    }
    return best;
}

int main() {
    int bad = 0;
    for (int units : {1, 30, 512, 1024, 2816, 11264, 28672, 12288, 1000003})
        for (int blocks : {1, 32, 232, 256})
            for (int max : {8, 12, 16})
                for (int min : {1, 4, 8}) {
                    const int got = moei::plan_waves(units, blocks, max, min, 0);
                    if (got != expected(units, blocks, max, min)) {
                        std::printf("%d units, %d workgroups, %d .. %d: %d\n", units, blocks, min, max, got);
                        ++bad;
                    }
                }
    // threads that plan different calls at the same time: each gets its own answer, also one that must not be below its minimum
    std::vector<std::thread> threads;
    std::vector<int> wrong(4, 0);
    for (int t = 0; t < 4; ++t)
        threads.emplace_back([t, &wrong] {
            const int units = t < 2 ? 64 : 1024 + t, min = t == 0 ? 8 : 4;
            const int want = expected(units, 232, 16, min);
            for (int i = 0; i < 2000000; ++i) wrong[t] += moei::plan_waves(units, 232, 16, min, 0) != want;
        });
    for (auto& th : threads) th.join();
    for (int t = 0; t < 4; ++t)
        if (wrong[t]) {
            std::printf("thread %d: %d wrong plans\n", t, wrong[t]);
            ++bad;
        }
    return bad != 0;
}
"""


def _run(tmp_path, main):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(main)
    subprocess.run([cxx, "-O2", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_2401_14361_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout


def test_plan_is_the_rule_in_every_thread(tmp_path):
    _run(tmp_path, RULE)


FORCED = r"""
#include "ffn_plan.hpp"
#include <cstdio>
#include <initializer_list>

int main() {
    int bad = 0;
    for (int max : {8, 12, 16})
        for (int forced = 1; forced <= max; ++forced) {
            if (moei::plan_waves(11264, 232, max, 4, forced) != forced) {
                std::printf("%d of at most %d wavefronts asked for, %d planned\n", forced, max, moei::plan_waves(11264, 232, max, 4, forced));
                ++bad;
            }
            // a launch that also matches takes the count where its workgroups are large enough, else the match is not put there
            const bool takes = moei::forced_takes_match(forced);
            bad += takes != (forced >= 8);
            bad += takes && moei::plan_waves(11264, 232, max, 8, forced) != forced;
        }
    for (int none : {-1, 0}) bad += !moei::forced_takes_match(none) || moei::plan_waves(11264, 232, 16, 8, none) < 8;
    bad += moei::plan_waves(11264, 232, 8, 4, 9) > 8;  // more than the kernel takes: as if nothing was asked for
    return bad != 0;
}
"""


def test_a_forced_count_is_taken(tmp_path):
    _run(tmp_path, FORCED)
