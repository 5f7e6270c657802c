"""The streams that caches leave to later ones (csrc/stream_sets.hpp), compiled for the host (CPU only)."""
from test_ffn_plan import _run

SETS = r"""
#include "stream_sets.hpp"
#include <atomic>
#include <cstdio>
#include <set>
#include <thread>

using Set = moei::StreamSet<int>;

int main() {
    int bad = 0, made = 0;
    auto expect = [&](bool ok, const char* what) { if (!ok) { std::printf("%s\n", what); ++bad; } };
    auto any = [](const Set&) { return true; };
    auto make = [&](Set* s) { s->prefetch = 3 * made, s->copy = 3 * made + 1, s->side = 3 * made + 2; ++made; return 0; };
    int dropped = 0;
    auto drop = [&](const Set&) { ++dropped; };
    moei::StreamSets<int, 6> sets;
    Set s[9];
    for (auto& t : s) expect(sets.take(0, &t, any, make, drop) == 0, "made");
    expect(made == 12, "four at a time");
    for (int i = 0; i < 9; ++i) expect(s[i].side == 3 * i + 2, "a set of its own for each cache that lives, in the order made");
    // three are idle; given back in another order than made, the first made is handed out first, whole
    expect(sets.keep(s[2]) && sets.keep(s[0]) && sets.keep(s[5]), "kept");
    expect(!sets.keep(s[3]), "no more than six");
    Set t;
    for (int i : {0, 2, 5, 9, 10, 11})
        expect(sets.take(0, &t, any, make, drop) == 0 && t.prefetch == 3 * i && t.copy == 3 * i + 1 && t.side == 3 * i + 2, "the first made");
    expect(made == 12, "nothing made while there are some");
    // devices
    expect(sets.keep(s[0]) && sets.take(1, &t, any, make, drop) == 0 && made == 16 && t.device == 1 && t.side == 38, "none of another device");
    expect(sets.take(0, &t, any, make, drop) == 0 && t.side == s[0].side, "its own device's");
    for (int i : {1, 2, 3, 4, 5, 6}) expect(sets.keep(s[i]), "six of a device beside another's");
    // a set that can no longer be used is forgotten
    expect(sets.take(0, &t, [&](const Set& x) { return x.side != s[1].side && x.side != s[2].side; }, make, drop) == 0 && t.side == s[3].side, "unusable sets");
    for (int i : {4, 5, 6}) expect(sets.take(0, &t, any, make, drop) == 0 && t.side == s[i].side, "the others");
    // a first set that cannot be made is said, a later one is done without
    expect(sets.take(0, &t, any, [](Set*) { return -4; }, drop) == -4 && t.side == 0 && dropped == 0, "a failure");
    int left = 2;
    expect(sets.take(0, &t, any, [&](Set* x) { return left-- > 0 ? make(x) : -4; }, drop) == 0 && t.side == 50 && dropped == 1, "fewer than four");
    expect(sets.take(0, &t, any, make, drop) == 0 && t.side == 53, "the second");
    // threads: no set in two hands
    moei::StreamSets<int, 4> shared;
    std::atomic<int> next{0}, twice{0};
    static std::atomic<int> held[700000];  // (a set that finds no room is made again)
    std::vector<std::thread> threads;
    for (int n = 0; n < 8; ++n)
        threads.emplace_back([&] {
            for (int i = 0; i < 20000; ++i) {
                Set mine;
                shared.take(0, &mine, any, [&](Set* x) { x->side = next++; return 0; }, [](const Set&) {});
                if (held[mine.side]++) ++twice;
                --held[mine.side];
                shared.keep(mine);
            }
        });
    for (auto& th : threads) th.join();
    expect(twice == 0, "one set in two hands");
    return bad != 0;
}
"""


def test_a_cache_gets_the_set_that_was_made_first(tmp_path):
    _run(tmp_path, SETS)
