// How ffn_fused_kernel's workgroups are shaped.  Host code on plain numbers: it keeps nothing between calls, so
// threads that drive caches of their own do not meet here.
#pragma once

namespace moei {

constexpr int kMatchWaves = 8;  // a workgroup that matches and scores beside the experts has at least these many wavefronts

// Whether steps may match beside the experts where MOEI_FFN_WAVES asks for `forced` wavefronts (0: for none).
inline bool forced_takes_match(int forced) { return forced < 1 || forced >= kMatchWaves; }

// Wavefronts per workgroup: `forced`, or else the count in [min_waves, max_waves] that wastes the fewest unit slots when
// n_units are dealt out to blocks * waves wavefronts (ties go to more wavefronts).  A handful of divisions (0.1 us), made anew at
// every call: a plan kept for the next one would be shared by all threads, and one thread's could reach another's launch.
inline int plan_waves(int n_units, int blocks, int max_waves, int min_waves, int forced) {
    if (forced >= 1 && forced <= max_waves) return forced;
    int best = max_waves;
    long long best_slots = -1;
    for (int m = max_waves; m >= min_waves; --m) {
        const unsigned w = (unsigned)(blocks * m);
        const long long slots = (long long)(((unsigned)n_units + w - 1) / w) * w;
        if (best_slots < 0 || slots < best_slots) {
            best_slots = slots;
            best = m;
        }
    }
    return best;
}

}  // namespace moei
