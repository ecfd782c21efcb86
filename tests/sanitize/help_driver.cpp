// Workgroups of the two-pass kernels' one launch that miss others' words (csrc/snapkv_help.h): some of a unit's workgroups have no place, the
// rest take turns together.  How long until none of them misses anything: one patience and few turns, whoever has a place.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../../paper_2404_14469_amd/csrc/snapkv_help.h"

using namespace snapkv;

static void check(bool ok, const char* what, int slices, int present) {
    if (ok) return;
    std::printf("%s: %d of %d\n", what, present, slices);
    std::exit(1);
}

int main() {
    std::mt19937 rng(5);
    constexpr unsigned kLimit = 512;
    for (int slices : {2, 3, 15, 37, 64, 256})
        for (int trial = 0; trial < 200; ++trial) {
            const int present = 1 + (int)(rng() % (unsigned)slices);
            std::vector<int> place(slices);
            for (int i = 0; i < slices; ++i) place[i] = i;
            if (trial % 2) std::shuffle(place.begin(), place.end(), rng);   // (else the first ones, as they are handed out in order)
            place.resize(present);
            std::vector<bool> there(slices, false);
            for (int p : place) there[p] = true;
            const int missing = slices - present;
            unsigned polls = 0;
            int turns = 0;
            for (;; ++turns) {
                std::vector<int> takes;
                for (int p : place) {
                    int key = kNoneMissing;
                    for (int s = 0; s < slices; ++s)
                        if (!there[s]) key = std::min(key, help_key(s, p));
                    if (key != kNoneMissing) takes.push_back(help_slice(key, p));
                }
                if (takes.empty()) break;
                polls += patience(turns, kLimit);
                for (int s : takes) {
                    check(s >= 0 && s < slices && !there[s], "a missing slice", slices, present);
                }
                for (int s : takes) there[s] = true;
            }
            check(polls <= kLimit, "patience", slices, present);
            check(turns <= 2 * ((missing + present - 1) / present) + 1, "turns", slices, present);
        }
    std::printf("all cases passed\n");
    return 0;
}
