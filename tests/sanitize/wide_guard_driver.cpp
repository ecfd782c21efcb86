// The two-pass kernels' launcher (csrc/snapkv_wide.hip) refuses prompts without their buffers before it asks the device for anything.
#include <cstdio>

#include "../../paper_2404_14469_amd/csrc/snapkv_internal.h"

using namespace snapkv;

int main() {
    char* const somewhere = reinterpret_cast<char*>(0x10000);   // never dereferenced: the launch is refused
    ScoreGeom G = make_geom(140001, 32, 8, 128, 16);
    G.k_rs = 256;
    G.k_hs = G.k_rs * G.L;
    if (!wide_ok(0, 128, G) || wide_part_bytes(G) == 0) return std::printf("not a prompt of the two passes\n"), 1;
    for (int missing = 0; missing < 4; ++missing) {
        WidePrompt P[2];
        for (WidePrompt& p : P) p = WidePrompt{somewhere, somewhere, reinterpret_cast<float*>(somewhere), reinterpret_cast<float2*>(somewhere), &G};
        if (missing == 0) P[1].q = nullptr;
        if (missing == 1) P[1].k = nullptr;
        if (missing == 2) P[1].vote = nullptr;
        if (missing == 3) P[1].part = nullptr;
        const hipError_t e = launch_score_wide(0, 128, 2, P, nullptr);
        if (e != hipErrorInvalidValue) return std::printf("buffer %d missing: %d\n", missing, (int)e), 1;
    }
    std::printf("all cases passed\n");
    return 0;
}
