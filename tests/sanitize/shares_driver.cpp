// How the two-pass kernels' launches are shared out (csrc/snapkv_shares.h): every round has one workgroup, and a launch of a few
// layers, of whose slices a workgroup has two or three, leaves no part of the chip idle for long.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2404_14469_amd/csrc/snapkv_shares.h"

using namespace snapkv;

static void check(bool ok, const char* what, int a, int b) {
    if (ok) return;
    std::printf("%s: %d %d\n", what, a, b);
    std::exit(1);
}

struct Launch {                          // layers of `rounds` rounds a unit, in slices of rps
    unsigned rps, total, grid, share, more;
    Launch(int layers, int units, unsigned rounds, unsigned rps_) : rps(rps_) {
        const unsigned slices = (rounds + rps - 1) / rps * units * layers;
        total = slices * rps;
        grid = std::min(slices, 512u);
        share = total / grid;
        more = total % grid;
    }
    unsigned rounds_of(unsigned wg) const { return begin_rounds(share, more, wg + 1) - begin_rounds(share, more, wg); }
    unsigned slices_of(unsigned wg) const { return begin_slices(share, more, wg + 1) - begin_slices(share, more, wg); }
    unsigned begin_slices(unsigned s, unsigned m, unsigned wg) const { return std::min(total, whole_slices(begin_rounds(s, m, wg), rps)); }
};

int main() {
    for (int layers : {1, 2, 3, 4, 5, 6, 8, 32})
        for (int units : {1, 8, 12, 16, 33})
            for (unsigned rounds : {8u, 47u, 67u, 97u, 133u, 157u, 188u, 1024u})
                for (unsigned rps : {1u, 2u, 4u, 5u, 32u}) {
                    const Launch l(layers, units, rounds, rps);
                    unsigned all = 0, whole = 0, most = 0;
                    for (unsigned w = 0; w < l.grid; ++w) {
                        check(l.slices_of(w) % rps == 0 && l.slices_of(w) <= (l.total + l.grid - 1) / l.grid + rps, "whole slices", layers, (int)rounds);
                        all += l.rounds_of(w);
                        whole += l.slices_of(w);
                        most = std::max(most, l.rounds_of(w));
                    }
                    check(all == l.total && whole == l.total, "all rounds", layers, (int)rounds);
                    // the votes' pass: no workgroup has more than an equal share (of whole slices it may have up to rps - 1 more)
                    check(most == (l.total + l.grid - 1) / l.grid, "equal shares", layers, (int)rounds);
                }
    std::printf("all cases passed\n");
    return 0;
}
