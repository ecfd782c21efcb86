// How the two-pass kernels' launches are shared out (csrc/snapkv_shares.h): every round has one workgroup, and a launch of a few
// layers, of whose slices a workgroup has two or three, leaves no part of the chip idle for long.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <utility>
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
    // the largest sum of the shares that a compute unit has, and how many have it
    std::pair<unsigned, unsigned> meeting(bool reversed) const {
        std::pair<unsigned, unsigned> m{0, 0};
        for (unsigned w = 0; w < grid / 2; ++w) {
            const unsigned sum = slices_of(share_of(w, grid, reversed)) + slices_of(share_of(w + grid / 2, grid, reversed));
            if (sum > m.first) m = {sum, 0};
            m.second += sum == m.first;
        }
        return m;
    }
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
                    if (l.grid < 512) continue;
                    // the statistics' pass: every share has one workgroup, and no order is worse than the other
                    const bool rev = reverse_shares(l.total, l.grid, rps);
                    std::vector<int> had(l.grid, 0);
                    for (unsigned w = 0; w < l.grid; ++w) ++had[share_of(w, l.grid, rev)];
                    check(*std::min_element(had.begin(), had.end()) == 1, "a share each", layers, (int)rounds);
                    if (l.total / rps / l.grid < 32) check(l.meeting(rev) <= l.meeting(!rev), "the better order", layers, (int)rounds);
                }
    // launches in which every second compute unit had two long shares, or one in four: now none has, or one in eight
    struct { int layers, units; unsigned rounds, rps, sum, at_most; } const few[] = {
        {2, 16, 97, 4, 16, 32}, {3, 16, 97, 4, 24, 0}, {4, 16, 83, 3, 24, 0}, {2, 12, 128, 4, 16, 0}, {8, 12, 469, 12, 192, 0}, {2, 8, 129, 3, 12, 5}};
    for (const auto& f : few) {
        const Launch l(f.layers, f.units, f.rounds, f.rps);
        const auto m = l.meeting(reverse_shares(l.total, l.grid, f.rps));
        check(m.first < f.sum || (m.first == f.sum && m.second <= f.at_most), "long shares meet", f.layers, (int)f.rounds);
    }
    std::printf("all cases passed\n");
    return 0;
}
