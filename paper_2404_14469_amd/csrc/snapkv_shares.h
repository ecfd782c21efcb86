// How the launches of the two-pass scoring kernels (snapkv_wide.hip) hand the rounds of all their units out to a persistent grid (host and
// device, nothing of the GPU's).
#pragma once

namespace snapkv {

// Equal shares of the launch's rounds, one more for the first `more` workgroups: where that of workgroup wg begins.
constexpr unsigned begin_rounds(unsigned share, unsigned more, unsigned wg) { return share * wg + (wg < more ? wg : more); }

// The first round at or after `in` (counted from an entry's first one) that a slice of rps rounds begins with.
constexpr unsigned whole_slices(unsigned in, unsigned rps) { return (in + rps - 1) / rps * rps; }

// Which share workgroup wg has.  Of the shares of whole slices some are a slice longer than others, and workgroup wg has its compute unit together
// with wg + grid / 2 (as the chip hands them out; only the time depends on it): where that lets many long shares meet, the
// second half of the grid has its shares in reverse order.  Microseconds per call, in order / so, layers of 32/8 heads: W = 64, 2 of 12300 keys
// 74.2 / 73.7, 3 of 12300 96.6 / 93.0, 4 of 10500 100.7 / 98.4;  W = 32: 3 of 20000 87.0 / 84.9, 4 of 28000 136.5 / 133.5;  12 KV heads, 2 of 16384
// 82.5 / 78.1.  Longer shares for the first workgroups, the same sums, are slower where they part slices of the same keys that
// met in one L2 (4 layers of 15000, W = 64: 112 / 120).
constexpr unsigned share_of(unsigned wg, unsigned grid, bool reversed) { return reversed && wg >= grid / 2 ? grid / 2 + (grid - 1 - wg) : wg; }

// Whether it does: which order has the smaller largest sum of two such shares, or fewer of that size.  (Many slices a share, or a grid of more workgroups
// than any chip has places for: it hardly matters, or is not looked at.)  A share's end is the one before moved on by whole slices, not a
// division: 1.7 us of host time for 512 workgroups, with divisions 3.7.
inline bool reverse_shares(unsigned rounds, unsigned grid, unsigned rps) {
    constexpr unsigned kMost = 1024;
    if (grid < 2 || grid > kMost || rounds / rps / grid >= 32) return false;
    const unsigned share = rounds / grid, more = rounds % grid, half = grid / 2, whole = share / rps * rps;
    unsigned length[kMost], begin = 0, from = 0;
    for (unsigned wg = 0; wg < grid; ++wg) {
        begin += share + (wg < more);
        unsigned to = from + whole;      // (at most whole_slices(begin, rps))
        while (to < begin) to += rps;
        length[wg] = to - from;
        from = to;
    }
    unsigned most[2] = {0, 0}, times[2] = {0, 0};
    for (unsigned wg = 0; wg < half; ++wg)
        for (int r = 0; r < 2; ++r) {
            const unsigned sum = length[wg] + length[share_of(wg + half, grid, r == 1)];
            if (sum > most[r]) most[r] = sum, times[r] = 0;
            times[r] += sum == most[r];
        }
    return most[1] < most[0] || (most[1] == most[0] && times[1] < times[0]);
}

}  // namespace snapkv
