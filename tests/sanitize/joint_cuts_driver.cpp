// The cuts of batches into joint launches (csrc/snapkv_joint.h) against a price that hands the spare workgroups out one step
// at a time, as a launch does: the same cuts for drawn batches, runs within a launch's limits, and no more time than a
// plan may take in front of a launch.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../../paper_2404_14469_amd/csrc/snapkv_joint.h"

using namespace snapkv;

static void check(bool ok, const char* what, int trial) {
    if (ok) return;
    std::printf("batch %d: %s\n", trial, what);
    std::exit(1);
}

// Iterations of the prompt that has most, once nobody's next step fits.
static int handed_out(const JointUnits& u, const std::vector<int>& Gg, int slots) {
    std::vector<int> n(Gg.size(), 1);
    int total = 0;
    for (int x : Gg) total += x;
    auto next = [&](int k) {
        if (k >= u.split) return k + u.split;
        for (++k; u.split % k; ++k) {}
        return k;
    };
    auto iterations = [&](int k) { return (u.units + k - 1) / k; };
    for (;;) {
        int best = -1;
        for (size_t t = 0; t < Gg.size(); ++t) {
            const int nx = next(n[t]);
            if (nx > u.units || total + (nx - n[t]) * Gg[t] > slots) continue;
            if (best < 0 || iterations(n[t]) > iterations(n[best])) best = (int)t;
        }
        if (best < 0 || iterations(n[best]) <= 1) break;
        total += (next(n[best]) - n[best]) * Gg[best];
        n[best] = next(n[best]);
    }
    int most = 0;
    for (int k : n) most = std::max(most, iterations(k));
    return most;
}

static int reference(const JointUnits& u, const std::vector<int>& Gg, int slots, int* cut) {
    const int count = (int)Gg.size();
    auto price = [&](const std::vector<int>& run) { return 2 * handed_out(u, run, slots) + kJointStart; };
    int filled = 0;
    for (std::vector<int> rest = Gg; !rest.empty();) {
        std::vector<int> taken, left;
        int sum = 0;
        for (int x : rest) {
            if ((int)taken.size() < kMaxJointPrompts && sum + x <= slots) {
                taken.push_back(x);
                sum += x;
            } else {
                left.push_back(x);
            }
        }
        filled += price(taken);
        rest = left;
    }
    std::vector<int> cost(count + 1, INT_MAX), from(count + 1, 0);
    cost[0] = 0;
    for (int i = 0; i < count; ++i)
        for (int j = i, sum = 0; j < count && j - i < kMaxJointPrompts && (sum += Gg[j]) <= slots; ++j) {
            const int c = cost[i] + price(std::vector<int>(Gg.begin() + i, Gg.begin() + j + 1));
            if (c < cost[j + 1]) cost[j + 1] = c, from[j + 1] = i;
        }
    if (50 * cost[count] > 49 * filled) return 0;
    std::vector<int> runs;
    for (int i = count; i > 0; i = from[i]) runs.push_back(i - from[i]);
    std::copy(runs.rbegin(), runs.rend(), cut);
    return (int)runs.size();
}

int main() {
    std::mt19937 rng(17);
    auto between = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
    int cut_batches = 0;
    for (int trial = 0; trial < 4000; ++trial) {
        const int splits[] = {1, 2, 4, 8, 3, 6};
        JointUnits u;
        u.split = splits[between(0, 5)];
        u.units = u.split * between(1, 32);
        const int slots = between(0, 3) ? 256 : between(8, 512), count = between(1, kMaxBatch);
        const int lo = between(1, slots / 2), hi = between(lo, between(0, 1) ? slots : std::min(slots, lo + 8));
        std::vector<int> Gg(count);
        for (int& x : Gg) x = between(lo, hi);
        std::sort(Gg.rbegin(), Gg.rend());
        int cut[kMaxBatch], want[kMaxBatch];
        const int launches = joint_cuts(u, Gg.data(), count, slots, cut);
        check(launches == reference(u, Gg, slots, want), "another number of launches", trial);
        int at = 0;
        for (int l = 0; l < launches; ++l) {
            check(cut[l] == want[l], "another cut", trial);
            check(cut[l] >= 1 && cut[l] <= kMaxJointPrompts, "more prompts than a launch takes", trial);
            int sum = 0;
            for (int i = 0; i < cut[l]; ++i) sum += Gg[at + i];
            check(sum <= slots, "more workgroups than the chip holds", trial);
            at += cut[l];
        }
        check(launches == 0 || at == count, "prompts left over", trial);
        cut_batches += launches > 0;
    }
    check(cut_batches > 100, "hardly a batch was cut", -1);

    // eight prompts of 8500 keys, 32/8 heads, W = 16: the longest by itself, then seven
    const int eight[8] = {17, 17, 17, 17, 17, 17, 17, 17};
    int cut[kMaxBatch];
    check(joint_cuts(JointUnits{16, 2}, eight, 8, 256, cut) == 2 && cut[0] == 1 && cut[1] == 7, "eight equal prompts", -1);

    const int split_units[][2] = {{32, 1}, {16, 2}, {64, 2}};
    for (const auto& x : split_units)
        for (int keys : {1, 4}) {
            std::vector<int> Gg(kMaxBatch, keys);
            const auto begin = std::chrono::steady_clock::now();
            int sink = 0;
            for (int i = 0; i < 2000; ++i) {
                Gg[kMaxBatch - 1] = 1 + i % keys;
                sink += joint_cuts(JointUnits{x[0], x[1]}, Gg.data(), kMaxBatch, 256, cut);
            }
            const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - begin).count() / 2000;
            std::printf("32 prompts of %d workgroups, %d units: %.2f us (%d)\n", keys, x[0], us, sink);
            check(us < 20, "the plan takes too long", -1);
        }
    std::printf("all cases passed\n");
    return 0;
}
