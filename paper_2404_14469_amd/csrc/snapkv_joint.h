// Where a batch of prompts is cut into joint launches of the single-read scoring kernel (host only, nothing of the GPU's).
//
// A launch lasts as long as its prompt with the most iterations, so one more prompt can cost more than it brings: eight prompts of
// 8500 keys, 32/8 heads fill a launch in which one of them has a single group, 16 iterations; the first by itself takes 2, and
// the seven others, with two groups each, 8.
//
// All prompts of a batch have the same units (parts of KV heads) and the same numbers of groups to choose from, and a launch
// hands its spare workgroups, step by step, to a prompt with the most iterations.  That ends where the next step of such a
// prompt does not fit, i.e. at the fewest iterations that all prompts can have together: those of the largest number of groups
// that fits the chip for every one of them.  So a launch is priced by a division, without handing anything out: the cuts of 32
// prompts take 2 us at most.  With the steps of every run carried out, 32 prompts of 500-2000 keys, 32/8 heads took 252 us a call, all of it host
// time; now 156, as where nothing is priced (32 of 1-4K keys 224 / 154, 32 of 600-700, W = 32 269 / 154).
#pragma once

#include <climits>

namespace snapkv {

constexpr int kMaxBatch = 32;         // prompts of a batch
constexpr int kMaxJointPrompts = 8;   // and of a joint launch
constexpr int kJointStart = 7;        // halves of an iteration that a launch's first keys and its drain take

struct JointUnits {
    int units;   // of a prompt: its KV heads times split
    int split;   // parts of a KV head, which run side by side or one after another
};

// Iterations of a launch whose prompts take sum workgroups (at most slots) with one group each.  The groups of a prompt are a
// divisor of split, or a multiple of it up to the units.
inline int joint_iterations(const JointUnits& u, int sum, int slots) {
    int n = slots / sum;
    if (n >= u.split) {
        n = (n < u.units ? n : u.units) / u.split * u.split;
    } else {
        while (u.split % n != 0) --n;
    }
    return (u.units + n - 1) / n;
}

// Gg: workgroups of a group of each prompt, in the order in which launches take them (longest prompt first), none above slots.
// The cuts into runs of neighbours that cost least are compared with filling launch after launch, each with whatever of the
// rest still fits it.  Returns the number of launches and their prompts in cut[], or 0: fill them one by one.
inline int joint_cuts(const JointUnits& u, const int* Gg, int count, int slots, int* cut) {
    if (count < 1 || count > kMaxBatch) return 0;
    int filled = 0;
    bool done[kMaxBatch] = {};
    for (int left = count; left > 0;) {
        int taken = 0, sum = 0;
        for (int i = 0; i < count && taken < kMaxJointPrompts; ++i)
            if (!done[i] && sum + Gg[i] <= slots) {
                sum += Gg[i];
                done[i] = true;
                ++taken;
            }
        if (taken == 0) return 0;
        left -= taken;
        filled += 2 * joint_iterations(u, sum, slots) + kJointStart;
    }
    const int least = (count + kMaxJointPrompts - 1) / kMaxJointPrompts * (2 + kJointStart);   // no cut costs less
    if (50 * least > 49 * filled) return 0;
    int cost[kMaxBatch + 1], from[kMaxBatch + 1];   // of the first i prompts; where their last launch begins
    cost[0] = 0;
    for (int i = 1; i <= count; ++i) cost[i] = INT_MAX;
    for (int i = 0; i < count; ++i) {
        int sum = 0;
        for (int j = i; j < count && j - i < kMaxJointPrompts; ++j) {
            sum += Gg[j];
            if (sum > slots) break;
            const int c = cost[i] + 2 * joint_iterations(u, sum, slots) + kJointStart;
            if (c < cost[j + 1]) {
                cost[j + 1] = c;
                from[j + 1] = i;
            }
        }
    }
    if (50 * cost[count] > 49 * filled) return 0;   // (no less than 2 %)
    int launches = 0;
    for (int i = count; i > 0; i = from[i]) ++launches;
    for (int i = count, l = launches; i > 0; i = from[i]) cut[--l] = i - from[i];
    return launches;
}

}  // namespace snapkv
