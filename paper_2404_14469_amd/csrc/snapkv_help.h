// How workgroups of wide_once (snapkv_wide.hip) that miss the words of their unit's other slices help themselves (host and device, nothing
// of the GPU's).
//
// Only the first look at the words is a patient one: a workgroup that has waited in vain once waits no more, but takes the statistics of
// slice after slice until no word is missing.  Each takes the missing slice of the smallest key, whose number differs least from the
// workgroup's own in the high bits, so that r workgroups which miss the same m slices mostly take different ones: they are done
// after one patience and about m / r slices' times, 2 m / r at most or so, and not after m of each.
#pragma once

namespace snapkv {

constexpr int kNoneMissing = 0x7fffffff;

constexpr unsigned patience(int turn, unsigned limit) { return turn == 0 ? limit : 0u; }
constexpr int help_key(int slice, int own) { return slice ^ own; }
constexpr int help_slice(int key, int own) { return key ^ own; }

}  // namespace snapkv
