// How the launches of the two-pass scoring kernels (snapkv_wide.hip) hand the rounds of all their units out to a persistent grid (host and
// device, nothing of the GPU's).
#pragma once

namespace snapkv {

// Equal shares of the launch's rounds, one more for the first `more` workgroups: where that of workgroup wg begins.
constexpr unsigned begin_rounds(unsigned share, unsigned more, unsigned wg) { return share * wg + (wg < more ? wg : more); }

// The first round at or after `in` (counted from an entry's first one) that a slice of rps rounds begins with.
constexpr unsigned whole_slices(unsigned in, unsigned rps) { return (in + rps - 1) / rps * rps; }

}  // namespace snapkv
