// Hand-off words of the scoring kernels that wait for one another (snapkv_fused.hip, wide_once in snapkv_wide.hip): a row's (maximum, sum of
// exponentials) as one aligned 64-bit word, moved with relaxed device-scope atomics.  A word that has not been written holds a
// pattern that no pair can have, so it proves its own freshness and no order between addresses is relied on.
#ifndef SNAPKV_HANDOFF_H_
#define SNAPKV_HANDOFF_H_

#include <hip/hip_runtime.h>

namespace snapkv {

constexpr unsigned long long kInvalidPair = ~0ull;   // a sum-exp is never NaN: no real pair looks like this
constexpr int kSlicesPerBlock = 32;                  // slices merged by one half-wave in step L1
constexpr unsigned kSpinLimit = 1u << 15;            // polls before a hand-off wait gives up (tens of ms)

__device__ __forceinline__ unsigned long long pack_pair(float m, float z) {
    return ((unsigned long long)__float_as_uint(z) << 32) | (unsigned long long)__float_as_uint(m);
}
__device__ __forceinline__ void unpack_pair(unsigned long long bits, float& m, float& z) {
    m = __uint_as_float((unsigned)(bits & 0xffffffffull));
    z = __uint_as_float((unsigned)(bits >> 32));
}
__device__ __forceinline__ void publish_pair(float2* p, float m, float z) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), pack_pair(m, z), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long load_pair_bits(const float2* p) {
    return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}
// Waits (bounded) until the word at p is a published pair; `bits` is what an earlier load saw.
__device__ __forceinline__ unsigned long long await_pair(const float2* p, unsigned long long bits,
                                                         unsigned limit, bool& gave_up) {
    unsigned spins = 0;
    while (bits == kInvalidPair) {
        if (gave_up || ++spins > limit) {   // once a wait has given up, later ones do not wait again
            gave_up = true;
            return pack_pair(-INFINITY, 0.f);
        }
        __builtin_amdgcn_s_sleep(2);
        bits = load_pair_bits(p);
    }
    return bits;
}

}  // namespace snapkv
#endif
