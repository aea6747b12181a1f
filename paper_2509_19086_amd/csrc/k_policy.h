// The policy key of a pair (Sec. 3.5 phase 3), and which batches a form serves: what the kernels that compare jobs share.
#pragma once

#include "sja_internal.h"

namespace sja {

// The batches that a form serves: those whose plan, which only the device knows, has class tables and at most so many classes.
constexpr int kAnyClasses = kMaxClasses, kNoClasses = -1;
__device__ __forceinline__ bool serves(const int32_t *plan, int most_classes) { return plan[kPlanTabled] && plan[kPlanClasses] <= most_classes; }

struct PolicyDev {
    int policy;
    int wait_scale;
    int w0, w1, w2;
    int class0_override;
};

// Per-job multiplier and tier of the policy key: key = (tier, F * mult [, F]).
__device__ __forceinline__ void job_policy(const PolicyDev &pol, const int32_t *wait,
                                           const uint8_t *sla_class, int j,
                                           unsigned long long &mult, unsigned long long &tier)
{
    const int cls = sla_class ? sla_class[j] : 0;
    const long long wt = wait ? wait[j] : 0;
    mult = 1;
    tier = 0;
    switch (pol.policy) {
    case SJA_POLICY_FAIRNESS: mult = (unsigned long long)(pol.wait_scale + wt); break;
    case SJA_POLICY_SLA:
        mult = (unsigned long long)(cls == 0 ? pol.w0 : (cls == 1 ? pol.w1 : pol.w2));
        tier = (pol.class0_override && cls == 0) ? 1 : 0;
        break;
    case SJA_POLICY_MIXED:
        mult = (unsigned long long)(pol.wait_scale + wt);
        tier = (unsigned long long)(2 - cls);
        break;
    default: break;
    }
}

// F = duration x peak and F x multiplier with as few of the (slow) 32-bit integer
// multiplies as the value ranges allow: durations, peaks and multipliers are
// non-negative and fit 32 bits, and a score stays below 2^62.
__device__ __forceinline__ unsigned long long rect_of(int dur, int peak)
{
    return static_cast<unsigned long long>(uint32_t(dur)) * uint32_t(peak);
}

__device__ __forceinline__ unsigned long long times_mult(unsigned long long F, unsigned long long mult)
{
    const uint32_t m = uint32_t(mult);            // wait_scale + wait, or an SLA weight: below 2^32
    return static_cast<unsigned long long>(uint32_t(F)) * m +
           (static_cast<unsigned long long>(uint32_t(F >> 32) * m) << 32);
}

// The leading 32 bits of a key as they matter: tier, exponent and the leading bits of the score, which grow with
// the key.  Scores spread over tens of octaves, so a byte of this orders more than a byte of the key.
__device__ __forceinline__ uint32_t key_digest(const PolicyDev &pol, unsigned long long tier, unsigned long long score)
{
    const int tier_bits = pol.policy == SJA_POLICY_MIXED ? 2 : pol.policy == SJA_POLICY_SLA ? 1 : 0, rest = 26 - tier_bits;
    const int e = score ? 63 - __clzll((long long)score) : 0;
    const unsigned long long mantissa = e ? score << (64 - e) : 0ull;
    return (tier_bits ? uint32_t(tier) << (32 - tier_bits) : 0u) | (uint32_t(e) << rest) | uint32_t(mantissa >> (64 - rest));
}

}  // namespace sja
