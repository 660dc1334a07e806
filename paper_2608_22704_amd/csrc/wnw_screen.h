// Error bound of the voice-hits screen (voice_screen_kernel): how far a logit from the bf16 matrix cores
// may be from the exact one, and for which values that holds.  Plain arithmetic that runs on the CPU too.
//
// Let S = sum |q_d| kmax_d >= sum |q_d k_d| (kmax_d: the largest |k_d| of the keys in question).  Products of
// bf16 values are exact in fp32; 127 additions that may each lose a unit of the last place (2^-23) of at
// most S lose under 2^-16 S, and VF_GAMMA leaves a factor of four for the order and alignment inside the
// instruction, which is not documented.  Nothing is assumed about subnormal values: a unit that flushes
// them loses 2^-126 per product and addition (under 2^-118 in all, 2^-18 S from S = 2^-100 up) and 2^-126
// |q|_1 or 128 * 2^-126 max kmax_d where it flushes elements of k or q (2^-19 S at most, by the range check).
#pragma once

#ifdef __HIPCC__
#define WNW_HOST_DEVICE __host__ __device__
#else
#define WNW_HOST_DEVICE
#endif

namespace wnw {

constexpr float VF_GAMMA = 0x1p-14f;

// Whether the bound VF_GAMMA * S holds (false for NaN and infinite values); q1 = |q|_1, kmax = max kmax_d.
WNW_HOST_DEVICE inline bool screen_in_range(float S, float q1, float kmax)
{
    return S >= 0x1p-100f && S < 0x1p120f && q1 * 0x1p-100f <= S && kmax * 0x1p-100f <= S;
}

}  // namespace wnw
