// Pieces shared by the matrix-core kernels (resident and streaming): fragment types, the error
// bound of the f16 hi/lo screen and the exchange between half-waves.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cham {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kRecCap = 64;            // queued rows whose knob values are kept in LDS
constexpr float kHalfMax = 65504.0f;   // largest f16 value

// The bias |mu'|^2 of a centroid is hi + lo (f16) times the value of the bias slot in B, a power of two such that
// kHalfMax of them, the score of a padding centroid row, exceed every score: with squared norms of rows and centroids up to
// N a score is at most 3 N, and inside the knobs' range N is 32 * 255^2 for byte knobs and 63 * 2047^2 for
// two-byte knobs below 2048.
constexpr float bias_scale(bool byte_knobs) { return byte_knobs ? 256.0f : 16384.0f; }
// The largest N the screen is used with (above both).  Starting centroids may lie anywhere.
constexpr float max_screened(bool byte_knobs) { return bias_scale(byte_knobs) * kHalfMax / 3.2f; }
static_assert(max_screened(true) > 32.0f * 255.0f * 255.0f && max_screened(false) > 63.0f * 2047.0f * 2047.0f, "rows never leave the range");

// Where the chain starts from |mu'|^2 in fp32, padding centroid rows start from kPadScore (real scores of usable starts stay far
// below: 4 * 32 * 255^2 for byte knobs).  Starts beyond the range of the operands take kFarNorm for their squared norm in the bound,
// which makes some 1e25 of it, and their scores are cut off at kFarScore: every centroid is a candidate of every row and padding never is.
constexpr float kPadScore = 1.0e30f, kFarNorm = 1.0e30f, kFarScore = 1.0e13f;

// Error bound of the matrix-core screen, relative to (|x'|^2 + 2 max|mu'|^2), in units of 2^-24:
// w = fl32(-2mu') and the bias are rounded once (1 each) and hi + lo keeps 22 bits (4);
// each instruction adds 16 exact products to the running value: the hardware aligns the 17 addends
// to the largest and rounds once, modelled generously as 18 units per instruction (NS2 chained
// instructions).  The factor 2.5 = 2 (two scores are compared) x 1.25 headroom.  The absolute
// term covers f16 underflow of the low parts: 2.5 * 2^-25 (half the spacing of subnormal values, which the
// instruction honours) times the bias slot of 256 is 1.9e-5, of 16384 1.2e-3.
template <int NS2, bool BYTE_KNOBS = true>
__device__ __forceinline__ float mfma_bound(float x2, float m2)
{
    constexpr float kE = 2.5f * (float)(18 * NS2 + 6) * 5.9604644775390625e-8f;
    return kE * (x2 + 2.0f * m2) + (BYTE_KNOBS ? 4.0e-5f : 2.5e-3f);
}

template <int NS2>
constexpr float mfma_bound_slope() { return 2.5f * (float)(18 * NS2 + 6) * 5.9604644775390625e-8f; }      // ... per |x'|^2

// Both 32-lane halves of a value: lo = the value held by lanes 0..31, hi = by lanes 32..63
// (v_permlane32_swap: a VALU exchange, no LDS round trip).
__device__ __forceinline__ void both_halves(unsigned v, unsigned &lo, unsigned &hi)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    lo = r[0];
    hi = r[1];
}

}  // namespace cham
