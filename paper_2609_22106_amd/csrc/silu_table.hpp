// SiLU of a bf16 gate by a fixed sequence of IEEE float32 operations, and the
// same sequence's results tabulated at compile time.
//
// SiLU(g) = g / (1 + e^-g) with e^x by a fixed sequence, one operation per step
// (contraction off), so the result does not depend on the device's own exp: x
// clamped to [-104, 89]; n = rint(x log2 e); r = (x - n ln2_hi) - n ln2_lo with
// ln 2 split into a 15-bit head (n ln2_hi exact) and a tail; e^r by its degree-6
// Taylor polynomial in Horner form; e^x = r's polynomial scaled by 2^n (exact,
// or one rounding where it is subnormal).
//
// A gate has 65536 values, and outside 2^-25 <= |g| < 2^7 the sequence reduces
// to one exact operation, so the 8192 gates inside (32 binades of 128 values,
// two signs) are all that a table needs: 32 KiB, which fits in LDS beside the
// workgroups that use it.  The table holds exactly what the sequence gives
// (evaluated by the compiler, operation by operation).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace prq {
namespace dev {

constexpr float kSiluLog2e = 0x1.715476p+0f;
constexpr float kSiluLn2Hi = 0x1.62e4p-1f, kSiluLn2Lo = 0x1.7f7d1cp-20f;
constexpr float kSiluTaylor[7] = {0x1.6c16c2p-10f, 0x1.111112p-7f, 0x1.555556p-5f,   // 1/6! 1/5! 1/4!
                                  0x1.555556p-3f, 0.5f, 1.0f, 1.0f};                 // 1/3! 1/2! 1 1

__device__ __forceinline__ float silu_seq(float g) {
#pragma clang fp contract(off)
  const float x = fminf(fmaxf(-g, -104.0f), 89.0f);
  const float n = rintf(x * kSiluLog2e);
  const float r = (x - n * kSiluLn2Hi) - n * kSiluLn2Lo;
  float p = kSiluTaylor[0];
#pragma unroll
  for (int i = 1; i < 7; ++i) p = p * r + kSiluTaylor[i];
  const float e = ldexpf(p, static_cast<int>(n));
  return __fdiv_rn(g, 1.0f + e);
}

// The sequence's result for a gate outside the table: below 2^-25 e^-g rounds to 1,
// from 2^7 on 1 + e^-g rounds to 1, from -2^7 down e^-g is infinite (-inf / inf is the
// device's NaN of an invalid division); NaN stays NaN.
__device__ __forceinline__ float silu_outside(float g) {
#pragma clang fp contract(off)
  const float scaled = g * (__builtin_fabsf(g) < 1.0f ? 0.5f : g > 0.0f ? 1.0f : 0.0f);
  return g == -INFINITY ? __uint_as_float(0xFFC00000u) : scaled;
}

// The table: entry sign * 4096 + (magnitude bits - kSiluTableBase) for the bf16
// gate with those bits, magnitude bits 0x3300 (2^-25) .. 0x42FF (just below 2^7).
constexpr uint32_t kSiluTableBase = 0x3300;
constexpr uint32_t kSiluTableHalf = 4096;

struct SiluTable {
  alignas(16) float v[2 * kSiluTableHalf];
};

// p 2^n in one rounding (two power-of-two products, the first of them exact).
constexpr float silu_table_scale(float p, int n) {
  const int far = n < -100 ? -60 : n > 100 ? 60 : 0;
  float a = 1.0f, b = 1.0f;
  for (int i = 0; i < (far < 0 ? -far : far); ++i) a *= far < 0 ? 0.5f : 2.0f;
  for (int i = 0; i < (n < 0 ? far - n : n - far); ++i) b *= n < 0 ? 0.5f : 2.0f;
  return (p * a) * b;
}

constexpr float silu_table_value(float g) {
#pragma clang fp contract(off)
  const float x = -g < -104.0f ? -104.0f : -g > 89.0f ? 89.0f : -g;
  const float big = 12582912.0f;                 // 1.5 2^23: adding and subtracting it is rint
  const float n = (x * kSiluLog2e + big) - big;
  const float r = (x - n * kSiluLn2Hi) - n * kSiluLn2Lo;
  float p = kSiluTaylor[0];
  for (int i = 1; i < 7; ++i) p = p * r + kSiluTaylor[i];
  return g / (1.0f + silu_table_scale(p, static_cast<int>(n)));
}

constexpr SiluTable make_silu_table() {
  SiluTable t{};
  for (int s = 0; s < 2; ++s) {
    float binade = 0x1p-25f;
    for (int e = 0; e < 32; ++e, binade *= 2.0f)
      for (int m = 0; m < 128; ++m) {
        const float g = binade * (1.0f + m * 0x1p-7f);
        t.v[s * kSiluTableHalf + e * 128 + m] = silu_table_value(s ? -g : g);
      }
  }
  return t;
}

}  // namespace dev
}  // namespace prq
