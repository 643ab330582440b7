// Device-side MXFP4 helpers for gfx950: E8M0 scale rule, E2M1 rounding,
// cross-lane reductions, and the block-scaled FP4 MFMA wrapper.
//
// MXFP4 (the format arXiv 2609.22106 uses for W4A4, after the OCP Microscaling
// specification it cites): 32 elements along K share an E8M0 scale
// 2^(code-127); code = clamp(biased_exp(amax) - 2, 0, 254) so the block
// maximum lands in E2M1's top binade [4, 8); each element divided by the scale
// is rounded to the nearest E2M1 value (0, .5, 1, 1.5, 2, 3, 4, 6), ties to
// the even code, saturating at 6.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace prq {
namespace dev {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16 bytes of a stream read once: a non-temporal load.  Used for the expert
// decode kernel's weight (128 experts' weights in one call, back to back:
// 24.9 -> 23.3 us); the dense decode kernel's weight loads measured the same
// back to back and 2.8 us slower over the graph-replayed decode step, and the
// quantizer's X copies slower at 2048 and 8192 rows, so both stay cached.
__device__ __forceinline__ uint4 load_stream16(const uint8_t* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// E8M0 code of a block with largest magnitude `amax` (finite, >= 0).  The
// float32 exponent field is floor(log2 amax) + 127 for normal amax and 0 for
// zero/subnormal amax, so subtracting emax(E2M1) = 2 and clamping at 0 is the
// whole rule (a finite amax has exponent field <= 254, so code <= 252).
__device__ __forceinline__ uint32_t e8m0_code(float amax) {
  int bexp = static_cast<int>((__float_as_uint(amax) >> 23) & 0xFFu);
  return static_cast<uint32_t>(bexp > 2 ? bexp - 2 : 0);
}

// 2^(127 - code): multiplying by it divides by the block scale exactly.
__device__ __forceinline__ float e8m0_reciprocal(uint32_t code) {
  return __uint_as_float((254u - code) << 23);
}

// Nearest E2M1 code of t (|t| < 8 after scaling), ties to the even code,
// saturating at 6.  The sign bit is taken from v, the unscaled value, so a
// negative value that underflows in the scaling still encodes as -0.
__device__ __forceinline__ uint32_t e2m1_code(float t, float v) {
  float a = fabsf(t);
  uint32_t idx = static_cast<uint32_t>(a > 0.25f) + static_cast<uint32_t>(a >= 0.75f) +
                 static_cast<uint32_t>(a > 1.25f) + static_cast<uint32_t>(a >= 1.75f) +
                 static_cast<uint32_t>(a > 2.5f) + static_cast<uint32_t>(a >= 3.5f) +
                 static_cast<uint32_t>(a > 5.0f);
  return idx | ((__float_as_uint(v) >> 31) << 3);
}

// Max over the 4 lanes of a quad (lanes 4q .. 4q+3) with two DPP quad
// permutations (xor 1, xor 2); every lane of the quad must be active.
__device__ __forceinline__ float quad_max(float x) {
  int xi = __float_as_int(x);
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, xi, 0xB1, 0xF, 0xF, false)));
  xi = __float_as_int(x);
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, xi, 0x4E, 0xF, 0xF, false)));
  return x;
}

// A quad's 32-block, 8 values per lane -> the lane's word of 8 codes and the
// block's scale code (in every lane).  t = z * 2^-e is exact (a power-of-two
// product whose magnitude stays below 8, or a signed zero/denormal that encodes
// as a signed zero either way); its E2M1 code comes from the hardware converter
// at scale 1, which rounds to nearest even and saturates at 6 exactly like the
// software rule on every float32 (checked exhaustively on the GPU).  Four
// converts, each writing its pair into one byte of the word.
__device__ __forceinline__ uint32_t quantize8(const float (&z)[8], uint32_t* scale) {
  float amax = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf(z[j]));
  const uint32_t code = e8m0_code(quad_max(amax));
  const float mul = e8m0_reciprocal(code);
  uint32_t w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, z[0] * mul, z[1] * mul, 1.0f, 0);
  w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, z[2] * mul, z[3] * mul, 1.0f, 1);
  w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, z[4] * mul, z[5] * mul, 1.0f, 2);
  w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, z[6] * mul, z[7] * mul, 1.0f, 3);
  *scale = code;
  return w;
}

// One 16x16x128 block-scaled MFMA with FP4 (E2M1) A and B operands:
//   C[i][j] += sum_{k<128} 2^(sa-127) A[i][k] * 2^(sb-127) B[k][j]
// Lane l supplies A row (l % 16), K elements [32*(l/16), 32*(l/16)+32) as 16
// bytes of packed nibbles, and that 32-block's E8M0 scale in bits 0-7 of sa;
// likewise B column (l % 16).  Lane l receives C[4*(l/16) + r][l % 16], r=0..3.
__device__ __forceinline__ v4f mfma_fp4_16x16x128(const uint4& a, const uint4& b, uint32_t sa,
                                                   uint32_t sb, v4f c) {
  v8i av = {static_cast<int>(a.x), static_cast<int>(a.y), static_cast<int>(a.z),
            static_cast<int>(a.w), 0, 0, 0, 0};
  v8i bv = {static_cast<int>(b.x), static_cast<int>(b.y), static_cast<int>(b.z),
            static_cast<int>(b.w), 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, c, 4, 4, 0,
                                                          static_cast<int>(sa), 0,
                                                          static_cast<int>(sb));
}

typedef float v16f __attribute__((ext_vector_type(16)));

// 32x32x64 block-scaled FP4 MFMA (the full-rate form: twice the products of
// the 16x16x128 form per issue slot): lane l supplies row l % 32, K elements
// [32 (l / 32), +32) of each operand with that block's E8M0 scale, and holds
// C[8 (j / 4) + 4 (l / 32) + j % 4][l % 32] in element j of the result.
__device__ __forceinline__ v16f mfma_fp4_32x32x64(const uint4& a, const uint4& b, uint32_t sa,
                                                  uint32_t sb, v16f c) {
  v8i av = {static_cast<int>(a.x), static_cast<int>(a.y), static_cast<int>(a.z),
            static_cast<int>(a.w), 0, 0, 0, 0};
  v8i bv = {static_cast<int>(b.x), static_cast<int>(b.y), static_cast<int>(b.z),
            static_cast<int>(b.w), 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 4, 0,
                                                         static_cast<int>(sa), 0,
                                                         static_cast<int>(sb));
}

// The same instruction with the scale bytes taken from byte kSelA of sa and
// byte kSelB of sb (the instruction's scale byte selects), so one register
// can carry the scales of several blocks.
template <int kSelA, int kSelB>
__device__ __forceinline__ v16f mfma_fp4_32x32x64_sel(const uint4& a, const uint4& b, uint32_t sa,
                                                      uint32_t sb, v16f c) {
  static_assert(kSelA >= 0 && kSelA < 4 && kSelB >= 0 && kSelB < 4, "byte select");
  v8i av = {static_cast<int>(a.x), static_cast<int>(a.y), static_cast<int>(a.z),
            static_cast<int>(a.w), 0, 0, 0, 0};
  v8i bv = {static_cast<int>(b.x), static_cast<int>(b.y), static_cast<int>(b.z),
            static_cast<int>(b.w), 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 4, kSelA,
                                                         static_cast<int>(sa), kSelB,
                                                         static_cast<int>(sb));
}

// Group g with off[g] <= row < off[g+1] for non-decreasing offsets
// (empty groups are skipped): the largest g in [0, G) with off[g] <= row.  A
// whole wave looks for one row (every lane active): up to 256 groups it counts the
// offsets at or below the row, 64 to a load; more groups are first cut to one of 64
// equal pieces by their first offsets (two round trips up to 4096 groups).  A binary
// search waits for its loads one after the other, counting alone takes one for every
// 64 groups (us, 64 rows of 768, row-major, binary / counted / this: 128 groups 3.28 /
// 2.91 / 2.82, 512 3.53 / 3.64 / 2.86, 4096 3.96 / 11.1 / 2.91).
__device__ __forceinline__ int wave_find_group(const int32_t* __restrict__ off, int G, int row) {
  const int lane = static_cast<int>(threadIdx.x) & 63;
  int lo = 0, n = G;                       // the group is in [lo, lo + n)
  while (n > 256) {
    const int piece = (n + 63) >> 6;
    const bool in = lane * piece < n;
    const int at = off[in ? lo + lane * piece : lo];
    const int k = max(__popcll(__ballot(in && at <= row)), 1) - 1;
    lo += k * piece;
    n = min(piece, n - k * piece);
  }
  int c = 0;
#pragma unroll 4
  for (int b = 0; b < n; b += 64) {
    const int i = b + lane;
    const int at = off[lo + (i < n ? i : n - 1)];
    c += __popcll(__ballot(i < n && at <= row));
  }
  return lo + max(c, 1) - 1;
}

// Group of rows visited in increasing order, from the group of some row before
// them.  When a row leaves its group: a step forward (a load each, the last one the
// end of the group it stops at), after two of them (a group for every row, empty
// groups) steps that double and a binary search over the last one: 4096 rows of 64
// in 4096 groups, whose threads start up to 63 groups ahead, 12.3 us with single
// steps, 5.3 so.  Same result as the search for non-decreasing offsets; g stays in [0, G)
// whatever they hold.
struct GroupCursor {
  int g, g_end = 0;
  __device__ __forceinline__ explicit GroupCursor(int start) : g(start) {}
  __device__ __forceinline__ int at(const int32_t* __restrict__ off, int G, int row) {
    if (row >= g_end) {
      for (int steps = 0; g + 1 < G && off[g + 1] <= row; ++steps) {
        ++g;
        if (steps == 1) {
          int stride = 1;
          for (; g + stride < G && off[g + stride] <= row; stride <<= 1) g += stride;
          for (int end = min(g + stride, G); end - g > 1;) {
            const int mid = (g + end) >> 1;
            if (off[mid] <= row)
              g = mid;
            else
              end = mid;
          }
          break;
        }
      }
      g_end = g + 1 < G ? off[g + 1] : 0x7fffffff;
    }
    return g;
  }
};

}  // namespace dev
}  // namespace prq
