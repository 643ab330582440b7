// Packed weight layout for the block-scaled FP4 MFMA (an invertible byte
// permutation of the exported Q([W~, R_W]) of Eq. 3, applied once per weight).
//
// Canonical (prq_prepare output): Wq [E][N][K_aug/2], Wsc [E][N][K_aug/32].
// Packed, with S = ceil(K_aug / 128) K steps and T = N / 16 feature tiles:
//   Wp  [E][T][S][64 lanes][16 bytes]: lane l of block (t, s) holds the 16
//       code bytes of weight row 16t + (l % 16), K elements
//       [128 s + 32 (l / 16), +32), i.e. exactly what lane l feeds to the
//       v_mfma_scale_f32_16x16x128_f8f6f4 A/B operand; zero past K_aug.
//   Wps [E][T][ceil(S/4)][64 lanes][4 bytes]: byte j of lane l's dword in
//       group (t, q) is the E8M0 scale of row 16t + (l % 16), 32-block
//       4 (4q + j) + l / 16; 127 past K_aug.
// So one wave reads one contiguous kilobyte per MFMA operand and one dword of
// scales per four K steps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "prq_internal.h"

namespace prq {
namespace {

constexpr int kPackThreads = 256;

// One launch for both (128 experts of 2048 x 832, 232 MB: two launches 52.2 us, one
// 49.0, 4.7 TB/s where a plain copy reaches 5.1):
// workgroups [0, scale_blocks) gather scales -- first, so that their short loads
// run beside the code copies -- the rest copy codes.  (A launch holds 2^32 - 1
// threads: where both together are more, one launch each.)
//
// Codes: one thread per (e, t, s, lane), 16 bytes (4 dwords of one row).  Scales:
// one thread per (e, t, q, lane), 4 scale bytes into a dword.  Block numbers are
// divided in 32 bits: a launch has fewer than 2^26 of them.
__global__ __launch_bounds__(kPackThreads) void pack_weight_kernel(
    const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ Wsc, int N, int K_aug, int E,
    uint8_t* __restrict__ Wp, uint32_t* __restrict__ Wps, uint32_t scale_blocks) {
  const int S = (K_aug + 127) / 128;
  const int T = N / 16;
  const int l = static_cast<int>(threadIdx.x) & 63;
  if (blockIdx.x < scale_blocks) {
    const int Q = (S + 3) / 4;
    const int nb = K_aug / 32;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kPackThreads + threadIdx.x;
    if (i >= static_cast<int64_t>(E) * T * Q * 64) return;
    const uint32_t grp = static_cast<uint32_t>(i >> 6);        // (e * T + t) * Q + q
    const int q = static_cast<int>(grp % static_cast<uint32_t>(Q));
    const uint8_t* const row = Wsc + (static_cast<int64_t>(grp / static_cast<uint32_t>(Q)) * 16 + (l & 15)) * nb;
    uint32_t d = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int b = 4 * (4 * q + j) + (l >> 4);
      const uint32_t sc = b < nb ? row[b] : 127u;
      d |= sc << (8 * j);
    }
    Wps[i] = d;
    return;
  }
  const int64_t i = static_cast<int64_t>(blockIdx.x - scale_blocks) * kPackThreads + threadIdx.x;
  if (i >= static_cast<int64_t>(E) * T * S * 64) return;
  const uint32_t blk = static_cast<uint32_t>(i >> 6);          // (e * T + t) * S + s
  const int s = static_cast<int>(blk % static_cast<uint32_t>(S));
  const int64_t row = static_cast<int64_t>(blk / static_cast<uint32_t>(S)) * 16 + (l & 15);   // within [E * N]
  const int kel = s * 128 + (l >> 4) * 32;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (kel < K_aug)
    v = *reinterpret_cast<const uint4*>(Wq + row * (K_aug / 2) + kel / 2);
  *reinterpret_cast<uint4*>(Wp + i * 16) = v;
}

}  // namespace

size_t packed_code_bytes(int N, int K_aug, int E) {
  return static_cast<size_t>(E) * (N / 16) * ((K_aug + 127) / 128) * 1024;
}

size_t packed_scale_bytes(int N, int K_aug, int E) {
  return static_cast<size_t>(E) * (N / 16) * (((K_aug + 127) / 128 + 3) / 4) * 256;
}

int pack_launches(int N, int K_aug, int E, int64_t max_blocks, int64_t* code_blocks, int64_t* scale_blocks) {
  const int64_t nc = static_cast<int64_t>(packed_code_bytes(N, K_aug, E) / 16);
  const int64_t ns = static_cast<int64_t>(packed_scale_bytes(N, K_aug, E) / 4);
  *code_blocks = (nc + kPackThreads - 1) / kPackThreads;
  *scale_blocks = (ns + kPackThreads - 1) / kPackThreads;
  if (std::max(*code_blocks, *scale_blocks) > max_blocks) return 0;
  return *code_blocks + *scale_blocks > max_blocks ? 2 : 1;
}

hipError_t launch_pack_weight(const uint8_t* Wq, const uint8_t* Wsc, int N, int K_aug, int E,
                              uint8_t* Wp, uint8_t* Wps, hipStream_t stream, int64_t max_blocks) {
  int64_t code_blocks, scale_blocks;
  const int launches = pack_launches(N, K_aug, E, max_blocks, &code_blocks, &scale_blocks);
  if (launches == 0) return hipErrorInvalidValue;
  const auto launch = [&](int64_t blocks, int64_t scales) {
    pack_weight_kernel<<<static_cast<unsigned>(blocks), kPackThreads, 0, stream>>>(
        Wq, Wsc, N, K_aug, E, Wp, reinterpret_cast<uint32_t*>(Wps), static_cast<uint32_t>(scales));
  };
  if (launches == 1) {
    launch(code_blocks + scale_blocks, scale_blocks);
  } else {
    launch(scale_blocks, scale_blocks);
    launch(code_blocks, 0);
  }
  return hipGetLastError();
}

}  // namespace prq
