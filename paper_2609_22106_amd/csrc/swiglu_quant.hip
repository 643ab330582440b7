// Offline copy, producer side (arXiv 2609.22106, Sec. Method, "Activation tail
// construction"; Eq. 1 with sigma = SiLU): the expanded up/gate projections emit
// gate and up outputs K_aug = C + k wide whose product SiLU(gate) * up is
// already [Z~, Z~_tail], so the down-projection's MXFP4 input is that product
// quantized -- no gather, no scaling, no tail copy.  The product is formed in
// float32 and never rounded to bf16.
//
// Bytes: 4 in and 17/32 out per element, so memory should bound it; the SiLU
// sequence (about 40 operations and a correctly rounded division) made it bound
// by the vector units instead.  From kTableMinUnits on, SiLU is therefore
// looked up: the 8192 gates whose SiLU is not one exact operation, tabulated by
// the compiler (silu_table.hpp), are copied into each workgroup's LDS (32 KiB,
// four workgroups of 512 threads per CU) and gathered; a wave with a gate outside
// the table selects between the entry and that operation.  Measured at M = 8192,
// K_aug = 9984 (371 MB): packed 113 -> 75.6 us (4.9 TB/s; a plain copy of as many bytes
// takes 73), row-major 99 -> 75.6; one gate in twenty zero 79.6 and 80.6, all zero 80.6
// and 81.1 (107 to 118 when such a thread ran the sequence for its eight gates).
//
// A wave's task in the packed layout is one K step (128 elements) of a 16-row
// block: 8 lanes read 128 contiguous bytes of a row, and the wave writes the
// step's whole contiguous kilobyte of codes.  (One thread per unit in row order,
// as the row-major output has it, writes 16 bytes of every 256: eight rows, far
// apart in time, to complete a line.)  Row-major: a task is 512 elements of a
// row, 1 KiB read and 256 bytes written contiguously.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "mx_device.hpp"
#include "prq_internal.h"
#include "silu_table.hpp"

namespace prq {
namespace {

// Threads of a workgroup with the table, and without; passes of a wave's task.
constexpr int kThreads[2] = {256, 512};
constexpr int kPasses[2] = {1, 4};
constexpr int kPerCu = 4;            // workgroups with tables a CU holds (2048 threads, 128 KiB; 64 registers)

// Type that task numbers are divided in: 32 bits without the table (few tasks:
// a 64-bit division there costs 0.1 us of a 2.4 us call).
template <bool kTable>
using TaskIndex = std::conditional_t<kTable, uint64_t, uint32_t>;

__device__ constexpr dev::SiluTable kSiluTable = dev::make_silu_table();

// 8 gates and ups (bf16 pairs, low half first) -> SiLU(gate) * up.
template <bool kTable>
__device__ __forceinline__ void gated8(const uint4& gv, const uint4& uv, const float* tab,
                                       float (&z)[8]) {
#pragma clang fp contract(off)
  const uint32_t gw[4] = {gv.x, gv.y, gv.z, gv.w};
  const uint32_t uw[4] = {uv.x, uv.y, uv.z, uv.w};
  float s[8];
  if constexpr (kTable) {
    uint32_t at[8], most = 0;   // byte offset of the magnitude in its half of the table
    constexpr uint32_t kHalf = 4 * dev::kSiluTableHalf;
    auto entry = [&](uint32_t offset, uint32_t sign) {
      return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(tab) + (offset + sign * kHalf));
    };
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t mag = (j & 1) ? (gw[j >> 1] >> 16) & 0x7FFFu : gw[j >> 1] & 0x7FFFu;
      at[j] = 4 * mag - 4 * dev::kSiluTableBase;
      most = max(most, at[j]);
    }
    if (__all(most < kHalf)) {   // (the whole wave's branches)
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] = entry(at[j], (j & 1) ? gw[j >> 1] >> 31 : (gw[j >> 1] >> 15) & 1u);
    } else {
      // Two gates at a time, from words that the compiler cannot take for those
      // above: 64 registers hold four workgroups a CU.
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t w = gw[j];
        asm volatile("" : "+v"(w));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float g = __uint_as_float(h ? w & 0xFFFF0000u : w << 16);
          const uint32_t offset = (__float_as_uint(fabsf(g)) >> 14) - 4 * dev::kSiluTableBase;
          const float t = entry(min(offset, kHalf - 4), __float_as_uint(g) >> 31);
          s[2 * j + h] = offset < kHalf ? t : dev::silu_outside(g);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s[2 * j] = dev::silu_seq(__uint_as_float(gw[j] << 16));
      s[2 * j + 1] = dev::silu_seq(__uint_as_float(gw[j] & 0xFFFF0000u));
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    z[2 * j] = s[2 * j] * __uint_as_float(uw[j] << 16);
    z[2 * j + 1] = s[2 * j + 1] * __uint_as_float(uw[j] & 0xFFFF0000u);
  }
}

// Copy the table into LDS (every thread; a barrier follows).
__device__ __forceinline__ void fill_table(float* tab) {
  constexpr int kVecs = sizeof(dev::SiluTable) / 16;
  static_assert(alignof(dev::SiluTable) == 16 && kVecs % kThreads[1] == 0, "moved 16 bytes a thread at a time");
  const uint4* src = reinterpret_cast<const uint4*>(kSiluTable.v);
#pragma unroll
  for (int i = 0; i < kVecs / kThreads[1]; ++i)
    reinterpret_cast<uint4*>(tab)[threadIdx.x + i * kThreads[1]] = src[threadIdx.x + i * kThreads[1]];
}

// Packed layout.  A K step of a 16-row block is four passes of 8 rows x 64
// elements; in a pass, lane l holds row l / 8, K part (l / 4) % 2, quarter l % 4.
// Wave task t = (row block t / steps, K step t % steps), all four passes with
// their loads in flight (with the table), or a single pass: then four
// consecutive tasks are a step's.  A wave takes tasks t, t + stride, ...
// K parts past K_aug and rows past M: zero codes, scale byte 127; the last step's
// tasks also write the scale bytes up to the end of its group of four steps.
template <bool kTable>
__global__ __launch_bounds__(kThreads[kTable]) void swiglu_quant_packed_kernel(
    const uint16_t* __restrict__ G, const uint16_t* __restrict__ U, int64_t ld, int M, int K_aug,
    int64_t tasks, uint8_t* __restrict__ Ap, uint8_t* __restrict__ Aps) {
  __shared__ __align__(16) float tab[kTable ? 2 * dev::kSiluTableHalf : 4];
  if constexpr (kTable) {
    fill_table(tab);
    __syncthreads();
  }
  const int steps = (K_aug + 127) >> 7;
  const int sgroups = (steps + 3) >> 2;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int q = lane & 3, pp = (lane >> 2) & 1, r8 = lane >> 3;
  using Index = TaskIndex<kTable>;
  constexpr int kWaves = kThreads[kTable] / 64, kP = kPasses[kTable];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kWaves;
  const int64_t first = static_cast<int64_t>(blockIdx.x) * kWaves + wave;
  // (row block, step) of the task, advanced by the stride without a division
  const int per_block = steps * (4 / kP);
  int rb = static_cast<int>(Index(first) / Index(per_block)), at_task = static_cast<int>(Index(first) % Index(per_block));
  const int drb = static_cast<int>(Index(stride) / Index(per_block)), ds = static_cast<int>(Index(stride) % Index(per_block));
  for (int64_t t = first; t < tasks; t += stride) {
    const int s = kP == 4 ? at_task : at_task >> 2;
    const int c0 = kP == 4 ? 0 : at_task & 3;
    uint4 gv[kP], uv[kP];
    bool ok[kP];
#pragma unroll
    for (int i = 0; i < kP; ++i) {
      const int c = c0 + i;             // 8-row half c / 2, K part pair c % 2
      const int row = rb * 16 + (c >> 1) * 8 + r8;
      const int k = s * 128 + ((c & 1) * 2 + pp) * 32 + q * 8;
      ok[i] = row < M && k < K_aug;     // quad-uniform (K_aug % 32 == 0)
      gv[i] = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);   // 1 x 0
      uv[i] = make_uint4(0, 0, 0, 0);
      if (ok[i]) {
        const int64_t at = static_cast<int64_t>(row) * ld + k;
        gv[i] = *reinterpret_cast<const uint4*>(G + at);
        uv[i] = *reinterpret_cast<const uint4*>(U + at);
      }
    }
    uint8_t* const code = Ap + (static_cast<int64_t>(rb) * steps + s) * 1024 + pp * 256 + r8 * 16 + q * 4;
    uint32_t mine = 127;                // lane q of a quad stores pass q's scale byte
#pragma unroll
    for (int i = 0; i < kP; ++i) {
      const int c = c0 + i;
      float z[8];
      gated8<kTable>(gv[i], uv[i], tab, z);
      uint32_t sc;
      const uint32_t w = dev::quantize8(z, &sc);
      *reinterpret_cast<uint32_t*>(code + (c & 1) * 512 + (c >> 1) * 128) = w;
      mine = q == c ? (ok[i] ? sc : 127u) : mine;
    }
    if (kP == 4 || q == c0) {
      uint8_t* const sp = Aps + (static_cast<int64_t>(rb) * sgroups + (s >> 2)) * 256 +
                          ((q & 1) * 2 + pp) * 64 + ((q >> 1) * 8 + r8) * 4;
      sp[s & 3] = static_cast<uint8_t>(mine);
      if (s == steps - 1)
        for (int j = (s & 3) + 1; j < 4; ++j) sp[j] = 127;
    }
    rb += drb;
    at_task += ds;
    if (at_task >= per_block) {
      at_task -= per_block;
      ++rb;
    }
  }
}

// Row-major.  Wave task t = (row t / chunks, 512-element chunk t % chunks); with
// the table a wave takes four at a time, their loads all in flight.
template <bool kTable>
__global__ __launch_bounds__(kThreads[kTable]) void swiglu_quant_rows_kernel(
    const uint16_t* __restrict__ G, const uint16_t* __restrict__ U, int64_t ld, int K_aug,
    int64_t tasks, uint8_t* __restrict__ Aq, uint8_t* __restrict__ Asc) {
  __shared__ __align__(16) float tab[kTable ? 2 * dev::kSiluTableHalf : 4];
  if constexpr (kTable) {
    fill_table(tab);
    __syncthreads();
  }
  const int units = K_aug >> 3, nb = K_aug >> 5;
  const int chunks = (units + 63) >> 6;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  using Index = TaskIndex<kTable>;
  constexpr int kWaves = kThreads[kTable] / 64, kBatch = kPasses[kTable];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kWaves;
  const int64_t first = static_cast<int64_t>(blockIdx.x) * kWaves + wave;
  int r = static_cast<int>(Index(first) / Index(chunks)), ch = static_cast<int>(Index(first) % Index(chunks));
  const int dr = static_cast<int>(Index(stride) / Index(chunks)), dc = static_cast<int>(Index(stride) % Index(chunks));
  for (int64_t t = first; t < tasks; t += kBatch * stride) {
    uint4 gv[kBatch], uv[kBatch];
    int row[kBatch], u[kBatch];
#pragma unroll
    for (int c = 0; c < kBatch; ++c) {
      row[c] = r;
      u[c] = t + c * stride < tasks ? ch * 64 + lane : units;
      if (u[c] < units) {               // quad-uniform
        const int64_t at = static_cast<int64_t>(r) * ld + u[c] * 8;
        gv[c] = *reinterpret_cast<const uint4*>(G + at);
        uv[c] = *reinterpret_cast<const uint4*>(U + at);
      }
      r += dr;
      ch += dc;
      if (ch >= chunks) {
        ch -= chunks;
        ++r;
      }
    }
#pragma unroll
    for (int c = 0; c < kBatch; ++c) {
      if (u[c] < units) {
        float z[8];
        gated8<kTable>(gv[c], uv[c], tab, z);
        uint32_t sc;
        const uint32_t w = dev::quantize8(z, &sc);
        *reinterpret_cast<uint32_t*>(Aq + static_cast<int64_t>(row[c]) * (K_aug >> 1) + 4 * u[c]) = w;
        if ((lane & 3) == 0) Asc[static_cast<int64_t>(row[c]) * nb + (u[c] >> 2)] = static_cast<uint8_t>(sc);
      }
    }
  }
}

// From this many 8-element units on SiLU is looked up (row-major, packed).
// Below, filling the tables costs more than the sequence (us, looked up /
// computed, M x K_aug): row-major 48 x 9984 2.71 / 2.65, 64 x 9984 2.69 / 3.12;
// packed 128 x 9984 4.35 / 4.08 (a task is 2048 elements: few waves), 256 x 9984
// 5.01 / 5.29, 512 x 9984 7.27 / 9.03.
constexpr int64_t kTableMinUnits[2] = {70000, 200000};

template <bool kTable>
void launch_mode(const uint16_t* G, const uint16_t* U, int64_t ld, int M, int K_aug, uint8_t* Aq,
                 uint8_t* Asc, bool packed, int num_cus, hipStream_t stream) {
  constexpr int kWaves = kThreads[kTable] / 64;
  const int64_t tasks = packed ? static_cast<int64_t>((M + 15) / 16) * ((K_aug + 127) / 128) * (4 / kPasses[kTable])
                               : static_cast<int64_t>(M) * ((K_aug / 8 + 63) / 64);
  // With tables: one round of workgroups, each filling its table once.
  const int64_t most = kTable ? static_cast<int64_t>(std::max(num_cus, 1)) * kPerCu : int64_t{1} << 22;
  const dim3 grid(static_cast<unsigned>(std::min<int64_t>((tasks + kWaves - 1) / kWaves, most)));
  if (packed)
    swiglu_quant_packed_kernel<kTable><<<grid, kThreads[kTable], 0, stream>>>(G, U, ld, M, K_aug, tasks, Aq, Asc);
  else
    swiglu_quant_rows_kernel<kTable><<<grid, kThreads[kTable], 0, stream>>>(G, U, ld, K_aug, tasks, Aq, Asc);
}

}  // namespace

// mode: 0 = by size, 1 = the sequence, 2 = the table.
hipError_t launch_swiglu_quant(const uint16_t* G, const uint16_t* U, int64_t ld, int M, int K_aug,
                               uint8_t* Aq, uint8_t* Asc, bool packed, int num_cus,
                               hipStream_t stream, int mode) {
  const bool table = mode == 2 || (mode == 0 && static_cast<int64_t>(M) * (K_aug / 8) >= kTableMinUnits[packed]);
  if (table)
    launch_mode<true>(G, U, ld, M, K_aug, Aq, Asc, packed, num_cus, stream);
  else
    launch_mode<false>(G, U, ld, M, K_aug, Aq, Asc, packed, num_cus, stream);
  return hipGetLastError();
}

}  // namespace prq
