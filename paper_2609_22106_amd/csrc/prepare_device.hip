// The construction of one export on the device, for the offline alpha search
// (arXiv 2609.22106, Algorithm 1, steps 1-10): channel maxima, column-wise
// MXFP4 error of W D_alpha, top-k tail selection and permutation, Q(W~) and the
// quantized tail residual.  Every float operation, and the order of the error
// sums, is prq_prepare_ex's, so the codes, scales and permutation are the same
// bits; the scales themselves (C library pow) stay on the host.
//
// The host construction took ~80 ms per alpha on the 9728 -> 2560 down_proj (one
// pass after another over 100 MB float intermediates); here the weight is read
// as bf16 (50 MB) once for all alphas' column errors, whose serial double sums
// bound that kernel (three alphas 0.10 ms; ranking them 0.09), and once per alpha
// for the codes (0.026 ms, 2.5 TB/s).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mx_device.hpp"
#include "prq_internal.h"

// Every product and sum rounds as written (as in prepare.cpp).
#pragma clang fp contract(off)

namespace prq {
namespace {

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Value of an E2M1 code under an E8M0 code (exact; subnormal where it must be).
__device__ __forceinline__ float e2m1_value(uint32_t code, uint32_t scale) {
  const uint32_t m = code & 7u;   // 0 .5 1 1.5 2 3 4 6: exponent m / 2, mantissa bit m % 2
  const float mag = m < 2u ? 0.5f * static_cast<float>(m)
                           : __uint_as_float(((m >> 1) + 126u) << 23 | (m & 1u) << 22);
  const float s = __uint_as_float(scale ? scale << 23 : 0x00400000u);   // 2^(scale - 127)
  const float v = mag * s;
  return (code & 8u) ? -v : v;
}

// Largest |x| of each column as bits of its bf16 magnitude shifted to float32
// position (0 where the column holds only NaN, which is skipped); out starts at 0.
__global__ __launch_bounds__(256) void channel_maxima_kernel(const uint16_t* __restrict__ X, int rows,
                                                             int K, int rows_per_wg,
                                                             uint32_t* __restrict__ out) {
  const int c = (blockIdx.x * 256 + threadIdx.x) * 8;
  if (c >= K) return;
  const int r0 = blockIdx.y * rows_per_wg, r1 = min(rows, r0 + rows_per_wg);
  uint32_t m[8] = {};
  for (int r = r0; r < r1; ++r) {
    const uint4 v = *reinterpret_cast<const uint4*>(X + static_cast<int64_t>(r) * K + c);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t a = ((j & 1) ? w[j >> 1] & 0x7FFF0000u : (w[j >> 1] << 16) & 0x7FFF0000u);
      m[j] = a <= 0x7F800000u ? max(m[j], a) : m[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (m[j]) atomicMax(out + c + j, m[j]);
}

// Column errors of one 32-column block (blockIdx.x) for one alpha (blockIdx.y):
// err_j = sum over n, in increasing n, of (W_s - Q(W_s))^2 in double.  A tile is
// 64 rows, a quad of threads per row block; the 32 columns' sums run serially
// over a tile's rows (one lane each of the first wave, a double fma per row whose
// square is exact), while the next tile's errors go to the other buffer.
__global__ __launch_bounds__(256) void column_error_kernel(const uint16_t* __restrict__ W, int N, int K,
                                                           const float* __restrict__ scale,
                                                           double* __restrict__ err) {
  __shared__ float e[2][64][33];
  const int tid = threadIdx.x, r = tid >> 2, q = tid & 3;
  const int c = blockIdx.x * 32 + q * 8;
  const float* sc = scale + static_cast<int64_t>(blockIdx.y) * K + c;
  float s[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) s[j] = sc[j];
  double sum = 0.0;
  const int tiles = (N + 63) / 64;
  auto load = [&](int t) {
    const int n = t * 64 + r;
    return n < N ? *reinterpret_cast<const uint4*>(W + static_cast<int64_t>(n) * K + c) : make_uint4(0, 0, 0, 0);
  };
  uint4 next = load(0);
  for (int t = 0; t < tiles; ++t) {
    const uint32_t w[4] = {next.x, next.y, next.z, next.w};
    if (t + 1 < tiles) next = load(t + 1);
    float v[8], amax = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = ((j & 1) ? bf16_hi(w[j >> 1]) : bf16_lo(w[j >> 1])) * s[j];
      amax = fmaxf(amax, fabsf(v[j]));
    }
    const uint32_t code = dev::e8m0_code(dev::quad_max(amax));
    const float mul = dev::e8m0_reciprocal(code);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      e[t & 1][r][q * 8 + j] = v[j] - e2m1_value(dev::e2m1_code(v[j] * mul, v[j]), code);   // exact
    __syncthreads();
    if (tid < 32) {
#pragma unroll 8
      for (int i = 0; i < 64; ++i) {   // rows past N hold zero errors
        const double d = static_cast<double>(e[t & 1][i][tid]);
        sum = fma(d, d, sum);
      }
    }
  }
  if (tid < 32) err[static_cast<int64_t>(blockIdx.y) * K + blockIdx.x * 32 + tid] = sum;
}

// Rank of each column's error (number of columns before it: larger error, then
// smaller index), added up over blockIdx.z slices of the columns.  Errors are
// non-negative, so their bits order them (and give NaN a place too).
__global__ __launch_bounds__(256) void error_rank_kernel(const double* __restrict__ err, int K,
                                                         int32_t* __restrict__ rank) {
  __shared__ uint64_t part[256];
  const uint64_t* bits = reinterpret_cast<const uint64_t*>(err) + static_cast<int64_t>(blockIdx.y) * K;
  const int j = blockIdx.x * 256 + threadIdx.x;
  const uint64_t mine = j < K ? bits[j] : 0;
  const int per = (K + static_cast<int>(gridDim.z) - 1) / static_cast<int>(gridDim.z);
  const int i0 = blockIdx.z * per, i1 = min(K, i0 + per);
  int before = 0;
  for (int b = i0; b < i1; b += 256) {
    __syncthreads();
    if (b + static_cast<int>(threadIdx.x) < i1) part[threadIdx.x] = bits[b + threadIdx.x];
    __syncthreads();
    const int n = min(256, i1 - b);
    for (int i = 0; i < n; ++i) before += part[i] > mine || (part[i] == mine && b + i < j);
  }
  if (j < K && before) atomicAdd(rank + static_cast<int64_t>(blockIdx.y) * K + j, before);
}

// The permutation of one alpha (a workgroup each): columns of rank >= k in
// increasing order, then the k selected ones in increasing order, and the scales
// and inverse scales in position order.
constexpr int kPermThreads = 1024;

__global__ __launch_bounds__(kPermThreads) void tail_permutation_kernel(
    const int32_t* __restrict__ rank, const float* __restrict__ scale, const float* __restrict__ inv,
    int K, int k_tail, int32_t* __restrict__ perm, float* __restrict__ scale_pos,
    float* __restrict__ inv_pos) {
  __shared__ int scan[kPermThreads];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * K;
  const int tid = threadIdx.x;
  const int per = (K + kPermThreads - 1) / kPermThreads;
  const int j0 = min(K, tid * per), j1 = min(K, j0 + per);
  int mine = 0;
  for (int j = j0; j < j1; ++j) mine += rank[base + j] < k_tail;
  scan[tid] = mine;
  __syncthreads();
  for (int d = 1; d < kPermThreads; d <<= 1) {
    const int v = tid >= d ? scan[tid - d] : 0;
    __syncthreads();
    scan[tid] += v;
    __syncthreads();
  }
  int selected = scan[tid] - mine;   // selected columns before j
  for (int j = j0; j < j1; ++j) {
    const bool sel = rank[base + j] < k_tail;
    const int p = sel ? K - k_tail + selected : j - selected;   // ranks are distinct: p in [0, K)
    selected += sel;
    perm[base + p] = j;
    scale_pos[base + p] = scale[base + j];
    inv_pos[base + p] = inv[base + j];
  }
}

// sum_i (v_i - deq_i)^2 of a quad's block in double, one element at a time in
// index order: the four lanes add their eight in turn.
__device__ __forceinline__ double block_error(const float (&v)[8], uint32_t code) {
  const float mul = dev::e8m0_reciprocal(code);
  double d2[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const double d = static_cast<double>(v[j]) -
                     static_cast<double>(e2m1_value(dev::e2m1_code(v[j] * mul, v[j]), code));
    d2[j] = d * d;
  }
  double sum = 0.0;
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    double s = sum;
#pragma unroll
    for (int j = 0; j < 8; ++j) s += d2[j];
    sum = __shfl(s, (threadIdx.x & 60) + l, 64);   // lane l of the quad's
  }
  return sum;
}

// E8M0 code of a quad's block: the OCP code, or with kSearch the first of c0,
// c0 - 1, c0 + 1 (clamped to [0, 254]) with the smallest block error.
template <bool kSearch>
__device__ __forceinline__ uint32_t block_code(const float (&v)[8]) {
  float amax = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf(v[j]));
  const int c0 = static_cast<int>(dev::e8m0_code(dev::quad_max(amax)));
  uint32_t best = c0;
  if constexpr (kSearch) {
    double best_err = block_error(v, best);
#pragma unroll
    for (int off = -1; off <= 1; off += 2) {
      const uint32_t c = min(max(c0 + off, 0), 254);
      const double e = block_error(v, c);
      if (e < best_err) {
        best_err = e;
        best = c;
      }
    }
  }
  return best;
}

// Rows of Q([W~, R]) (canonical layout), a row at a time staged in LDS: a thread
// gathers the 8 channels of a unit (quarter block), a quad quantizes its block;
// a tail block's residual is quantized by the same quad.
constexpr int kAugThreads = 512;

template <bool kSearch>
__global__ __launch_bounds__(kAugThreads) void augment_kernel(
    const uint16_t* __restrict__ W, int N, int K, int k_tail, const int32_t* __restrict__ perm,
    const float* __restrict__ scale_pos, uint8_t* __restrict__ Wq, uint8_t* __restrict__ Wsc) {
  extern __shared__ __align__(16) uint16_t row_lds[];
  const int units = K >> 3, tail_unit0 = (K - k_tail) >> 3;
  const int nb = (K + k_tail) >> 5;
  for (int n = blockIdx.x; n < N; n += gridDim.x) {
    const uint4* src = reinterpret_cast<const uint4*>(W + static_cast<int64_t>(n) * K);
    __syncthreads();
    for (int u = threadIdx.x; u < units; u += kAugThreads) reinterpret_cast<uint4*>(row_lds)[u] = src[u];
    __syncthreads();
    uint32_t* const out = reinterpret_cast<uint32_t*>(Wq + static_cast<int64_t>(n) * ((K + k_tail) >> 1));
    uint8_t* const osc = Wsc + static_cast<int64_t>(n) * nb;
    for (int u = threadIdx.x; u < units; u += kAugThreads) {   // quad-uniform: units % 4 == 0
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        v[j] = __uint_as_float(static_cast<uint32_t>(row_lds[perm[8 * u + j]]) << 16) * scale_pos[8 * u + j];
      auto put = [&](int unit, uint32_t code) {
        const float mul = dev::e8m0_reciprocal(code);
        uint32_t w = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) w |= dev::e2m1_code(v[j] * mul, v[j]) << (4 * j);
        out[unit] = w;
        if ((unit & 3) == 0) osc[unit >> 2] = static_cast<uint8_t>(code);
        return w;
      };
      const uint32_t code = block_code<kSearch>(v);
      const uint32_t w = put(u, code);
      if (u >= tail_unit0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = v[j] - e2m1_value((w >> (4 * j)) & 15u, code);   // exact (Eq. 2)
        put(u + (k_tail >> 3), block_code<kSearch>(v));
      }
    }
  }
}

}  // namespace

hipError_t launch_channel_maxima(const uint16_t* X, int rows, int K, uint32_t* out, hipStream_t stream) {
  const int per = std::max(8, (rows + 127) / 128);
  const dim3 grid((K / 8 + 255) / 256, (rows + per - 1) / per);
  channel_maxima_kernel<<<grid, 256, 0, stream>>>(X, rows, K, per, out);
  return hipGetLastError();
}

hipError_t launch_tail_selection(const uint16_t* W, int N, int K, int k_tail, int n_alpha,
                                 const float* scale, const float* inv, double* err, int32_t* rank,
                                 int32_t* perm, float* scale_pos, float* inv_pos, hipStream_t stream) {
  column_error_kernel<<<dim3(K / 32, n_alpha), 256, 0, stream>>>(W, N, K, scale, err);
  const hipError_t e = hipMemsetAsync(rank, 0, static_cast<size_t>(n_alpha) * K * sizeof(int32_t), stream);
  if (e != hipSuccess) return e;
  error_rank_kernel<<<dim3((K + 255) / 256, n_alpha, 8), 256, 0, stream>>>(err, K, rank);
  tail_permutation_kernel<<<n_alpha, kPermThreads, 0, stream>>>(rank, scale, inv, K, k_tail, perm,
                                                                scale_pos, inv_pos);
  return hipGetLastError();
}

hipError_t launch_augment_weight(const uint16_t* W, int N, int K, int k_tail, const int32_t* perm,
                                 const float* scale_pos, bool search, uint8_t* Wq, uint8_t* Wsc,
                                 hipStream_t stream) {
  const size_t lds = static_cast<size_t>(K) * 2;   // at most 32 KiB (K <= 16384)
  if (lds > 65536) return hipErrorInvalidValue;
  const int grid = std::min(N, 4096);
  if (search)
    augment_kernel<true><<<grid, kAugThreads, lds, stream>>>(W, N, K, k_tail, perm, scale_pos, Wq, Wsc);
  else
    augment_kernel<false><<<grid, kAugThreads, lds, stream>>>(W, N, K, k_tail, perm, scale_pos, Wq, Wsc);
  return hipGetLastError();
}

}  // namespace prq
