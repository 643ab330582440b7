// Offline evaluation of the reconstruction error and the alpha search of
// Algorithm 1 (arXiv 2609.22106): for every candidate alpha, construct the
// scaling, selection, permutation and augmented weight (prepare_device.hip: the
// same bits as prq_prepare_ex), then evaluate Eq. 3 on the calibration
// activations with the device path (prq_pack_weight, prq_quant_act, prq_gemm)
// and keep the alpha whose normalized reconstruction error
// ||Y_hat - X W^T||_F / ||X W^T||_F is smallest (the first on equal errors).  The
// unquantized reference X W^T is computed once on the device from the bf16
// inputs with float32 accumulation.  Three alphas on the 9728 -> 2560 down_proj
// with 256 rows: 264 ms with the host construction, 2.96 ms now, about 2 ms of
// it the copy of W from pageable host memory.
//
// These calls are offline: they take host arrays, allocate their own device
// buffers, run on the given stream and synchronize it before returning.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "prq.h"
#include "prq_internal.h"

namespace prq {
namespace {

constexpr int kRefTile = 64;     // 64 x 64 outputs per 256-thread workgroup
constexpr int kRefK = 64;        // K chunk staged in LDS
constexpr int kRefPitch = kRefK + 8;   // elements: 16-byte rows off by 4 banks each
constexpr int kErrThreads = 256;

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Y[m, n] = sum_k X[m, k] W[n, k] (bf16 inputs, float32 accumulation) on the bf16
// 16x16x32 MFMA; four waves, 32 x 32 outputs each.  K % 32 == 0.  The next K
// chunk loads into registers while the staged one is multiplied, one barrier a
// chunk (two LDS buffers).  256 x 2560 x 9728: a scalar fma version took 1.79 ms,
// this one 0.10 (128 TFLOP/s; 160 workgroups, bound by the chunks' load latency).
// The search's NRMSE over 21 layers (16 to 256 rows, 1024 x 2560 to 2560 x 9728) is off
// from 64 bits by 1.8e-8 (root mean square; 5.1e-8 at most), by 3.3e-8 (1.2e-7) with
// the scalar sum in k order.
__global__ __launch_bounds__(256) void reference_product_kernel(const uint16_t* __restrict__ X,
                                                                const uint16_t* __restrict__ W,
                                                                int M, int N, int K,
                                                                float* __restrict__ Y) {
  __shared__ __align__(16) uint16_t xs[2][kRefTile * kRefPitch];
  __shared__ __align__(16) uint16_t ws[2][kRefTile * kRefPitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * kRefTile, n0 = blockIdx.x * kRefTile;
  const int r = tid >> 2, c = (tid & 3) * 16;   // staged row, first of 16 columns
  uint4 px[2], pw[2];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = k0 + c + 8 * i;
      const bool in = k < K;
      px[i] = in && m0 + r < M ? *reinterpret_cast<const uint4*>(X + static_cast<int64_t>(m0 + r) * K + k)
                               : make_uint4(0, 0, 0, 0);
      pw[i] = in && n0 + r < N ? *reinterpret_cast<const uint4*>(W + static_cast<int64_t>(n0 + r) * K + k)
                               : make_uint4(0, 0, 0, 0);
    }
  };
  v4f acc[2][2] = {};
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int frag = (lane & 15) * kRefPitch + (lane >> 4) * 8;   // row l % 16, K part l / 16
  fetch(0);
  for (int k0 = 0, p = 0; k0 < K; k0 += kRefK, p ^= 1) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *reinterpret_cast<uint4*>(&xs[p][r * kRefPitch + c + 8 * i]) = px[i];
      *reinterpret_cast<uint4*>(&ws[p][r * kRefPitch + c + 8 * i]) = pw[i];
    }
    if (k0 + kRefK < K) fetch(k0 + kRefK);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kRefK; h += 32) {
      v8bf a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = *reinterpret_cast<const v8bf*>(&xs[p][(wm + 16 * i) * kRefPitch + h + frag]);
        b[i] = *reinterpret_cast<const v8bf*>(&ws[p][(wn + 16 * i) * kRefPitch + h + frag]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {   // lane l holds C[4 (l / 16) + e][l % 16]
        const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + e, n = n0 + wn + 16 * j + (lane & 15);
        if (m < M && n < N) Y[static_cast<int64_t>(m) * N + n] = acc[i][j][e];
      }
}

// Per-workgroup sums of (Y - R)^2 and R^2 in double: partial[2 b], partial[2 b + 1].
__global__ __launch_bounds__(kErrThreads) void squared_error_kernel(const float* __restrict__ Y,
                                                                    const float* __restrict__ R,
                                                                    int64_t n, int64_t per_block,
                                                                    double* __restrict__ partial) {
  __shared__ double s_e[kErrThreads], s_r[kErrThreads];
  const int64_t b0 = static_cast<int64_t>(blockIdx.x) * per_block;
  const int64_t b1 = b0 + per_block < n ? b0 + per_block : n;
  double e = 0.0, r = 0.0;
  for (int64_t i = b0 + threadIdx.x; i < b1; i += kErrThreads) {
    const double d = static_cast<double>(Y[i]) - static_cast<double>(R[i]);
    e += d * d;
    r += static_cast<double>(R[i]) * static_cast<double>(R[i]);
  }
  s_e[threadIdx.x] = e;
  s_r[threadIdx.x] = r;
  __syncthreads();
  for (int s = kErrThreads / 2; s > 0; s >>= 1) {
    if (static_cast<int>(threadIdx.x) < s) {
      s_e[threadIdx.x] += s_e[threadIdx.x + s];
      s_r[threadIdx.x] += s_r[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = s_e[0];
    partial[2 * blockIdx.x + 1] = s_r[0];
  }
}

// One device allocation cut into the call's buffers, freed on scope exit.
struct DeviceArena {
  char* base = nullptr;
  size_t size = 0;
  ~DeviceArena() {
    if (base) (void)hipFree(base);
  }
  template <class T>
  size_t reserve(size_t count) {   // offset of a 256-byte aligned buffer
    const size_t at = size;
    size += (count * sizeof(T) + 255) & ~size_t{255};
    return at;
  }
  int allocate() { return hipMalloc(reinterpret_cast<void**>(&base), size + 256) == hipSuccess ? PRQ_OK : PRQ_EDEVICE; }
  template <class T>
  T* at(size_t offset) const { return reinterpret_cast<T*>(base + offset); }
};

#define PRQ_TRY(expr)              \
  do {                             \
    const int st_ = (expr);        \
    if (st_ != PRQ_OK) return st_; \
  } while (0)

// Alphas whose exports are chosen together (one read of W for their column errors):
// the scratch of a call and its launches don't grow with the number of candidates.
constexpr int32_t kAlphaBatch = 64;

int hip_status(hipError_t e) { return e == hipSuccess ? PRQ_OK : PRQ_EDEVICE; }

// Evaluation of one or more alphas on M rows X (host bf16), against the
// reference on the same rows; writes nrmse[a] for each alpha.  The export of each
// alpha is built on the device (prepare_device.hip) from one copy of W; the host
// only turns the channel maxima into scales.
int evaluate_alphas(const uint16_t* W_bf16, int32_t N, int32_t K, const uint16_t* Xcal_bf16,
                    int32_t T, const uint16_t* X_bf16, int32_t M, const double* alphas,
                    int32_t n_alpha, int32_t k_tail, int32_t scale_mode, int32_t flags,
                    double* nrmse, hipStream_t stream) {
  const int64_t K_aug = static_cast<int64_t>(K) + k_tail;
  size_t code_bytes = 0, scale_bytes = 0;
  PRQ_TRY(prq_packed_weight_bytes(1, N, static_cast<int32_t>(K_aug), &code_bytes, &scale_bytes));
  if (flags & ~PRQ_PREPARE_E8M0_SEARCH) return PRQ_EINVAL;
  for (int a = 0; a < n_alpha; ++a)
    if (!(alphas[a] >= 0.0 && alphas[a] <= 1.0)) return PRQ_EINVAL;
  if (scale_mode != PRQ_SCALE_SMOOTH && scale_mode != PRQ_SCALE_ACT_ONLY && scale_mode != PRQ_SCALE_NONE)
    return PRQ_EINVAL;
  if (K % PRQ_BLOCK || k_tail < 0 || k_tail % PRQ_BLOCK || k_tail > K) return PRQ_EALIGN;
  const size_t ws_bytes = prq_gemm_workspace_bytes(M, N, static_cast<int32_t>(K_aug));
  const int64_t outs = static_cast<int64_t>(M) * N;
  const int err_blocks = static_cast<int>(std::min<int64_t>(1024, (outs + 4095) / 4096));
  const int64_t per_block = (outs + err_blocks - 1) / err_blocks;
  const bool own_rows = X_bf16 == Xcal_bf16 && M == T;   // evaluated on the calibration rows
  const size_t nW = static_cast<size_t>(N) * K, nX = static_cast<size_t>(M) * K,
               nCal = static_cast<size_t>(T) * K;
  const int32_t batch = std::min(n_alpha, kAlphaBatch);
  const size_t nScale = static_cast<size_t>(batch) * K;

  DeviceArena mem;
  const size_t oW = mem.reserve<uint16_t>(nW), oX = mem.reserve<uint16_t>(nX),
               oCal = own_rows ? oX : mem.reserve<uint16_t>(nCal);
  const size_t oMax = mem.reserve<uint32_t>(2 * static_cast<size_t>(K));
  const size_t oScale = mem.reserve<float>(2 * nScale);   // scales, then inverse scales
  const size_t oErr = mem.reserve<double>(nScale), oRank = mem.reserve<int32_t>(nScale),
               oPerm = mem.reserve<int32_t>(nScale), oScalePos = mem.reserve<float>(nScale),
               oInvPos = mem.reserve<float>(nScale);
  const size_t oYref = mem.reserve<float>(outs), oY = mem.reserve<float>(outs);
  const size_t oWq = mem.reserve<uint8_t>(static_cast<size_t>(N) * K_aug / 2),
               oWsc = mem.reserve<uint8_t>(static_cast<size_t>(N) * K_aug / 32);
  const size_t oAq = mem.reserve<uint8_t>(static_cast<size_t>(M) * K_aug / 2),
               oAsc = mem.reserve<uint8_t>(static_cast<size_t>(M) * K_aug / 32);
  const size_t oWp = mem.reserve<uint8_t>(code_bytes), oWps = mem.reserve<uint8_t>(scale_bytes);
  const size_t oWs = mem.reserve<uint8_t>(ws_bytes);
  const size_t nPartial = static_cast<size_t>(2) * err_blocks * batch;
  const size_t oPartial = mem.reserve<double>(nPartial);
  PRQ_TRY(mem.allocate());
  uint16_t *const dW = mem.at<uint16_t>(oW), *const dX = mem.at<uint16_t>(oX),
           *const dCal = mem.at<uint16_t>(oCal);
  uint32_t* const dMax = mem.at<uint32_t>(oMax);
  float *const dScale = mem.at<float>(oScale), *const dYref = mem.at<float>(oYref),
        *const dY = mem.at<float>(oY);
  double* const dPartial = mem.at<double>(oPartial);

  // The rows first: their maxima are taken while the weight is still on its way.
  PRQ_TRY(hip_status(hipMemsetAsync(dMax, 0, 2 * static_cast<size_t>(K) * sizeof(uint32_t), stream)));
  if (ws_bytes) PRQ_TRY(hip_status(hipMemsetAsync(mem.at<uint8_t>(oWs), 0, ws_bytes, stream)));
  PRQ_TRY(hip_status(hipMemcpyAsync(dCal, Xcal_bf16, nCal * 2, hipMemcpyHostToDevice, stream)));
  PRQ_TRY(hip_status(launch_channel_maxima(dCal, T, K, dMax, stream)));
  if (!own_rows) PRQ_TRY(hip_status(hipMemcpyAsync(dX, X_bf16, nX * 2, hipMemcpyHostToDevice, stream)));
  PRQ_TRY(hip_status(hipMemcpyAsync(dW, W_bf16, nW * 2, hipMemcpyHostToDevice, stream)));
  PRQ_TRY(hip_status(launch_channel_maxima(dW, N, K, dMax + K, stream)));
  std::vector<uint32_t> maxima(2 * static_cast<size_t>(K));
  PRQ_TRY(hip_status(hipMemcpyAsync(maxima.data(), dMax, maxima.size() * sizeof(uint32_t),
                                    hipMemcpyDeviceToHost, stream)));
  PRQ_TRY(hip_status(hipStreamSynchronize(stream)));
  // The reference product runs while the host takes the scales.
  reference_product_kernel<<<dim3((N + kRefTile - 1) / kRefTile, (M + kRefTile - 1) / kRefTile), 256, 0,
                             stream>>>(dX, dW, M, N, K, dYref);
  PRQ_TRY(hip_status(hipGetLastError()));
  std::vector<float> scales(2 * nScale);   // as dScale: scales, then inverse scales
  std::vector<double> partial(nPartial);
  uint8_t *const dWq = mem.at<uint8_t>(oWq), *const dWsc = mem.at<uint8_t>(oWsc),
          *const dAq = mem.at<uint8_t>(oAq), *const dAsc = mem.at<uint8_t>(oAsc),
          *const dWp = mem.at<uint8_t>(oWp), *const dWps = mem.at<uint8_t>(oWps);
  for (int32_t a0 = 0; a0 < n_alpha; a0 += batch) {
    const int32_t n = std::min(batch, n_alpha - a0);
    for (int32_t a = 0; a < n; ++a) {
      const size_t at = static_cast<size_t>(a) * K;
      channel_scales(maxima.data(), maxima.data() + K, K, alphas[a0 + a], scale_mode, scales.data() + at,
                     scales.data() + nScale + at);
    }
    PRQ_TRY(hip_status(hipMemcpyAsync(dScale, scales.data(), scales.size() * sizeof(float),
                                      hipMemcpyHostToDevice, stream)));
    PRQ_TRY(hip_status(launch_tail_selection(dW, N, K, k_tail, n, dScale, dScale + nScale,
                                             mem.at<double>(oErr), mem.at<int32_t>(oRank),
                                             mem.at<int32_t>(oPerm), mem.at<float>(oScalePos),
                                             mem.at<float>(oInvPos), stream)));
    for (int32_t a = 0; a < n; ++a) {
      const size_t at = static_cast<size_t>(a) * K;
      const int32_t* perm = mem.at<int32_t>(oPerm) + at;
      PRQ_TRY(hip_status(launch_augment_weight(dW, N, K, k_tail, perm, mem.at<float>(oScalePos) + at,
                                               (flags & PRQ_PREPARE_E8M0_SEARCH) != 0, dWq, dWsc, stream)));
      PRQ_TRY(prq_pack_weight(dWq, dWsc, 1, N, static_cast<int32_t>(K_aug), dWp, dWps, stream));
      PRQ_TRY(prq_quant_act(dX, K, M, K, k_tail, mem.at<float>(oInvPos) + at, perm, nullptr, 1, dAq, dAsc, stream));
      PRQ_TRY(prq_gemm(dAq, dAsc, M, dWp, dWps, N, static_cast<int32_t>(K_aug), dY, mem.at<uint8_t>(oWs),
                       ws_bytes, stream));
      squared_error_kernel<<<err_blocks, kErrThreads, 0, stream>>>(
          dY, dYref, outs, per_block, dPartial + static_cast<size_t>(2) * err_blocks * a);
      PRQ_TRY(hip_status(hipGetLastError()));
    }
    PRQ_TRY(hip_status(hipMemcpyAsync(partial.data(), dPartial,
                                      static_cast<size_t>(2) * err_blocks * n * sizeof(double),
                                      hipMemcpyDeviceToHost, stream)));
    PRQ_TRY(hip_status(hipStreamSynchronize(stream)));   // also: the host's scales are free again
    for (int32_t a = 0; a < n; ++a) {
      double e = 0.0, r = 0.0;
      for (int b = 0; b < err_blocks; ++b) {   // fixed order
        e += partial[2 * (static_cast<size_t>(err_blocks) * a + b)];
        r += partial[2 * (static_cast<size_t>(err_blocks) * a + b) + 1];
      }
      nrmse[a0 + a] = r > 0.0 ? std::sqrt(e / r) : (e > 0.0 ? INFINITY : 0.0);
    }
  }
  return PRQ_OK;
}

}  // namespace
}  // namespace prq

extern "C" {

int prq_evaluate_nrmse(const uint16_t* W_bf16, int32_t N, int32_t K, const uint16_t* Xcal_bf16,
                       int32_t T, const uint16_t* X_bf16, int32_t M, double alpha, int32_t k_tail,
                       int32_t scale_mode, int32_t flags, double* nrmse, hipStream_t stream) {
  if (!W_bf16 || !Xcal_bf16 || !X_bf16 || !nrmse || N <= 0 || K <= 0 || T <= 0 || M <= 0)
    return PRQ_EINVAL;
  if (N % 16) return PRQ_EALIGN;
  if (K > 16384) return PRQ_EUNSUPPORTED;
  return prq::evaluate_alphas(W_bf16, N, K, Xcal_bf16, T, X_bf16, M, &alpha, 1, k_tail, scale_mode,
                              flags, nrmse, stream);
}

int prq_search_alpha(const uint16_t* W_bf16, int32_t N, int32_t K, const uint16_t* Xcal_bf16,
                     int32_t T, const double* alphas, int32_t n_alpha, int32_t k_tail,
                     int32_t scale_mode, int32_t flags, double* nrmse, int32_t* best,
                     hipStream_t stream) {
  if (!W_bf16 || !Xcal_bf16 || !alphas || !nrmse || !best || N <= 0 || K <= 0 || T <= 0 ||
      n_alpha <= 0)
    return PRQ_EINVAL;
  for (int a = 0; a < n_alpha; ++a)
    if (!(alphas[a] >= 0.0 && alphas[a] <= 1.0)) return PRQ_EINVAL;
  if (N % 16) return PRQ_EALIGN;
  if (K > 16384) return PRQ_EUNSUPPORTED;
  const int st = prq::evaluate_alphas(W_bf16, N, K, Xcal_bf16, T, Xcal_bf16, T, alphas, n_alpha,
                                      k_tail, scale_mode, flags, nrmse, stream);
  if (st != PRQ_OK) return st;
  int b = 0;
  for (int a = 1; a < n_alpha; ++a)
    if (nrmse[a] < nrmse[b]) b = a;
  *best = b;
  return PRQ_OK;
}

}  // extern "C"
