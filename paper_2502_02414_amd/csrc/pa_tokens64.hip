// Token attention forward in double precision (gfx950), used for fp32
// storage.  Attention among the M <= 64 states (Eq. 2) is a tiny product,
// but its result S' feeds the slice backward through the differences
// s'_j - s'_k of nearly equal tokens: an fp32 rounding error of 1e-7 in S'
// moves dA by about 1e-5 at the synthetic workloads' shapes.  So for fp32
// storage Q, K, V, the attention and S' are formed in double and S' is
// rounded once.
//
//   k_mm64    batches of small products out = sum_t op(A_t) op(B_t) + b
//             (operands fp32 or fp64 with arbitrary strides): one block per
//             16 x 16 output tile, K split over its four waves
//   k_core64  P = softmax(Q_h K_h^T / sqrt(D)), O_h = P V_h: one wave per head
//             and 16 query rows, no LDS
// Both run on v_mfma_f64_16x16x4_f64 and are bound by latency (a few hundred
// kilobytes and a few MFLOP): every wave reads its operands straight from
// global memory in MFMA layout, all of a chunk's loads at once, so a kernel
// is about one load round, a short MFMA chain and the stores, on as many CUs
// as there are tiles.  (Before: 32 x 32 tiles through LDS chunk by chunk, and
// one block per head; M = 64, C = 128, H = 8: 20 + 21 us; now 7 + 8 us.)
#include "pa_device.hpp"
#include "pa_internal.h"

namespace pa {

namespace {

constexpr int kT = 16;           // output tile edge
constexpr int kMMWaves = 4;      // K split over the block's waves
constexpr int kMMThreads = 64 * kMMWaves;
constexpr int kSteps = 16;       // K4 steps of a wave per chunk (64 of K)

// Element (i, k) of an operand with rows i < ni and k < K; 0 outside.
template <typename S>
__device__ __forceinline__ double opnd_ld(const void* p, int64_t off, bool in) {
  const double v = (double)static_cast<const S*>(p)[in ? off : 0];
  return in ? v : 0.0;
}
// A wave's operand of the K chunk at k0: lane (r, g) holds index m of step q,
// k = k0 + 4 q + g (the same k on both operands of the product; a lane row's
// four groups read 16 or 32 contiguous bytes of a row).
__device__ __forceinline__ void opnd_chunk(double (&v)[kSteps], const Opnd64& o, int64_t sm,
                                           int64_t sk, int m, int mn, int k0, int K) {
  const int g = lane_id() >> 4;
  if (!o.p) {
#pragma unroll
    for (int q = 0; q < kSteps; ++q) v[q] = m < mn && k0 + 4 * q + g < K ? 1.0 : 0.0;
  } else if (o.dbl) {
#pragma unroll
    for (int q = 0; q < kSteps; ++q) {
      const int k = k0 + 4 * q + g;
      v[q] = opnd_ld<double>(o.p, m * sm + k * sk, m < mn && k < K);
    }
  } else {
#pragma unroll
    for (int q = 0; q < kSteps; ++q) {
      const int k = k0 + 4 * q + g;
      v[q] = opnd_ld<float>(o.p, m * sm + k * sk, m < mn && k < K);
    }
  }
}

// One 16 x 16 tile (tile index blockIdx.x) of product q.  Wave w takes the
// chunks k0 = 64 w, 64 (w + 4), .. of every term; the waves' sums are added in
// wave order.
__device__ __forceinline__ void mm64_tile(const MM64& q) {
  __shared__ f64x4 part[kMMWaves - 1][64];
  const int tc = (q.cols + kT - 1) / kT;
  const int tiles = tc * ((q.rows + kT - 1) / kT);
  if ((int)blockIdx.x >= tiles) return;
  const int i0 = (blockIdx.x / tc) * kT, j0 = (blockIdx.x % tc) * kT;
  const int lane = lane_id(), r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f64x4 acc{0.0, 0.0, 0.0, 0.0};
  // terms by constant index (no run-time indexing of the argument struct)
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t >= q.nt) break;
    const Opnd64 A = q.A[t], B = q.B[t];
    const int K = q.K[t];
    for (int k0 = 64 * wave; k0 < K; k0 += 64 * kMMWaves) {
      double a[kSteps], b[kSteps];
      opnd_chunk(a, A, A.rs, A.cs, i0 + r, q.rows, k0, K);
      opnd_chunk(b, B, B.cs, B.rs, j0 + r, q.cols, k0, K);
#pragma unroll
      for (int s = 0; s < kSteps; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
    }
  }
  if (wave > 0) part[wave - 1][lane] = acc;
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int w = 0; w + 1 < kMMWaves; ++w) acc += part[w][lane];
  const int j = j0 + r;
  if (j >= q.cols) return;
  const double bias = q.bias ? (double)q.bias[j] : 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {  // (the fp64 MFMA's output row 4 e + g)
    const int i = i0 + 4 * e + g;
    if (i >= q.rows) continue;
    const double v = acc[e] + bias;
    const int64_t o = (int64_t)i * q.ld + j;
    if (q.out_type == kOutF64)
      static_cast<double*>(q.out)[o] = v;
    else if (q.out_type == kOutBF16)
      static_cast<bf16*>(q.out)[o] = (bf16)(float)v;
    else
      static_cast<float*>(q.out)[o] = (float)v;
  }
}

// The product of a batch is chosen with constant indices (a run-time index
// into the by-value argument array would copy the arguments to scratch).
__global__ void __launch_bounds__(kMMThreads) k_mm64(MM64Batch b) {
  switch (blockIdx.y) {
#define PA_MM64_CASE(I) \
    case I:             \
      if (I < b.n) mm64_tile(b.p[I]); \
      break;
    PA_MM64_CASE(0) PA_MM64_CASE(1) PA_MM64_CASE(2) PA_MM64_CASE(3)
    PA_MM64_CASE(4) PA_MM64_CASE(5) PA_MM64_CASE(6)
#undef PA_MM64_CASE
    default:
      break;
  }
}

// Head blockIdx.x, query rows 16 blockIdx.y ..: the scores are formed
// transposed (K_h Q_h^T), so that lane (r, g) holds query r's scores of the
// keys 16 t + 4 e + g: the softmax reduces in the lane and over the four lane
// groups, and the probabilities are already the B operand of O_h^T = V_h^T
// P^T (step (t, e): key 16 t + 4 e + g).
template <int MT, typename TO>
__global__ void __launch_bounds__(64) k_core64(const double* Q, const double* K, const double* V,
                                               TO* O, int M, int C, int H) {
  const int D = C / H, off = blockIdx.x * D;
  const int lane = lane_id(), r = lane & 15, g = lane >> 4;
  const int qi = 16 * blockIdx.y + r;
  const double* qp = Q + (int64_t)(qi < M ? qi : M - 1) * C + off;
  const double* kp[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int j = 16 * t + r;
    kp[t] = K + (int64_t)(j < M ? j : M - 1) * C + off;
  }
  f64x4 p[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) p[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int d0 = 0; d0 < D; d0 += 4) {
    const int d = d0 + g;
    const bool in = d < D;
    const double qv = in ? qp[in ? d : 0] : 0.0;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const double kv = in ? kp[t][in ? d : 0] : 0.0;
      p[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(kv, qv, p[t], 0, 0, 0);
    }
  }
  const double scale = 1.0 / sqrt((double)D);
  double mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[t][e] = 16 * t + 4 * e + g < M ? p[t][e] * scale : -INFINITY;
      mx = fmax(mx, p[t][e]);
    }
  mx = fmax(mx, __shfl_xor(mx, 16));
  mx = fmax(mx, __shfl_xor(mx, 32));
  double sum = 0.0;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[t][e] = exp(p[t][e] - mx);
      sum += p[t][e];
    }
  sum += __shfl_xor(sum, 16);
  sum += __shfl_xor(sum, 32);
  const double inv = 1.0 / sum;
#pragma unroll
  for (int t = 0; t < MT; ++t) p[t] *= inv;
  for (int d0 = 0; d0 < D; d0 += 16) {
    const int d = d0 + r < D ? d0 + r : D - 1;  // (rows d >= D are not stored)
    f64x4 o{0.0, 0.0, 0.0, 0.0};
    double v[MT][4];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 16 * t + 4 * e + g;
        v[t][e] = V[(int64_t)(j < M ? j : M - 1) * C + off + d];
      }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 16 * t + 4 * e + g;
        o = __builtin_amdgcn_mfma_f64_16x16x4f64(j < M ? v[t][e] : 0.0, p[t][e], o, 0, 0, 0);
      }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (d0 + 4 * e + g < D && qi < M) O[(int64_t)qi * C + off + d0 + 4 * e + g] = (TO)o[e];
  }
}

bool core64_ok(int M, int C, int H) { return M >= 1 && M <= 64 && H >= 1 && C % H == 0; }

}  // namespace

hipError_t launch_mm64(const MM64Batch& b, hipStream_t st) {
  if (b.n < 1 || b.n > kMM64Max) return hipErrorInvalidValue;
  int tiles = 0;
  for (int i = 0; i < b.n; ++i) {
    const MM64& q = b.p[i];
    if (q.rows < 1 || q.cols < 1 || q.nt < 0 || q.nt > 3 || !q.out || q.ld < q.cols)
      return hipErrorInvalidValue;
    for (int t = 0; t < q.nt; ++t)
      if (q.K[t] < 1) return hipErrorInvalidValue;
    const int n = ((q.rows + kT - 1) / kT) * ((q.cols + kT - 1) / kT);
    tiles = n > tiles ? n : tiles;
  }
  hipLaunchKernelGGL(k_mm64, dim3(tiles, b.n), dim3(kMMThreads), 0, st, b);
  return hipGetLastError();
}

hipError_t launch_core64(const double* Q, const double* K, const double* V, void* O, bool O_dbl,
                         int M, int C, int H, hipStream_t st) {
  if (!Q || !K || !V || !O || !core64_ok(M, C, H)) return hipErrorInvalidValue;
  const int MT = (M + 15) / 16;
#define PA_CORE64(T, TO)                                                               \
  hipLaunchKernelGGL((k_core64<T, TO>), dim3(H, MT), dim3(64), 0, st, Q, K, V,         \
                     static_cast<TO*>(O), M, C, H)
  switch (MT * 2 + (O_dbl ? 1 : 0)) {
    case 2: PA_CORE64(1, float); break;
    case 3: PA_CORE64(1, double); break;
    case 4: PA_CORE64(2, float); break;
    case 5: PA_CORE64(2, double); break;
    case 6: PA_CORE64(3, float); break;
    case 7: PA_CORE64(3, double); break;
    case 8: PA_CORE64(4, float); break;
    case 9: PA_CORE64(4, double); break;
    default: return hipErrorInvalidValue;
  }
#undef PA_CORE64
  return hipGetLastError();
}

}  // namespace pa
