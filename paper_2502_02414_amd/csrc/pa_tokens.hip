// Token side of the layer (gfx950): attention among the M <= 64 physical
// states (Eq. 2) and its backward, in fp32 (the fp32-storage forward runs in
// double, pa_tokens64.hip).  These products are tiny (M x C by C x C at most)
// and bound by latency: a kernel is one round of loads, a short MFMA chain
// (v_mfma_f32_16x16x4_f32) and its stores, and the work is spread over as many
// CUs as it has 16 x 16 tiles (k_core_bwd: over one block per head).
//   k_proj         out_p = In_p op(W_p) + b_p (op = W or W^T): a block per tile
//   k_core         per head h (channels [hD, hD + D)) and 16 query rows, one
//                  wave: P_h = softmax(Q_h K_h^T / sqrt(D)), O_h = P_h V_h
//   k_core_bwd     per head: the same P_h, then dV_h, dQ_h, dK_h (and O_h)
//   k_token_grads  dS = sum_p dX_p W_p^T, dW_p = A_p^T B_p, db_p = 1^T B_p,
//                  every output tile of every product in one launch
// (One block per head for projections and core together, staged through LDS,
// took at M = 32, C = 256, H = 8 13.0 us forward and 15.4 us backward, and at
// M = 64, C = 256, H = 8 22.9 and 26.9 us; the projections and the core apart
// take 5.6 + 5.2 and 5.6 + 7.8 us, and 5.7 + 7.7 and 5.7 + 14.0 us, and serve
// every head width.)
#include "pa_device.hpp"
#include "pa_internal.h"
#include "pa_layout.h"

namespace pa {

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// k_proj: one 16 x 16 tile of product blockIdx.z per block.  The K = Cin steps
// of 4 (lane group g: k = 4 s + g, so that a lane row's four groups read 16
// contiguous bytes) split over the four waves, their sums added in wave order.
// ---------------------------------------------------------------------------
constexpr int kProjSteps = 16;  // K4 steps per wave (Cin <= 256)

__global__ void __launch_bounds__(256) k_proj(Proj q) {
  __shared__ f32x4 part[3][64];
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p = blockIdx.z, M = q.M, Cin = q.Cin, Cout = q.Cout;
  // (by constant index: a run-time index would copy the arguments to scratch)
  auto pick = [p](auto const (&v)[kProjMax]) {
    return p == 0 ? v[0] : p == 1 ? v[1] : p == 2 ? v[2] : p == 3 ? v[3] : v[4];
  };
  const float* in = pick(q.in);
  const float* W = pick(q.W);
  const float* b = pick(q.b);
  const bool tr = pick(q.transW);
  const int i0 = 16 * blockIdx.y, j0 = 16 * blockIdx.x;
  const int row = i0 + r < M ? i0 + r : M - 1, col = j0 + r;  // (Cout a multiple of 16)
  const int n = Cin / 16, k0 = 4 * n * wave + g;              // steps per wave, its first k
  const int64_t wk = tr ? 1 : Cout;
  const float* ip = in + (int64_t)row * Cin + k0;
  const float* wp = W + (tr ? (int64_t)col * Cin : col) + k0 * wk;
  float x[kProjSteps], w[kProjSteps], c[kProjSteps];
  const bool center = pick(q.center);
#pragma unroll
  for (int s = 0; s < kProjSteps; ++s) {
    if (s < n) {
      x[s] = ip[4 * s];
      w[s] = wp[4 * s * wk];
      c[s] = center ? in[k0 + 4 * s] : 0.f;
    }
  }
#pragma unroll
  for (int s = 0; s < kProjSteps; ++s)
    if (s < n) x[s] -= c[s];
  f32x4 acc = zero4();
#pragma unroll
  for (int s = 0; s < kProjSteps; ++s)
    if (s < n) acc = mfma4(x[s], w[s], acc);
  if (wave > 0) part[wave - 1][lane] = acc;
  __syncthreads();
  if (wave > 0) return;
  acc = ((acc + part[0][lane]) + part[1][lane]) + part[2][lane];
  const float bj = b ? b[col] : 0.f;
  float* out = pick(q.out);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int orow = i0 + 4 * g + i;
    if (orow < M) out[(int64_t)orow * Cout + col] = acc[i] + bj;
  }
}

hipError_t launch_proj(const Proj& q, hipStream_t st) {
  // (Cin <= 256: kProjSteps K4 steps per wave)
  if (q.n < 1 || q.n > kProjMax || q.M < 1 || q.M > 64 || q.Cin < 16 || q.Cin % 16 || q.Cin > 256 ||
      q.Cout < 16 || q.Cout % 16)
    return hipErrorInvalidValue;
  for (int p = 0; p < q.n; ++p)
    if (!q.in[p] || !q.W[p] || !q.out[p]) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_proj, dim3(q.Cout / 16, (q.M + 15) / 16, q.n), dim3(256), 0, st, q);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Attention cores.  Scores are formed transposed, X Y^T with the keys as rows:
// lane (r, g) of tile t, element e, holds (query 16 qt + r, key 16 t + 4 g + e),
// so a query's softmax reduces in the lane and over the four lane groups, and
// the probabilities are already the B operand of (P V)^T = V^T P^T (step (t,
// e): key 16 t + 4 g + e).  Rows past M re-read row M - 1; their results are
// masked (keys) or not stored (queries).
// ---------------------------------------------------------------------------
// A head's matrix: element (row, d), in global memory or staged in LDS.
struct HeadMat {
  const float* p;
  int ld;
  __device__ __forceinline__ float operator()(int row, int d) const { return p[row * ld + d]; }
};

template <int MT>
__device__ __forceinline__ void core_scores(const HeadMat& X, const HeadMat& Y, int qt, int M,
                                            int D, f32x4 (&p)[MT]) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int qi = 16 * qt + r < M ? 16 * qt + r : M - 1;
  int yj[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    yj[t] = 16 * t + r < M ? 16 * t + r : M - 1;
    p[t] = zero4();
  }
  for (int d0 = 0; d0 < D; d0 += 32) {
    float x[8], y[MT][8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int d = d0 + 4 * s + g;
      const bool in = d < D;
      const int dd = in ? d : 0;
      x[s] = X(qi, dd);
      if (!in) x[s] = 0.f;
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        y[t][s] = Y(yj[t], dd);
        if (!in) y[t][s] = 0.f;
      }
    }
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (d0 + 4 * s < D)
#pragma unroll
        for (int t = 0; t < MT; ++t) p[t] = mfma4(y[t][s], x[s], p[t]);
  }
}

template <int MT>
__device__ __forceinline__ void core_softmax(f32x4 (&p)[MT], int M, float scale) {
  const int g = (threadIdx.x & 63) >> 4;
  float mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[t][e] = 16 * t + 4 * g + e < M ? p[t][e] * scale : -INFINITY;
      mx = fmaxf(mx, p[t][e]);
    }
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  float sum = 0.f;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[t][e] = expf(p[t][e] - mx);
      sum += p[t][e];
    }
  sum += __shfl_xor(sum, 16);
  sum += __shfl_xor(sum, 32);
  const float inv = 1.0f / sum;
#pragma unroll
  for (int t = 0; t < MT; ++t) p[t] *= inv;
}

// Channels d0 + r of the keys' rows, as the A operand of core_times.
template <int MT>
__device__ __forceinline__ void core_rows(float (&z)[MT][4], const HeadMat& Z, int d0, int M,
                                          int D) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int d = d0 + r < D ? d0 + r : D - 1;  // (channels past D are not stored)
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = 16 * t + 4 * g + e;
      z[t][e] = Z(j < M ? j : M - 1, d);
      if (j >= M) z[t][e] = 0.f;
    }
}
// dst (row stride C) rows 16 qt .., channels d0 .. d0 + 15 of scale A Z (A in
// the transposed layout above), in two chains of MFMAs.
template <int MT>
__device__ __forceinline__ void core_times(const f32x4 (&A)[MT], const float (&z)[MT][4],
                                           float* dst, int qt, int d0, int M, int D, int C,
                                           float scale) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int qi = 16 * qt + r;
  f32x4 o[2] = {zero4(), zero4()};
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e & 1] = mfma4(z[t][e], A[t][e], o[e & 1]);
  o[0] += o[1];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int od = d0 + 4 * g + e;
    if (od < D && qi < M) dst[(int64_t)qi * C + od] = scale * o[0][e];
  }
}

template <int MT>
__global__ void __launch_bounds__(64) k_core(CoreArgs a) {
  const int M = a.M, C = a.C, D = C / a.H, off = blockIdx.x * D, qt = blockIdx.y;
  const HeadMat V{a.V + off, C};
  float z[MT][4];
  core_rows<MT>(z, V, 0, M, D);  // (requested with Q and K)
  f32x4 p[MT];
  core_scores<MT>({a.Q + off, C}, {a.K + off, C}, qt, M, D, p);
  core_softmax<MT>(p, M, 1.0f / sqrtf((float)D));
  for (int d0 = 0; d0 < D; d0 += 16) {
    if (d0 > 0) core_rows<MT>(z, V, d0, M, D);
    core_times<MT>(p, z, a.O + off, qt, d0, M, D, C, 1.f);
  }
}

// One block of eight waves per head.  The head's Q, K, V, dO are staged in LDS
// in one round of loads (STAGE; heads too wide for it read global memory).
// Waves qt < MT: P, dP = dO V^T and dE = P o (dP - rowsum(dP o P)) of 16 query
// rows, to LDS; then all waves form the tiles of dQ = scale dE K, dK = scale
// dE^T Q, dV = P^T dO and, where wanted, O = P Vf.
constexpr int kCoreBwdWaves = 8;
__host__ __device__ constexpr int core_ld(int D) { return D + 4; }  // staged row stride

template <int MT, bool STAGE>
__global__ void __launch_bounds__(64 * kCoreBwdWaves) k_core_bwd(CoreArgs a) {
  constexpr int M16 = 16 * MT, PS = M16 + 4, TH = 64 * kCoreBwdWaves;
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float* ps = sm;               // P  [query][key]
  float* es = sm + M16 * PS;    // dE [query][key]
  float* st = sm + 2 * M16 * PS;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int M = a.M, C = a.C, D = C / a.H, off = blockIdx.x * D, NT = (D + 15) / 16;
  const float scale = 1.0f / sqrtf((float)D);
  const int ld = STAGE ? core_ld(D) : C;
  const HeadMat Q{STAGE ? st : a.Q + off, ld}, K{STAGE ? st + M * ld : a.K + off, ld},
      V{STAGE ? st + 2 * M * ld : a.V + off, ld}, dO{STAGE ? st + 3 * M * ld : a.dO + off, ld};
  if constexpr (STAGE) {
    const int n = M * D;
    for (int b = threadIdx.x; b < n; b += 4 * TH) {
      float v[4][4];
      int o[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = b + u * TH < n ? b + u * TH : n - 1;
        const int row = e / D, d = e - row * D, x = row * C + off + d;
        o[u] = row * ld + d;
        v[0][u] = a.Q[x];
        v[1][u] = a.K[x];
        v[2][u] = a.V[x];
        v[3][u] = a.dO[x];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)  // (past the end: the last element again)
#pragma unroll
        for (int m = 0; m < 4; ++m) st[m * M * ld + o[u]] = v[m][u];
    }
    __syncthreads();
  }
  if (wave < MT) {
    f32x4 p[MT], e[MT];
    core_scores<MT>(Q, K, wave, M, D, p);
    core_scores<MT>(dO, V, wave, M, D, e);
    core_softmax<MT>(p, M, scale);
    float rs = 0.f;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (16 * t + 4 * g + i >= M) e[t][i] = 0.f;  // (P is 0 there)
        rs += e[t][i] * p[t][i];
      }
    rs += __shfl_xor(rs, 16);
    rs += __shfl_xor(rs, 32);
    const bool qv = 16 * wave + r < M;  // rows past M contribute nothing below
#pragma unroll
    for (int t = 0; t < MT; ++t) {
#pragma unroll
      for (int i = 0; i < 4; ++i) e[t][i] = p[t][i] * (e[t][i] - rs);
      const int o = (16 * wave + r) * PS + 16 * t + 4 * g;
      *reinterpret_cast<f32x4*>(ps + o) = qv ? p[t] : zero4();
      *reinterpret_cast<f32x4*>(es + o) = qv ? e[t] : zero4();
    }
  }
  __syncthreads();
  // tile (which, row tile ct, channel tile dt); the contraction runs over the
  // keys (dQ, O: A^T = the row's probabilities) or over the queries (dK, dV)
  const int tiles = (a.O ? 4 : 3) * MT * NT;
  for (int t = wave; t < tiles; t += kCoreBwdWaves) {
    const int which = t / (MT * NT), rem = t - which * MT * NT;
    const int ct = rem / NT, dt = rem - ct * NT;
    const float* Am = which == 0 || which == 1 ? es : ps;
    const bool keys = which == 0 || which == 3;  // contraction over the keys
    const HeadMat Vf{a.Vf + off, C};  // (global memory: read for O only)
    const HeadMat Bm = which == 0 ? K : which == 1 ? Q : which == 2 ? dO : Vf;
    const int d = 16 * dt + r < D ? 16 * dt + r : D - 1;
    float b[4 * MT], x[4 * MT];
#pragma unroll
    for (int s = 0; s < 4 * MT; ++s) {
      const int q = 4 * s + g;
      b[s] = Bm(q < M ? q : M - 1, d);
      if (q >= M) b[s] = 0.f;
      x[s] = keys ? Am[(16 * ct + r) * PS + q] : Am[q * PS + 16 * ct + r];
    }
    f32x4 o[2] = {zero4(), zero4()};
#pragma unroll
    for (int s = 0; s < 4 * MT; ++s) o[s & 1] = mfma4(x[s], b[s], o[s & 1]);
    o[0] += o[1];
    float* dst = (which == 0 ? a.dQ : which == 1 ? a.dK : which == 2 ? a.dV : a.O) + off;
    const float sc = which < 2 ? scale : 1.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * ct + 4 * g + i;
      if (row < M && 16 * dt + r < D) dst[(int64_t)row * C + 16 * dt + r] = sc * o[0][i];
    }
  }
}

hipError_t launch_core(const CoreArgs& a, bool bwd, hipStream_t st) {
  if (!a.Q || !a.K || !a.V || a.M < 1 || a.M > 64 || a.H < 1 || a.C < 1 || a.C % a.H)
    return hipErrorInvalidValue;
  if (bwd ? (!a.dO || !a.dQ || !a.dK || !a.dV) : !a.O) return hipErrorInvalidValue;
  const int MT = (a.M + 15) / 16, D = a.C / a.H;
  // LDS of the backward: P, dE, and the head's four matrices where they fit
  const size_t core = (size_t)2 * 16 * MT * (16 * MT + 4) * sizeof(float);
  const size_t all = core + (size_t)4 * a.M * core_ld(D) * sizeof(float);
  const bool stage = all <= (size_t)kLdsBytes;
  if (bwd && a.O && !a.Vf) return hipErrorInvalidValue;
#define PA_CORE(T)                                                                             \
  case T:                                                                                      \
    if (!bwd)                                                                                  \
      hipLaunchKernelGGL(k_core<T>, dim3(a.H, T), dim3(64), 0, st, a);                         \
    else if (stage)                                                                            \
      hipLaunchKernelGGL((k_core_bwd<T, true>), dim3(a.H), dim3(64 * kCoreBwdWaves), all, st, a);   \
    else                                                                                       \
      hipLaunchKernelGGL((k_core_bwd<T, false>), dim3(a.H), dim3(64 * kCoreBwdWaves), core, st, a); \
    break;
  switch (MT) { PA_CORE(1) PA_CORE(2) PA_CORE(3) PA_CORE(4) }
#undef PA_CORE
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_token_grads: the parameter-side products of the token backward, all in
// one launch (256 threads per block, fp32 MFMA):
//   blocks [0, nSB): dS tiles (16 x 16) = sum_p X_p W_p^T, K = nS C split
//     over the 4 waves (each lane loads its operands as float4 runs of 4
//     consecutive k straight from global), the 4 partial tiles added in
//     wave order;
//   the rest: one 16 x 16 tile of dW_p = A_p^T B_p per wave (K = M), and for
//     the tiles of row 0 the column sums db_p of B_p.
// ---------------------------------------------------------------------------
constexpr int kGradQ = 12;  // dS K steps (of 16) per wave, at most (C <= 256, nS <= 3)

__global__ void __launch_bounds__(256) k_token_grads(GradArgs a) {
  __shared__ f32x4 red[4][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int M = a.M, C = a.C, CT = C / 16;
  const int nSB = a.nS ? ((M + 15) / 16) * CT : 0;
  if ((int)blockIdx.x < nSB) {
    const int rt = blockIdx.x / CT, ct = blockIdx.x - rt * CT;
    const int Q = a.nS * CT, q0 = wave * Q / 4, nq = (wave + 1) * Q / 4 - q0;
    const int row = 16 * rt + r, rr = row < M ? row : M - 1;
    f32x4 xa[kGradQ], wb[kGradQ];
#pragma unroll
    for (int i = 0; i < kGradQ; ++i) {
      if (i < nq) {
        const int q = q0 + i, p = q / CT, k = 16 * (q - p * CT) + 4 * g;
        const float* X = p == 0 ? a.X[0] : p == 1 ? a.X[1] : a.X[2];
        const float* W = p == 0 ? a.W[0] : p == 1 ? a.W[1] : a.W[2];
        xa[i] = *reinterpret_cast<const f32x4*>(X + (int64_t)rr * C + k);
        wb[i] = *reinterpret_cast<const f32x4*>(W + (int64_t)(16 * ct + r) * C + k);
      }
    }
    f32x4 acc = zero4();
#pragma unroll
    for (int i = 0; i < kGradQ; ++i) {
      if (i < nq) {
        const f32x4 x = row < M ? xa[i] : zero4();
        acc = mfma4(x[0], wb[i][0], acc);
        acc = mfma4(x[1], wb[i][1], acc);
        acc = mfma4(x[2], wb[i][2], acc);
        acc = mfma4(x[3], wb[i][3], acc);
      }
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0) {
      const f32x4 t = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int orow = 16 * rt + 4 * g + i;
        if (orow < M) a.dS[(int64_t)orow * C + 16 * ct + r] = t[i];
      }
    }
    return;
  }
  // dW / db tiles: wave -> (product p, row tile ct of channels of A, column tile jt)
  const int gw = ((int)blockIdx.x - nSB) * 4 + wave;
  const int p = gw / (CT * CT), tile = gw - p * CT * CT;
  if (p >= a.nO) return;
  const int ct = tile / CT, jt = tile - ct * CT;
  auto pick = [p](auto const (&v)[4]) { return p == 0 ? v[0] : p == 1 ? v[1] : p == 2 ? v[2] : v[3]; };
  float* dW = pick(a.dW);
  float* db = pick(a.db);
  const bool wantW = dW != nullptr, wantB = db != nullptr && ct == 0;
  if (!wantW && !wantB) return;
  const float* A = pick(a.A);
  const float* Bm = pick(a.B);
  const float a0 = pick(a.center) ? A[16 * ct + r] : 0.f;
  const int S4 = (M + 3) / 4;  // K steps: k = 4 s + g
  float av[16], bv[16];
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    if (s < S4) {
      const int k = 4 * s + g, kk = k < M ? k : M - 1;
      av[s] = A[(int64_t)kk * C + 16 * ct + r];
      bv[s] = Bm[(int64_t)kk * C + 16 * jt + r];
    }
  }
  f32x4 acc = zero4();
  float cs = 0.f;
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    if (s < S4) {
      const bool v = 4 * s + g < M;
      const float x = v ? av[s] - a0 : 0.f, y = v ? bv[s] : 0.f;
      acc = mfma4(x, y, acc);
      cs += y;
    }
  }
  if (wantW) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      dW[(int64_t)(16 * ct + 4 * g + i) * C + 16 * jt + r] = acc[i];
  }
  if (wantB) {
    cs += __shfl_xor(cs, 16);
    cs += __shfl_xor(cs, 32);
    if (g == 0) db[16 * jt + r] = cs;
  }
}

hipError_t launch_token_grads(const GradArgs& a, hipStream_t st) {
  if (a.M < 1 || a.M > 64 || a.C < 16 || a.C % 16 || a.C > 256 || a.nS < 0 || a.nS > 3 ||
      a.nO < 0 || a.nO > 4)
    return hipErrorInvalidValue;
  if (a.nS && !a.dS) return hipErrorInvalidValue;
  for (int p = 0; p < a.nS; ++p)
    if (!a.X[p] || !a.W[p]) return hipErrorInvalidValue;
  for (int p = 0; p < a.nO; ++p)
    if (!a.A[p] || !a.B[p]) return hipErrorInvalidValue;
  const int CT = a.C / 16;
  const int nSB = a.nS ? ((a.M + 15) / 16) * CT : 0;
  const int nOB = (a.nO * CT * CT + 3) / 4;
  if (nSB + nOB == 0) return hipSuccess;
  hipLaunchKernelGGL(k_token_grads, dim3(nSB + nOB), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace pa
