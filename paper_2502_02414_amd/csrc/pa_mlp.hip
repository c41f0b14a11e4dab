// The first product of a block's MLP with its activation in one kernel
// (bf16 storage, gfx950): the feed-forward layer of the Transformer block
// that Physics-Attention sits in (Figure 2a; the block stack of Table 5's
// industrial model), x2 = x1 + GELU(h W1 + b1) W2 + b2 with h = LN2(x1).
//
//   forward:   G[n, f]  = GELU(u[n, f]),             u = h W1 + b1
//   backward:  dU[n, f] = (dY W2^T)[n, f] GELU'(u[n, f])
//
// The pre-activation u is never stored: the forward writes only GELU(u)
// (which the second product and the weight gradient of W2 read), and the
// backward recomputes u from h (K = C channels: a cheap contraction next to
// the [N, 4C] tensors it saves writing and reading).  Both contractions run
// on v_mfma_f32_16x16x32_bf16 with fp32 accumulation; the activation is
// applied to the fp32 accumulator and rounded to bf16 once.
//
// A block is persistent on its CU: each of its eight waves keeps the weights
// of 16 NCT output columns in registers (the MFMA A operand; W1 transposed
// once through LDS), and the block walks a range of the points in tiles of 32.
// A tile's rows of h (and dY) come from HBM in whole rows, two tiles ahead,
// through a double-buffered LDS tile that all eight waves read as the B
// operand; the results leave through a triple-buffered LDS tile as whole rows
// of the block's 128 NCT columns, so a tile costs one block barrier.  The
// activation of one 16-point half is issued step by step beside the products of
// the next.  The F / (128 NCT) column blocks of one range of points are placed on
// one XCD, so that h and dY come from HBM once and from that XCD's L2 after
// that.
// Measured in runs of one call at N = 500,000, K = 256, F = 1024: forward 503 ->
// 424 us, backward 761 -> 677 us; N = 4,000 46 -> 13 and 85 -> 15 us; K = 128, F =
// 512 219 -> 173 and 305 -> 238 us.  (Before: weights staged chunk by chunk by
// every block of 128 or 256 points, two barriers a chunk, and a rational erf.)
// Among the other products of a feed-forward layer, where the clock is lower,
// 512 and 740 us under the profiler.
// What bounds it, from copies of the kernel with parts removed (made with the
// shorter polynomials named below): backward 690 us of events, without stores 612, without the activation 597, without
// its loads 621, with only loads and LDS traffic 372; LDS (20 GB at 128 bytes
// a clock and CU: 290 us), the matrix cores (240 us), the VALU (280 us) and
// HBM (300 us) are about equally loaded and overlap in part.  Also tried:
// weights in LDS and the rows read from global memory as B operands (422 and
// 708 us: 16 bytes per lane 512 bytes apart), the same with four waves of
// twice the points (490 and 760 us), deeper LDS prefetch and scheduling groups
// of MFMAs and VALU (no change).
#include <type_traits>

#include "pa_internal.h"
#include "pa_stream.hpp"

namespace pa {

namespace {

// GELU(x) = x Phi(x) = max(x, 0) - z Q(z) and GELU'(x) = Phi(x) + x phi(x),
// z = |x|, Q(z) = 1 - Phi(z) the upper tail, phi(z) = exp(-z^2 / 2) /
// sqrt(2 pi).  The activation is the bulk of the kernel's VALU work (a
// transcendental takes the time of four other instructions), so each uses one
// exp2 and a polynomial of the logarithm, which is smooth (both decay like
// exp(-z^2 / 2)); fitted for this kernel over [0, 13.25] (weighted minimax,
// linear programming over 3,000 points):
//   Q(z) = exp2(p(z)), degree 10;
//   Q(z) - z phi(z) = (z0 - z) exp2(p(z)), z0 its only root, degree 11; then
//     GELU'(x) is 1 + v for x >= 0 and -v for x < 0, v = (z - z0) exp2(p).
// bf16 keeps fp32's exponents, so the lower tails need their own digits: the
// weights bound the relative error.  Evaluated in fp32 against 64 bits, x < 0:
//   GELU   7.0e-7 for z < 1, 3.8e-5 up to 3, 2.4e-4 up to 5, 1.5e-3 up to 12.9
//   GELU'  1.4e-7 absolute up to z = 3, 2.2e-5 up to 4, 5.1e-5 up to 6, 2.7e-4
//          up to 13
// and absolute at most 1.6e-7 (of the value where that exceeds 1) and 1.8e-7 (x
// > 0: relative 5e-7 and 3e-7); half a bf16 step is 2e-3 to 3.9e-3 of a value.  The rational erf of Abramowitz and Stegun
// 7.1.26, evaluated the same way, has 7.0e-7, 5.2e-5, 1.6e-3, 3.7e-2 and, for
// the slope, 3.0e-5, 1.0e-4, 2.3e-4, and takes a reciprocal more.  (Degrees 7
// and 8 weighted by the absolute error alone, 374 and 638 us where these take
// 404 and 678 us on the same box, N = 500,000, K = 256, F = 1024, lose all digits
// below x = -6.)
// From z = 13 exp2 has no normal result and both are 0 (below 1e-36; slope 1
// for x > 0).  The clamp keeps the polynomials finite and propagates NaN (IEEE
// minimum): GELU(+inf) = inf, GELU(-inf) = 0.
__device__ __forceinline__ float gelu_ap(float x) {
  const float z = __builtin_elementwise_minimum(fabsf(x), 14.f);
  float p = -1.005718064384098e-09f;
  p = fmaf(p, z, 5.430629101965678e-08f);
  p = fmaf(p, z, -1.151717242464656e-06f);
  p = fmaf(p, z, 1.1231582902837545e-05f);
  p = fmaf(p, z, -2.5174234906444326e-05f);
  p = fmaf(p, z, -0.0005898026865907013f);
  p = fmaf(p, z, 0.007740595377981663f);
  p = fmaf(p, z, -0.05302676558494568f);
  p = fmaf(p, z, -0.4590100646018982f);
  p = fmaf(p, z, -1.1511328220367432f);
  p = fmaf(p, z, -0.9999993443489075f);
  return fmaf(-z, fast_exp2(p), __builtin_elementwise_maximum(x, 0.f));
}
__device__ __forceinline__ float dgelu_ap(float x) {
  const float z = __builtin_elementwise_minimum(fabsf(x), 14.f);
  float p = -1.0389065302485179e-10f;
  p = fmaf(p, z, 7.800505130717283e-09f);
  p = fmaf(p, z, -2.573670201400091e-07f);
  p = fmaf(p, z, 4.93322613692726e-06f);
  p = fmaf(p, z, -6.138220487628132e-05f);
  p = fmaf(p, z, 0.0005271713016554713f);
  p = fmaf(p, z, -0.003265825565904379f);
  p = fmaf(p, z, 0.015184481628239155f);
  p = fmaf(p, z, -0.05506233870983124f);
  p = fmaf(p, z, -0.5606260299682617f);
  p = fmaf(p, z, -0.3831914961338043f);
  p = fmaf(p, z, -0.5884047746658325f);
  const float v = (z - 0.7517915246935644f) * fast_exp2(p);
  return x < 0.f ? -v : 1.f + v;
}

// NCT 16-column tiles per wave.
template <int K, int NCT, bool BWD>
struct MlpGeo {
  static constexpr int FCB = 128 * NCT;         // columns per block
  static constexpr int PTS = 32;                // points per tile (two halves of 16)
  static constexpr int KS = K / 32;             // K32 steps
  static constexpr int XR = K * 2 + 32;         // LDS row of h, dY (padded)
  static constexpr int XB = PTS * XR;
  static constexpr int SR = FCB * 2 + 16;       // LDS row of the results
  static constexpr int SB = PTS * SR;
  static constexpr int OFF_Y = 2 * XB;
  static constexpr int OFF_S = (BWD ? 4 : 2) * XB;
  static constexpr int R1 = FCB * 2 + 32;       // row of a 32-channel slab of W1 (at the start)
  static constexpr int USED = OFF_S + 3 * SB;
  static constexpr int LDS = USED > 32 * R1 ? USED : 32 * R1;
  static constexpr int XQ = PTS * K / 8;        // 16-byte chunks of an h tile
  static constexpr int XN = (XQ + 511) / 512;   // ... per thread
  static constexpr int SQ = PTS * FCB / 8 / 512;   // chunks of a result tile per thread
  static constexpr int WQ = 32 * FCB / 8 / 512;    // chunks of a W1 slab per thread
  static_assert(LDS <= kLdsBytes, "one block per CU fits");
};

struct MlpArgs {
  int64_t N;
  int F;
  int PG;           // ranges of the points
  const bf16* X;    // [N, K]: h
  const bf16* DY;   // [N, K]: the MLP output's gradient (backward)
  const bf16* W1;   // [K, F]
  const bf16* W2;   // [F, K] (backward)
  const float* b1;  // [F]
  bf16* out;        // [N, F]: GELU(u), or dU
};

template <int K, int NCT, bool BWD>
__global__ void __launch_bounds__(512) k_mlp_up(MlpArgs a) {
  using Gm = MlpGeo<K, NCT, BWD>;
  constexpr int KS = Gm::KS, FCB = Gm::FCB, PTS = Gm::PTS;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = lane_id(), r = lane & 15, g = lane >> 4;
  const int F = a.F, ncg = (F + FCB - 1) / FCB;
  // blocks are dealt to the XCDs round robin: block b takes item l, so that
  // the column blocks of one range of points share an XCD's L2
  const int nb = gridDim.x, bl = blockIdx.x;
  const int l = nb % 8 == 0 ? (bl % 8) * (nb / 8) + bl / 8 : bl;
  const int pg = l / ncg, f0 = (l - pg * ncg) * FCB;
  const int64_t tiles = (a.N + PTS - 1) / PTS;
  const int64_t t0 = tiles * pg / a.PG, t1 = tiles * (pg + 1) / a.PG;  // t0 < t1 (PG <= tiles)
  const int fw = f0 + 16 * NCT * wave;  // the wave's first column
  const bool on = fw < F;               // (F a multiple of 64; NCT <= 4 divides the waves' share)

  // the rows of tile t, 16-byte chunks q < XQ (past the end: the last one
  // again); rows past N read row N - 1, their results are not stored
  uint4 xr[Gm::XN], yr[BWD ? Gm::XN : 1];
  auto chunk = [&](int j) {
    const int q = threadIdx.x + 512 * j;
    return Gm::XQ % 512 == 0 || q < Gm::XQ ? q : Gm::XQ - 1;
  };
  auto load = [&](int64_t t) {
    const int64_t p0 = (t < t1 ? t : t1 - 1) * PTS;
    const int lim = last_row<PTS>(p0, a.N);
    const char* xs = reinterpret_cast<const char*>(a.X + p0 * K);
    const char* ys = BWD ? reinterpret_cast<const char*>(a.DY + p0 * K) : nullptr;
#pragma unroll
    for (int j = 0; j < Gm::XN; ++j) {
      const int q = chunk(j), row = q / (K / 8), c = q % (K / 8);
      const uint32_t off = (uint32_t)((row < lim ? row : lim) * K * 2 + 16 * c);
      xr[j] = ld_global16<false>(xs + off);
      if constexpr (BWD) yr[j] = ld_global16<false>(ys + off);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int j = 0; j < Gm::XN; ++j) {
      const int q = chunk(j), row = q / (K / 8), c = q % (K / 8);
      char* d = smem + buf * Gm::XB + row * Gm::XR + 16 * c;
      *reinterpret_cast<uint4*>(d) = xr[j];
      if constexpr (BWD) *reinterpret_cast<uint4*>(d + Gm::OFF_Y) = yr[j];
    }
  };

  // the wave's weights: lane (r, g) holds column fw + 16 ct + r, channels
  // 32 s + 8 g .. + 7.  W1 [K, F] comes in slabs of 32 channels through LDS.
  K32<bf16> w1[NCT][KS], w2[BWD ? NCT : 1][BWD ? KS : 1];
  f32x4 bias[NCT];
  {
    uint4 v[KS][Gm::WQ];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int j = 0; j < Gm::WQ; ++j) {
        const int q = threadIdx.x + 512 * j, row = q / (FCB / 8), c = 8 * (q % (FCB / 8));
        const int col = f0 + c < F ? f0 + c : F - 8;  // (columns past F are not stored)
        v[s][j] = ld_global16<false>(a.W1 + (int64_t)(32 * s + row) * F + col);
      }
    const int tb = (8 * g + (r >> 2)) * Gm::R1 + 8 * (r & 3) + 32 * NCT * wave;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      block_sync();
#pragma unroll
      for (int j = 0; j < Gm::WQ; ++j) {
        const int q = threadIdx.x + 512 * j, row = q / (FCB / 8), c = q % (FCB / 8);
        *reinterpret_cast<uint4*>(smem + row * Gm::R1 + 16 * c) = v[s][j];
      }
      block_sync();
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        K16<bf16> lo, hi;
        ld_tr<bf16>(lo, smem, tb, 32 * ct, Gm::R1);
        ld_tr<bf16>(hi, smem, tb, 4 * Gm::R1 + 32 * ct, Gm::R1);
        w1[ct][s].v = __builtin_shufflevector(lo.v, hi.v, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    }
  }
  load(t0);
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    const int fc = on ? fw + 16 * ct : 0;
    bias[ct] = *reinterpret_cast<const f32x4*>(a.b1 + fc + 4 * g);
    if constexpr (BWD) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
        w2[ct][s].v = __builtin_bit_cast(
            bf16x8, ld_global16<false>(a.W2 + (int64_t)(fc + r) * K + 32 * s + 8 * g));
    }
  }
  block_sync();  // the last slab is read: its LDS becomes the tiles
  store(0);
  load(t0 + 1);

  const int xb = r * Gm::XR + 16 * g;  // B fragment: row 16 u + r, channels 32 s + 8 g ..
  const int sb = Gm::OFF_S + r * Gm::SR + (16 * NCT * wave + 4 * g) * 2;
  f32x4 accu[2][NCT], acc[2][BWD ? NCT : 1];  // X W1 + b1 and dY W2^T of two halves
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      accu[u][ct] = zero4();
      if constexpr (BWD) acc[u][ct] = zero4();
    }
  // columns 16 ct + 4 g .. + 3 of a half's point r, element e = 4 ct + i
  auto act = [&](int u, int e, bf16x4& o) {
    const int ct = e / 4, i = e % 4;
    if constexpr (BWD)
      o[i] = (bf16)(acc[u][ct][i] * dgelu_ap(accu[u][ct][i]));
    else
      o[i] = (bf16)gelu_ap(accu[u][ct][i]);
  };
  // products of half U of the tile in buffer `buf`, beside the activation of
  // the half before (its results to the staging rows at `out`)
  constexpr int EPS = 4 * NCT / KS > 0 ? 4 * NCT / KS : 1;  // elements per K32 step
  auto half = [&](auto UC, const char* buf, char* out) {
    constexpr int U = decltype(UC)::value;
    K32<bf16> xf[2], yf[2];
    auto frag = [&](int s) {
      ld_k32(xf[s % 2], buf + xb + 16 * U * Gm::XR + 64 * s);
      if constexpr (BWD) ld_k32(yf[s % 2], buf + Gm::OFF_Y + xb + 16 * U * Gm::XR + 64 * s);
    };
    frag(0);
    bf16x4 o{};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s + 1 < KS) frag(s + 1);
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        accu[U][ct] = mma32(w1[ct][s], xf[s % 2], s == 0 ? bias[ct] : accu[U][ct]);
        if constexpr (BWD)
          acc[U][ct] = mma32(w2[ct][s], yf[s % 2], s == 0 ? zero4() : acc[U][ct]);
      }
#pragma unroll
      for (int e = s * EPS; e < (s + 1) * EPS && e < 4 * NCT; ++e) {
        act(U ^ 1, e, o);
        if (e % 4 == 3) *reinterpret_cast<bf16x4*>(out + 32 * (e / 4)) = o;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // whole rows of a staged tile to memory
  auto write = [&](int64_t t, const char* stg) {
    const int64_t p0 = t * PTS;
#pragma unroll
    for (int j = 0; j < Gm::SQ; ++j) {
      const int q = threadIdx.x + 512 * j, row = q / (FCB / 8), c = q % (FCB / 8);
      const uint4 v = *reinterpret_cast<const uint4*>(stg + row * Gm::SR + 16 * c);
      if (p0 + row < a.N && f0 + 8 * c < F) st_global16(a.out + (p0 + row) * F + f0 + 8 * c, v);
    }
  };

  // Iteration t: tile t + 1 to the other buffer (last read before this
  // barrier), tile t + 2 requested, tile t - 2 written out (its second half
  // was staged during iteration t - 1), tile t computed.
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  int sp = 2, sc = 0;  // staging buffers of tiles t - 1 and t; the third is tile t - 2's
  for (int64_t t = t0; t < t1; ++t) {
    const int buf = (int)(t - t0) & 1;
    block_sync();
    if (t + 1 < t1) store(buf ^ 1);
    load(t + 2);
    const int sn = 3 - sp - sc;
    if (t >= t0 + 2) write(t - 2, smem + Gm::OFF_S + sn * Gm::SB);
    if (on) {
      // (the first tile's turn stages zeros where nothing is read)
      half(H0{}, smem + buf * Gm::XB, smem + sb + sp * Gm::SB + 16 * Gm::SR);
      half(H1{}, smem + buf * Gm::XB, smem + sb + sc * Gm::SB);
    }
    sp = sc;
    sc = sn;
  }
  if (on) {
    bf16x4 o{};
#pragma unroll
    for (int e = 0; e < 4 * NCT; ++e) {
      act(1, e, o);
      if (e % 4 == 3)
        *reinterpret_cast<bf16x4*>(smem + sb + sp * Gm::SB + 16 * Gm::SR + 32 * (e / 4)) = o;
    }
  }
  block_sync();
  if (t1 - t0 >= 2) write(t1 - 2, smem + Gm::OFF_S + (3 - sp - sc) * Gm::SB);
  write(t1 - 1, smem + Gm::OFF_S + sp * Gm::SB);
}

// One block per CU (256), or fewer where there are not as many tiles.
template <int K, int NCT, bool BWD>
hipError_t launch_k(MlpArgs a, hipStream_t st) {
  using Gm = MlpGeo<K, NCT, BWD>;
  const int64_t tiles = (a.N + Gm::PTS - 1) / Gm::PTS;
  const int ncg = (a.F + Gm::FCB - 1) / Gm::FCB;
  const int64_t PG = ncg < 256 ? 256 / ncg : 1;
  a.PG = (int)(PG < tiles ? PG : tiles);
  hipLaunchKernelGGL((k_mlp_up<K, NCT, BWD>), dim3(ncg * a.PG), dim3(512), Gm::LDS, st, a);
  return hipGetLastError();
}
// Columns per wave: 64 forward and 32 backward (two weight matrices) fill
// half of a wave's registers at K = 256 and read h the fewest times; fewer
// where F is no multiple of the block's columns (idle waves).
template <int K>
hipError_t launch_kf(const MlpArgs& a, hipStream_t st) {
  if (a.DY) return a.F % 256 == 0 ? launch_k<K, 2, true>(a, st) : launch_k<K, 1, true>(a, st);
  return a.F % 512 == 0   ? launch_k<K, 4, false>(a, st)
         : a.F % 256 == 0 ? launch_k<K, 2, false>(a, st)
                          : launch_k<K, 1, false>(a, st);
}

}  // namespace

bool mlp_up_served(int K, int F) {
  return (K == 64 || K == 128 || K == 256) && F >= 64 && F % 64 == 0;
}

hipError_t launch_mlp_up(int64_t N, int K, int F, const void* X, const void* W1, const float* b1,
                         const void* DY, const void* W2, void* out, hipStream_t st) {
  if (N < 1 || !mlp_up_served(K, F) || !X || !W1 || !b1 || !out) return hipErrorInvalidValue;
  if (DY && !W2) return hipErrorInvalidValue;
  MlpArgs a{N, F, 1, (const bf16*)X, (const bf16*)DY, (const bf16*)W1, (const bf16*)W2, b1,
            (bf16*)out};
  switch (K) {
    case 64: return launch_kf<64>(a, st);
    case 128: return launch_kf<128>(a, st);
    default: return launch_kf<256>(a, st);
  }
}

}  // namespace pa
