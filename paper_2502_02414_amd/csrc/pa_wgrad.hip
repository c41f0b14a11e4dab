// Weight gradients of the linear layers (gfx950):
//   D [m, n] = alpha A^T B,   A [k, m], B [k, n] row-major bf16 or fp32, D fp32,
// a long contraction over the k points into a small output (dW1 = h^T dU and
// dW2 = GELU(u)^T dY of a block's feed-forward layer).
//
// Bound: A and B are read once (k (m + n) 2 bytes; at k = 500,000, 256 x
// 1024, 1.28 GB) and 2 k m n operations run on the matrix cores.  One block
// per CU owns an output tile (up to 256 x 256: 128 accumulator registers per
// lane over eight waves, so an LDS byte read feeds eight MFMA operands) and a
// contiguous range of the points; the splits of the points give every CU a
// tile, and the fp32 partial tiles are added in split order by the ordered
// reduction (deterministic).  Stages of 32 points are loaded two ahead into
// registers and written to a double-buffered LDS tile in their row-major
// form; both MFMA operands are then read transposed (ds_read_b64_tr_b16;
// fp32: rows as they are, v_mfma_f32_16x16x4_f32, bound by the matrix cores'
// fp32 rate).
// Measured in runs of one product, with the reduction, against strided-batched
// library products with the same split: 1024 x 256 at k = 500,000 437 -> 300 us
// (the kernel alone 260 us from idle, 4.9 TB/s; the clock falls under a run of
// such products), k = 33,000 (one library product) 117 -> 39 us; 512 x 128 at k
// = 500,000 219 -> 131 us; 256 x 64 170 -> 61 us.  HBM reads: the operands, once.
#include <cmath>

#include "pa_internal.h"
#include "pa_stream.hpp"

namespace pa {
namespace {

struct WgradArgs {
  const void* A;  // [k, m]
  const void* B;  // [k, n]
  float* out;     // [P][m][n] (P = 1: D itself)
  int64_t k;
  int m, n, P;
  float alpha;
};

// Eight waves over a TM x TN tile: WM along m, 8 / WM along n.
template <typename T, int TM, int TN>
struct WgradGeo {
  static constexpr int SZ = sizeof(T);
  static constexpr int WM = TM >= 4 * TN ? 8 : TM >= TN ? 4 : TM * 4 <= TN ? 1 : 2;
  static constexpr int WN = 8 / WM;
  static constexpr int MT = TM / WM / 16, NT = TN / WN / 16;  // 16-wide tiles per wave
  // LDS rows, padded: a transposed bf16 read covers 16 rows of 32 bytes, a
  // fp32 read 4 rows of 64 bytes and more, each on banks of their own
  static constexpr int PAD = SZ == 2 ? 32 : 64;
  static constexpr int RA = TM * SZ + PAD, RB = TN * SZ + PAD;
  static constexpr int OFF_B = 32 * RA;
  static constexpr int BUF = OFF_B + 32 * RB;
  static constexpr int LDS = 2 * BUF;
  static constexpr int CA = TM * SZ / 16, CB = TN * SZ / 16;  // 16-byte chunks per row
  static constexpr int NQ = 32 * (CA + CB);                   // chunks of a stage
  static constexpr int NC = (NQ + 511) / 512;                 // ... per thread
  static_assert(MT >= 1 && NT >= 1, "a wave owns at least one MFMA tile");
};

template <typename T, int TM, int TN>
__global__ void __launch_bounds__(512) k_wgrad(WgradArgs a) {
  using G_ = WgradGeo<T, TM, TN>;
  constexpr int SZ = sizeof(T);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // blocks are dealt to the XCDs round robin: block b works on item l, so
  // that the tiles of one split (which read the same rows) share an L2
  const int nb = gridDim.x, b = blockIdx.x;
  const int l = nb % 8 == 0 ? (b % 8) * (nb / 8) + b / 8 : b;
  const int tn = a.n / TN, tiles = (a.m / TM) * tn;
  const int split = l / tiles, tile = l - split * tiles;
  const int m0 = tile / tn * TM, n0 = tile % tn * TN;
  const int64_t steps = (a.k + 31) / 32;
  const int64_t s0 = steps * split / a.P, s1 = steps * (split + 1) / a.P;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane_id() & 15, g = lane_id() >> 4;
  const int wm = wave / G_::WN * (16 * G_::MT), wn = wave % G_::WN * (16 * G_::NT);

  // thread t's chunks of a stage: chunk q < 32 CA of the A rows, then B's
  // (past the end: the last chunk again, the same bytes to the same place);
  // where a round of 512 chunks lies in one matrix, which one is known at
  // compile time and the address is a uniform base plus a 32-bit offset
  uint4 reg[2][G_::NC];
  struct Chunk { bool isA; int row, c; };
  auto chunk = [&](int j) {
    const int t = threadIdx.x + 512 * j;
    const int q = G_::NQ % 512 == 0 || t < G_::NQ ? t : G_::NQ - 1;
    constexpr int QA = 32 * G_::CA;
    const bool isA = QA % 512 == 0 ? 512 * j < QA : q < QA;
    const int e = isA ? q : q - QA, ch = isA ? G_::CA : G_::CB;
    return Chunk{isA, e / ch, e % ch};
  };
  auto load = [&](uint4 (&v)[G_::NC], int64_t s) {
    const int64_t p0 = (s < s1 ? s : s1 - 1) * 32;
    const int lim = a.k - 1 - p0 < 31 ? (int)(a.k - 1 - p0) : 31;
    const char* pa = reinterpret_cast<const char*>(a.A) + (p0 * a.m + m0) * SZ;
    const char* pb = reinterpret_cast<const char*>(a.B) + (p0 * a.n + n0) * SZ;
#pragma unroll
    for (int j = 0; j < G_::NC; ++j) {
      const Chunk q = chunk(j);
      const int row = q.row < lim ? q.row : lim;  // rows past k: row k - 1, zeroed below
      v[j] = ld_global16<false>((q.isA ? pa : pb) +
                                (uint32_t)(row * (q.isA ? a.m : a.n) * SZ + 16 * q.c));
    }
  };
  auto store = [&](char* buf, const uint4 (&v)[G_::NC], int64_t s) {
    auto put = [&](int j, const uint4& x) {
      const Chunk q = chunk(j);
      *reinterpret_cast<uint4*>(buf + (q.isA ? q.row * G_::RA : G_::OFF_B + q.row * G_::RB) +
                                16 * q.c) = x;
    };
    if (s * 32 + 32 <= a.k) {
#pragma unroll
      for (int j = 0; j < G_::NC; ++j) put(j, v[j]);
    } else {
      const int rows = (int)(a.k - s * 32);
#pragma unroll
      for (int j = 0; j < G_::NC; ++j) put(j, chunk(j).row < rows ? v[j] : uint4{0, 0, 0, 0});
    }
  };

  f32x4 acc[G_::MT][G_::NT];  // [n 4g+i][m r] of each 16 x 16 tile
#pragma unroll
  for (int i = 0; i < G_::MT; ++i)
#pragma unroll
    for (int j = 0; j < G_::NT; ++j) acc[i][j] = zero4();

  // bf16: transposed fragments, lane (r, g) elements = points 4g .. 4g+3 and
  // 16+4g .. 16+4g+3 of column r (the same points for both operands): a read
  // of 8 bytes per lane covers 16 consecutive rows, 32 bytes apart in the
  // banks.  fp32: point 4q + g of step q, MT (NT) consecutive columns from MT
  // r (NT r) in one read, the column of each of the wave's tiles.
  const int tra = (SZ == 2 ? tr_base<bf16>(G_::RA) : g * G_::RA + 4 * G_::MT * r) + wm * SZ;
  const int trb =
      (SZ == 2 ? tr_base<bf16>(G_::RB) : g * G_::RB + 4 * G_::NT * r) + wn * SZ + G_::OFF_B;
  auto frag = [&](const char* buf, int base, int off, int RB) {
    K16<bf16> lo, hi;
    ld_tr<bf16>(lo, buf, base, off, RB);
    ld_tr<bf16>(hi, buf, base, off + 16 * RB, RB);
    K32<bf16> f;
    f.v = __builtin_shufflevector(lo.v, hi.v, 0, 1, 2, 3, 4, 5, 6, 7);
    return f;
  };
  auto compute = [&](const char* buf) {
    if constexpr (SZ == 2) {
      K32<bf16> fa[G_::MT];
#pragma unroll
      for (int i = 0; i < G_::MT; ++i) fa[i] = frag(buf, tra, 32 * i, G_::RA);
      // (B's fragments one tile ahead of their MFMAs: more would spill)
      struct F { K32<bf16> b; };
      pipelined<G_::NT, 2, F>([&](int j, F& f) { f.b = frag(buf, trb, 32 * j, G_::RB); },
                              [&](int j, F& f) {
#pragma unroll
                                for (int i = 0; i < G_::MT; ++i)
                                  acc[i][j] = mma32(f.b, fa[i], acc[i][j]);
                              });
    } else {
      struct F { float a[G_::MT], b[G_::NT]; };
      pipelined<8, 2, F>(
          [&](int q, F& f) {
            __builtin_memcpy(f.a, __builtin_assume_aligned(buf + tra + 4 * q * G_::RA, 4 * G_::MT),
                             sizeof f.a);
            __builtin_memcpy(f.b, __builtin_assume_aligned(buf + trb + 4 * q * G_::RB, 4 * G_::NT),
                             sizeof f.b);
          },
          [&](int q, F& f) {
#pragma unroll
            for (int i = 0; i < G_::MT; ++i)
#pragma unroll
              for (int j = 0; j < G_::NT; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
          });
    }
  };

  // (P <= steps: every split has at least one step)
  load(reg[0], s0);
  load(reg[1], s0 + 1);
  store(smem, reg[0], s0);
  load(reg[0], s0 + 2);
  block_sync();
  // step s computes on buffer (s - s0) & 1 while step s + 1 is written to
  // the other one (last read before the previous barrier) and step s + 3 is
  // requested; whole rounds of two steps, a last single step after them
  int64_t s = s0;
  for (; s + 1 < s1; s += 2) {
    store(smem + G_::BUF, reg[1], s + 1);
    load(reg[1], s + 3);
    compute(smem);
    block_sync();
    store(smem, reg[0], s + 2 < s1 ? s + 2 : s1 - 1);
    load(reg[0], s + 4);
    compute(smem + G_::BUF);
    block_sync();
  }
  if (s < s1) compute(smem);

  // element e of tile (i, j): bf16 column n = 16 j + 4 g + e of row m = 16 i
  // + r; fp32 column NT (4 g + e) + j of row MT r + i
  float* out = a.out + (int64_t)split * a.m * a.n + (int64_t)n0 + wn;
#pragma unroll
  for (int i = 0; i < G_::MT; ++i) {
    float* row = out + (int64_t)(m0 + wm + (SZ == 2 ? 16 * i + r : G_::MT * r + i)) * a.n;
    if constexpr (SZ == 2) {
#pragma unroll
      for (int j = 0; j < G_::NT; ++j) {
        f32x4 v = acc[i][j];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] *= a.alpha;
        *reinterpret_cast<f32x4*>(row + 16 * j + 4 * g) = v;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v[G_::NT];
#pragma unroll
        for (int j = 0; j < G_::NT; ++j) v[j] = acc[i][j][e] * a.alpha;
        __builtin_memcpy(__builtin_assume_aligned(row + G_::NT * (4 * g + e), 4 * G_::NT), v,
                         sizeof v);
      }
    }
  }
}

template <typename T, int TM, int TN>
hipError_t launch_w(const WgradArgs& a, hipStream_t st) {
  const int blocks = (a.m / TM) * (a.n / TN) * a.P;
  hipLaunchKernelGGL((k_wgrad<T, TM, TN>), dim3(blocks), dim3(512), (WgradGeo<T, TM, TN>::LDS), st,
                     a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The same product with no room for partial tiles, and of any m, n and k: one
// block per 16 TI x 16 TI output tile over all points, its waves on every
// WAVES-th chunk of 32 points, their sums added in wave order.
// Operands go straight from global memory to the MFMA layout, chunks ahead:
// lane (r, g) holds points 4 s + g, s < 8, of TI columns (the same points for
// both operands), in one load of TI elements where the output is whole tiles
// (WHOLE), else element by element with the columns clamped.
// ---------------------------------------------------------------------------
struct WgradOneArgs {
  const void* A;  // [k, m]
  const void* B;  // [k, n]
  float* D;       // [m, n]
  int64_t k, m, n;
  float alpha;
};

template <int TI>
struct OneGeo {
  static constexpr int WAVES = TI == 1 ? 16 : TI == 2 ? 8 : 4;  // (the fewer, the more registers a lane)
  static constexpr int DEEP = TI == 2 ? 2 : TI == 1 ? 4 : 3;   // chunks in flight and at work
  static constexpr int LDS = WAVES * TI * TI * 64 * 16;
};

template <typename T, int TI, bool WHOLE>
__global__ void __launch_bounds__(64 * OneGeo<TI>::WAVES) k_wgrad_one(WgradOneArgs a) {
  constexpr int WAVES = OneGeo<TI>::WAVES, DEEP = OneGeo<TI>::DEEP;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  f32x4* part = reinterpret_cast<f32x4*>(smem);  // [wave][tile][lane]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = lane_id(), r = lane & 15, g = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * 16 * TI, n0 = (int64_t)blockIdx.x * 16 * TI;
  // Lane r's column of tile i: TI r + i (past the end: the last one; not
  // stored), as a byte offset into a row; a chunk's address is a uniform row
  // plus a 32-bit offset (m n <= 2^21, so 32 rows are below 2^28 bytes).
  struct Row { T v[TI]; };
  struct Chunk { Row a[8], b[8]; };
  const uint32_t lda = (uint32_t)a.m * sizeof(T), ldb = (uint32_t)a.n * sizeof(T);
  uint32_t ca[TI], cb[TI];
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    ca[i] = (uint32_t)(WHOLE || m0 + TI * r + i < a.m ? m0 + TI * r + i : a.m - 1) * sizeof(T);
    cb[i] = (uint32_t)(WHOLE || n0 + TI * r + i < a.n ? n0 + TI * r + i : a.n - 1) * sizeof(T);
  }
  auto row = [](Row& d, const char* p, uint32_t rows, const uint32_t (&c)[TI]) {
    if constexpr (WHOLE) {
      __builtin_memcpy(&d, p + (rows + c[0]), sizeof d);
    } else {
#pragma unroll
      for (int i = 0; i < TI; ++i) __builtin_memcpy(&d.v[i], p + (rows + c[i]), sizeof d.v[i]);
    }
  };
  auto load = [&](Chunk& v, int64_t c) {
    const char* A = reinterpret_cast<const char*>(a.A) + 32 * c * lda;
    const char* B = reinterpret_cast<const char*>(a.B) + 32 * c * ldb;
    if (32 * c + 32 <= a.k) {
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        row(v.a[s], A, g * lda, ca);
        row(v.b[s], B, g * ldb, cb);
        A += 4 * lda;
        B += 4 * ldb;
        // (uniform: without this an address per row and column stays in
        // registers, which spills; the one-load form is faster as it is)
        if constexpr (!WHOLE) asm volatile("" : "+s"(A), "+s"(B));
      }
    } else {
      const int last = (int)(a.k - 1 - 32 * c);  // (points past k: the last row)
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const uint32_t p = 4 * s + g < last ? 4 * s + g : last;
        row(v.a[s], A, p * lda, ca);
        row(v.b[s], B, p * ldb, cb);
      }
    }
  };
  f32x4 acc[TI][TI];  // [n TI (4g + e) + j][m TI r + i]
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TI; ++j) acc[i][j] = zero4();
  auto compute = [&](Chunk& v, int64_t c) {
    if (32 * c + 32 > a.k) {  // points past k: zeros
#pragma unroll
      for (int s = 0; s < 8; ++s)
        if (32 * c + 4 * s + g >= a.k) {
          v.a[s] = Row{};
          v.b[s] = Row{};
        }
    }
    if constexpr (sizeof(T) == 2) {
      K32<bf16> x[TI], y[TI];
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          x[i].v[s] = v.a[s].v[i];
          y[i].v[s] = v.b[s].v[i];
        }
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j) acc[i][j] = mma32(y[j], x[i], acc[i][j]);
    } else {
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v.b[s].v[j], v.a[s].v[i], acc[i][j],
                                                             0, 0, 0);
    }
  };
  // the wave's chunks wave, wave + WAVES, .. through a ring of DEEP
  const int64_t chunks = (a.k + 31) / 32;
  Chunk v[DEEP];
#pragma unroll
  for (int d = 0; d + 1 < DEEP; ++d)
    if (wave + d * WAVES < chunks) load(v[d], wave + d * WAVES);
  for (int64_t c0 = wave; c0 < chunks; c0 += DEEP * WAVES) {
#pragma unroll
    for (int d = 0; d < DEEP; ++d) {
      const int64_t c = c0 + d * WAVES, next = c + (DEEP - 1) * WAVES;
      if (next < chunks) load(v[(d + DEEP - 1) % DEEP], next);
      if (c < chunks) compute(v[d], c);
    }
  }
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TI; ++j) part[(wave * TI * TI + i * TI + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  for (int t = wave; t < TI * TI; t += WAVES) {
    f32x4 x = part[t * 64 + lane];
#pragma unroll
    for (int q = 1; q < WAVES; ++q) x += part[(q * TI * TI + t) * 64 + lane];
    const int64_t m = m0 + TI * r + t / TI;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t n = n0 + TI * (4 * g + e) + t % TI;
      if (WHOLE || (m < a.m && n < a.n)) a.D[m * a.n + n] = a.alpha * x[e];
    }
  }
}

template <typename T, int TI, bool WHOLE>
hipError_t launch_one_t(const WgradOneArgs& a, hipStream_t st) {
  const int e = 16 * TI;
  const dim3 grid((unsigned)((a.n + e - 1) / e), (unsigned)((a.m + e - 1) / e));
  hipLaunchKernelGGL((k_wgrad_one<T, TI, WHOLE>), grid, dim3(64 * OneGeo<TI>::WAVES),
                     OneGeo<TI>::LDS, st, a);
  return hipGetLastError();
}

// The largest tiles that still give half of the CUs a block: every one of them
// reads all points.  (Bound by the load path and latency; bf16: 1024 x 512 at k
// = 33,000, 128 blocks of 64 x 64: 207 us, 32 x 32: 306 us; 1024 x 256, 64 and
// 256 blocks: 263 and 119 us; 512 x 128, k = 500,000, 64 blocks of 32 x 32 and
// 256 of 16 x 16: 3.3 and 2.4 ms.)
template <typename T>
hipError_t launch_one(const WgradOneArgs& a, hipStream_t st) {
  auto whole = [&](int e) { return a.m % e == 0 && a.n % e == 0; };
  auto blocks = [&](int e) { return ((a.m + e - 1) / e) * ((a.n + e - 1) / e); };
  if (whole(64) && blocks(64) >= 128) return launch_one_t<T, 4, true>(a, st);
  if (blocks(32) >= 128)
    return whole(32) ? launch_one_t<T, 2, true>(a, st) : launch_one_t<T, 2, false>(a, st);
  return launch_one_t<T, 1, false>(a, st);
}

// ---------------------------------------------------------------------------
// D = the sum of P partial products, in split order: G groups of threads per
// output, each adding a range of the partials in fp64, their sums added in
// group order.  Bound by reading the partials once; 16 bytes per lane.  (The
// reduction of the block records, k_reduce, has 16 groups of one column each
// and reads the last record again where there are fewer: with it a 1024 x 256
// output took 25 us for 3 partials and 27 for 62, 2048 x 1024 183 us for 2; now
// 3.5, 11 and 4.)
// ---------------------------------------------------------------------------
template <int G>
__global__ void __launch_bounds__(256) k_add_parts(const f32x4* __restrict__ parts, int P,
                                                   int64_t quads, f32x4* __restrict__ D) {
  constexpr int Q = 256 / G;  // outputs of four columns per block
  __shared__ f64x4 sums[G > 1 ? G - 1 : 1][Q];
  const int q = threadIdx.x % Q, grp = threadIdx.x / Q;
  const int64_t i = (int64_t)blockIdx.x * Q + q, ic = i < quads ? i : quads - 1;
  const int p0 = P * grp / G, p1 = P * (grp + 1) / G;  // (P >= G: at least one)
  f64x4 acc{0.0, 0.0, 0.0, 0.0};
  for (int p = p0; p < p1; p += 4) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = parts[(int64_t)(p + u < p1 ? p + u : p1 - 1) * quads + ic];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (p + u < p1)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += (double)v[u][e];
  }
  if constexpr (G > 1) {
    if (grp > 0) sums[grp - 1][q] = acc;
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 0; g + 1 < G; ++g) acc += sums[g][q];
  }
  if (i < quads) D[i] = f32x4{(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
}

template <int G>
hipError_t launch_add(const float* parts, int P, int64_t quads, float* D, hipStream_t st) {
  constexpr int Q = 256 / G;
  hipLaunchKernelGGL(k_add_parts<G>, dim3((unsigned)((quads + Q - 1) / Q)), dim3(256), 0, st,
                     reinterpret_cast<const f32x4*>(parts), P, quads, reinterpret_cast<f32x4*>(D));
  return hipGetLastError();
}

// Tile edge along a dimension (a multiple of 64): the largest of 256, 128, 64
// up to cap that divides it.  (256 rows come with 256 columns only.)
int edge(int64_t v, int cap) {
  return cap >= 256 && v % 256 == 0 ? 256 : cap >= 128 && v % 128 == 0 ? 128 : 64;
}
int64_t tiles_of(int64_t m, int64_t n, int cap) { return (m / edge(m, cap)) * (n / edge(n, cap)); }

// 256 x 256, 128 x 256 and 64 x 256 tiles in bf16 for rows of whole 256-column
// tiles and at least 1.6e10 points x outputs.  Below that, blocks of smaller
// tiles fill the chip sooner (us, tiles up to 128 and 256): 256 x 256, k = 131,072
// 37 and 45; 1024 x 256, k = 50,000 51 and 54, k = 66,000 64 and 58; 2048 x 256, k =
// 24,000 49 and 54, k = 33,000 63 and 58; 2048 x 512, k = 12,000 47 and 55, k =
// 16,384 60 and 59; 2048 x 1024, k = 12,000 84 and 72, k = 50,000 313 and 207.  Tiles
// of 256 x 128 and 256 x 64 gain nothing (1024 x 384, k = 100,000 133 and 143; 1024
// x 192, k = 131,072 152 and 150), nor do any in fp32, which the matrix cores bind.
constexpr double kWideWork = 1.6e10;
int largest_edge(int64_t m, int64_t n, int64_t k, int dtype) {
  return dtype == 1 && n % 256 == 0 && (double)k * (double)(m * n) >= kWideWork ? 256 : 128;
}

// Splits of the points: one block per CU at most, and no more than pay for
// their partial tile.  A split costs a write and a read of m n floats (about
// 8 m n bytes at 4 TB/s); the points cost k / 32 steps of about 0.5 us (fp32
// 2 us) over the splits: P = sqrt(k / 32 x step / cost) minimises the sum.
int splits(int64_t m, int64_t n, int64_t k, int dtype, int cap) {
  const int64_t tiles = tiles_of(m, n, cap), steps = (k + 31) / 32;
  const double cost_us = 8.0 * (double)m * (double)n / 4e6;
  int64_t P = (int64_t)std::sqrt((double)steps * (dtype == 1 ? 0.5 : 2.0) / cost_us);
  P = P < 256 / tiles ? P : 256 / tiles;
  P = P < steps ? P : steps;
  return (int)(P < 1 ? 1 : P);
}

}  // namespace

// With room for fewer partials than the points are worth splitting into,
// smaller tiles (while one block per CU takes them) make up for the blocks:
// bf16 1024 x 256 at k = 500,000 with 1, 2, 4, 16 and 64 MB of workspace 1.9,
// 1.9, 1.2, 0.45 and 0.29 ms (256 x 256 tiles alone, and with half of the
// workspace: 12.0, 12.0, 6.1, 1.6 and 0.48 ms).  Below four partials the
// product in one piece is faster (two: 2.5 ms against 1.9 ms; four: 1.3 ms)
// unless larger tiles fill half of the CUs (1024 x 2048 at k = 100,000, 128
// blocks: 1.2 ms against 1.6 ms).
WgradPlan wgrad_plan(int64_t m, int64_t n, int64_t k, int dtype, int64_t most) {
  WgradPlan w{largest_edge(m, n, k, dtype), 0, true};
  w.P = splits(m, n, k, dtype, w.cap);
  while (w.P > most && w.cap > 64 && tiles_of(m, n, w.cap / 2) * (most > 1 ? most : 1) <= 256) {
    w.cap /= 2;
    w.P = splits(m, n, k, dtype, w.cap);
  }
  if (w.P > 1 && w.P > most) {
    w.P = most > 1 ? (int)most : 1;
    w.pays = w.P >= 4 || (w.cap >= 128 && tiles_of(m, n, w.cap) * w.P >= 128);
  }
  return w;
}

// What k_wgrad can form: whole 64 x 64 tiles.
bool wgrad_whole(int64_t m, int64_t n, int64_t k, int dtype) {
  return m >= 64 && n >= 64 && m % 64 == 0 && n % 64 == 0 && m * n <= (2 << 20) && k >= 512 &&
         (dtype == 1 || k < (1 << 17));
}

// ... and where it is the better product (us: hipBLASLt's, its candidates timed
// or the heuristic's first one, and this kernel's with its reduction).
// bf16: 512 x 256, k = 1,000 13, 15 and 10; 1024 x 256, k = 2,000 14, 20 and 14, k =
// 4,096 18, 28 and 18; 1024 x 512, k = 4,096 25, 28 and 22; 2048 x 1024, k = 4,096
// 35, 39 and 36, k = 33,000 184, 237 and 137.
// fp32, up to 128 Ki outputs: 128 x 512, k = 2,000 12, 17 and 18, k = 8,000 30, 47
// and 26; 512 x 256, k = 4,096 17, 25 and 28, k = 12,000 45, 81 and 40: slower where
// short, but its fp64 sum of many partials is closer to the product (128 x 512, k =
// 2,000: relative error 4.0e-7, 8.0e-7 and 1.5e-7).  1024 x 256: k = 12,000 65, 82
// and 64, k = 16,384 90, 103 and 82.  1024 x 512: slower at every length (k = 8,000
// 67, 68 and 82, k = 33,000 259, 326 and 286), as are larger ones.
// From 2^17 points fp32 stays with the split library products, which are as fast
// or faster (128 x 256, k = 131,072 88 and 83; 128 x 512 156 and 151; 512 x 256 247
// and 285; 1024 x 256 468 and 556) and whose partial sums are shorter.
bool wgrad_served(int64_t m, int64_t n, int64_t k, int dtype) {
  const int64_t out = m * n;
  if (!wgrad_whole(m, n, k, dtype)) return false;
  if (out <= (1 << 17)) return true;
  return dtype == 1 ? k >= 4096 : out <= (1 << 18) && k >= 16384;
}

hipError_t launch_wgrad(int64_t m, int64_t n, int64_t k, float alpha, const void* A,
                        const void* B, int dtype, float* out, const WgradPlan& w,
                        hipStream_t st) {
  if (!wgrad_whole(m, n, k, dtype) || w.P < 1 || w.P > (k + 31) / 32 || !A || !B || !out)
    return hipErrorInvalidValue;
  const WgradArgs a{A, B, out, k, (int)m, (int)n, w.P, alpha};
  const int e = edge(m, w.cap) * 1000 + edge(n, w.cap);
  if (dtype == 1) {
    switch (e) {
      case 256256: return launch_w<bf16, 256, 256>(a, st);
      case 128256: return launch_w<bf16, 128, 256>(a, st);
      case 128128: return launch_w<bf16, 128, 128>(a, st);
      case 128064: return launch_w<bf16, 128, 64>(a, st);
      case 64256: return launch_w<bf16, 64, 256>(a, st);
      case 64128: return launch_w<bf16, 64, 128>(a, st);
      case 64064: return launch_w<bf16, 64, 64>(a, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (e) {
    case 128128: return launch_w<float, 128, 128>(a, st);
    case 128064: return launch_w<float, 128, 64>(a, st);
    case 64128: return launch_w<float, 64, 128>(a, st);
    case 64064: return launch_w<float, 64, 64>(a, st);
    default: return hipErrorInvalidValue;
  }
}

// Groups: as many as keep a thread's loads few (256 Ki outputs, 62 partials: one
// group 12.5 us, 4 and 8 10.7, 16 11.4; 16 Ki outputs, 250 partials: 28, 8.2, 5.3
// and 3.9, 125 partials 15, 5.1, 5.0 and 3.5; 2 Mi outputs, 4 partials: 5.1 with one
// group, 8.5 with 4).
hipError_t launch_add_parts(const float* parts, int P, int64_t outputs, float* D, hipStream_t st) {
  if (!parts || !D || P < 1 || outputs < 4 || outputs % 4 || outputs > (2 << 20))
    return hipErrorInvalidValue;
  return P >= 96 ? launch_add<16>(parts, P, outputs / 4, D, st)
         : P >= 8 ? launch_add<8>(parts, P, outputs / 4, D, st)
                  : launch_add<1>(parts, P, outputs / 4, D, st);
}

hipError_t launch_wgrad_one(int64_t m, int64_t n, int64_t k, float alpha, const void* A,
                            const void* B, int dtype, float* D, hipStream_t st) {
  if (m < 1 || n < 1 || k < 1 || m * n > (2 << 20) || !A || !B || !D) return hipErrorInvalidValue;
  const WgradOneArgs a{A, B, D, k, m, n, alpha};
  return dtype == 1 ? launch_one<bf16>(a, st) : launch_one<float>(a, st);
}

}  // namespace pa
