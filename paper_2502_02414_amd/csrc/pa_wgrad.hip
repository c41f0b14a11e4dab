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
// Measured, with the reduction, against strided-batched library products with
// the same split: 1024 x 256 at k = 500,000 457 -> 354 us (the kernel alone
// 260 us from idle, 4.9 TB/s; the clock falls under a run of such products),
// k = 33,000 (one library product) 119 -> 46 us; 512 x 128 at k = 500,000
// 237 -> 137 us; 256 x 64 170 -> 65 us.  HBM reads: the operands, once.
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

// Tile edge along a dimension (a multiple of 64): the largest of 256, 128, 64
// up to cap that divides it.
int edge(int64_t v, int cap) {
  return cap >= 256 && v % 256 == 0 ? 256 : cap >= 128 && v % 128 == 0 ? 128 : 64;
}
int64_t tiles_of(int64_t m, int64_t n, int cap) { return (m / edge(m, cap)) * (n / edge(n, cap)); }

// At most 128 in fp32 (the matrix cores bind it at any tile) and for up to
// kShortK points in bf16, where blocks of four times as many smaller tiles fill
// the chip sooner and leave fewer partials (1024 x 256: k = 8,000 28 us against
// 39 us, k = 33,000 46 us against 58 us, k = 131,072 140 us against 115 us).
constexpr int64_t kShortK = 98304;
int largest_edge(int64_t k, int dtype) { return dtype == 1 && k > kShortK ? 256 : 128; }

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
// 1.9, 1.3, 0.52 and 0.34 ms (256 x 256 tiles alone, and with half of the
// workspace: 12.0, 12.0, 6.1, 1.6 and 0.48 ms).  Below four partials the
// product in one piece is faster (two: 2.5 ms against 1.9 ms; four: 1.3 ms)
// unless larger tiles fill half of the CUs (1024 x 2048 at k = 100,000, 128
// blocks: 1.2 ms against 1.6 ms).
WgradPlan wgrad_plan(int64_t m, int64_t n, int64_t k, int dtype, int64_t most) {
  WgradPlan w{largest_edge(k, dtype), 0, true};
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

// Whole 64 x 64 tiles, and lengths at which this kernel measured faster than
// the library product.  Outputs of up to 128 Ki elements (512 x 128): from k
// = 512 (14 us against 21 us); larger ones (1024 x 256): from 4,096 in bf16
// (k = 2,001 24 us against 21 us, 8,000 28 us against 36 us) and 16,384 in
// fp32 (8,000 60 us against 52 us, 33,000 165 us against 233 us).  fp32 from
// 2^17 points stays with the split library products (1024 x 256 at 131,072:
// 574 us against 528 us), whose partial sums are also shorter there.
bool wgrad_served(int64_t m, int64_t n, int64_t k, int dtype) {
  if (m < 64 || n < 64 || m % 64 != 0 || n % 64 != 0 || m * n > (2 << 20)) return false;
  if (m * n <= (1 << 17)) return k >= 512 && (dtype == 1 || k < (1 << 17));
  return dtype == 1 ? k >= 4096 : k >= 16384 && k < (1 << 17);
}

hipError_t launch_wgrad(int64_t m, int64_t n, int64_t k, float alpha, const void* A,
                        const void* B, int dtype, float* out, const WgradPlan& w,
                        hipStream_t st) {
  if (!wgrad_served(m, n, k, dtype) || w.P < 1 || w.P > (k + 31) / 32 || !A || !B || !out)
    return hipErrorInvalidValue;
  const WgradArgs a{A, B, out, k, (int)m, (int)n, w.P, alpha};
  const int e = edge(m, w.cap) * 1000 + edge(n, w.cap);
  if (dtype == 1) {
    switch (e) {
      case 256256: return launch_w<bf16, 256, 256>(a, st);
      case 256128: return launch_w<bf16, 256, 128>(a, st);
      case 256064: return launch_w<bf16, 256, 64>(a, st);
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

hipError_t launch_wgrad_one(int64_t m, int64_t n, int64_t k, float alpha, const void* A,
                            const void* B, int dtype, float* D, hipStream_t st) {
  if (m < 1 || n < 1 || k < 1 || m * n > (2 << 20) || !A || !B || !D) return hipErrorInvalidValue;
  const WgradOneArgs a{A, B, D, k, m, n, alpha};
  return dtype == 1 ? launch_one<bf16>(a, st) : launch_one<float>(a, st);
}

}  // namespace pa
