// The forward tables of the streaming passes (gfx950), built in LDS by every
// block at its start from the call's parameters and states: the biases, the
// logits table [A^T ; a] and the deslice table S'^T, in the byte layout of
// pa_layout.h.
//
// They are small (16 KB of A, 32 KB of S' at C = 256, M = 32) and come from L2
// after the first block; all of a thread's loads (up to a batch of registers)
// are issued before its LDS writes, so a table costs a block about one memory
// round trip, as copying a finished image from the workspace did, without the
// kernel that wrote the image before every pass (3 to 5 us per call: forward
// at N = 4096, fp32 44 -> 41 us, N = 100,003 47 -> 43 us).  The backward's
// tables need sums over all states and over all channels first; built by
// every block they measured slower than one kernel and a copy (N = 16,384,
// fp32, M = 64: step 197 -> 210 us; per-head slicing at N = 1M 1234 -> 1250
// us), so those come from k_prep_back (pa_small.hip).
#pragma once

#include "pa_device.hpp"
#include "pa_layout.h"

namespace pa {

// What the tables are built from (device pointers; NULL where a pass has none).
struct TableSrc {
  const void* A;     // [cr, M] dtype
  const float* b;    // [M], nullable
  const void* a;     // [cr] dtype, nullable
  const float* Sp;   // [M, cr]
};

// f(q) for q = thread, thread + THREADS, .. < N in batches of B: ld(q) of a
// whole batch before st(q, value) of it (past the end: the last item again,
// the same bytes to the same place).
template <int B, int N, int THREADS, typename V, typename Ld, typename St>
__device__ __forceinline__ void batched(Ld&& ld, St&& st) {
  constexpr int PER = (N + THREADS - 1) / THREADS;
#pragma unroll
  for (int u0 = 0; u0 < PER; u0 += B) {
    V v[B];
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (u0 + u < PER) {
        const int q = (int)threadIdx.x + (u0 + u) * THREADS;
        v[u] = ld(q < N ? q : N - 1);
      }
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (u0 + u < PER) {
        const int q = (int)threadIdx.x + (u0 + u) * THREADS;
        st(q < N ? q : N - 1, v[u]);
      }
  }
}

// Logits table: rows j < M16: A[:, j] (0 for j >= M and for columns c >= cr);
// row M16: a (0 without).  Biases: b_j, -inf for the padded slices j >= M, so
// that their softmax weight is exactly 0.
template <typename T, int C, int MB, int THREADS>
__device__ __forceinline__ void build_logits(char* smem, const TableSrc& s, int M, int cr) {
  using G_ = Geo<sizeof(T), C, MB>;
  constexpr int M16 = G_::M16, SZ = (int)sizeof(T), E = 16 / SZ;
  const T* A = reinterpret_cast<const T*>(s.A);
  const T* av = reinterpret_cast<const T*>(s.a);
  float* hdr = reinterpret_cast<float*>(smem);
  char* tab = smem + G_::OFF_L;
  for (int j = threadIdx.x; j < M16; j += THREADS)
    hdr[j] = j < M ? (s.b ? s.b[j] : 0.f) : -INFINITY;
  for (int c = threadIdx.x; c < C; c += THREADS)
    *reinterpret_cast<T*>(tab + M16 * G_::TROW + c * SZ) =
        av && c < cr ? av[c] : from_f<T>(0.f);
  if (M == M16 && cr == C) {
    // whole 16-byte chunks of A's rows: E slices of one channel
    struct Chunk { T v[E]; };
    batched<8, C * M16 / E, THREADS, uint4>(
        [&](int q) { return reinterpret_cast<const uint4*>(A)[q]; },
        [&](int q, const uint4& x) {
          const Chunk k = __builtin_bit_cast(Chunk, x);
          const int c = q / (M16 / E), j = q % (M16 / E) * E;
#pragma unroll
          for (int e = 0; e < E; ++e)
            *reinterpret_cast<T*>(tab + (j + e) * G_::TROW + c * SZ) = k.v[e];
        });
  } else {
    // padded rows or columns: element by element, consecutive threads on
    // consecutive slices of a channel
    batched<16, C * M16, THREADS, T>(
        [&](int q) {
          const int c = q / M16, j = q % M16;
          const bool in = c < cr && j < M;
          const T v = A[in ? c * M + j : 0];
          return in ? v : from_f<T>(0.f);
        },
        [&](int q, const T& v) {
          *reinterpret_cast<T*>(tab + (q % M16) * G_::TROW + (q / M16) * SZ) = v;
        });
  }
}

// Deslice table S'^T at tab: row c, column j (0 for j >= M, c >= cr).
template <typename T, int C, int MB, int THREADS>
__device__ __forceinline__ void build_deslice(char* tab, const TableSrc& s, int M, int cr) {
  using G_ = Geo<sizeof(T), C, MB>;
  constexpr int M16 = G_::M16, SZ = (int)sizeof(T);
  batched<8, C * M16 / 4, THREADS, f32x4>(
      [&](int q) {
        const int c = q % C, j = 4 * (q / C);
        f32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool in = c < cr && j + i < M;
          const float x = s.Sp[in ? (j + i) * cr + c : 0];
          v[i] = in ? x : 0.f;
        }
        return v;
      },
      [&](int q, const f32x4& v) {
        T* d = reinterpret_cast<T*>(tab + (q % C) * G_::SROW + 4 * (q / C) * SZ);
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = from_f<T>(v[i]);
      });
}

}  // namespace pa
