// Small kernels around the streaming passes (gfx950):
//   - the table image of the backward passes, in the exact byte layout the
//     streaming blocks copy into LDS (rows padded as in pa_layout.h);
//   - the ordered reduction of the per-block partial-sum records (the partial
//     sums of Section 4.2, here over point chunks of one GPU), with the states
//     s_j = num_j / max(den_j, eps) (Eq. 1) formed there.
#include <type_traits>

#include "pa_device.hpp"
#include "pa_internal.h"
#include "pa_layout.h"

namespace pa {

// A per-head batch: head blockIdx.y's tensor at the batch's byte stride.
template <typename Q>
__device__ __forceinline__ Q* head_at(Q* q, int64_t stride) {
  using B = typename std::conditional<std::is_const<Q>::value, const char*, char*>::type;
  return q ? reinterpret_cast<Q*>(reinterpret_cast<B>(q) + (int64_t)blockIdx.y * stride) : q;
}

// ---------------------------------------------------------------------------
// The backward passes' table image: header (biases, dden, centres, shares, a),
// logits table [A^T ; a] and the centred table [dnum - cN | s' - cS].
//
// Bound by latency: a few hundred kilobytes, so every block has one round of
// loads, one reduction and its stores, and the work is spread over M16 + 1 +
// 2C/64 blocks (the form before had two dependent rounds and all of the table
// in 2C/256 blocks: 10 to 12 us per call).
//
// Blocks [0, M16]: row j of the logits table (j = M16: a, and the header's
//   biases, shares and fp32 a), and dden_j (chain rule of Eq. 1; 0 when den_j
//   < eps), reduced over C in a fixed tree.
// The others: 64 columns cc of the backward table (dnum for cc < C, s' beyond),
//   a quarter of the slices per wave, and their centres cN[c], cS[c].
// Any centre common to all slices leaves the softmax backward unchanged; the
// mean weighted by w_j = max(den_j, 0) (the slices' share of the points) keeps
// a slice with a tiny or floored denominator -- whose dnum_j = dS_j /
// max(den_j, eps) can be huge -- from dragging the centre away from the rows
// that carry weight, and keeps the small differences between nearly equal
// rows out of the rounding.  Without the states term den is not given and the
// weights are uniform; kWeightsBwd has neither term (zeros).
// ---------------------------------------------------------------------------
struct PrepGeo {
  int C, M, M16, SZ;  // C: the tables' width (the parameters' cr <= C channels, zeros beyond)
  int TROW, WROW, OFF_L, OFF_2;
};

static PrepGeo prep_geo(int dtype, int C, int M, int MB) {
  PrepGeo g;
  g.C = C; g.M = M; g.M16 = 16 * MB; g.SZ = dtype == 1 ? 2 : 4;
  g.TROW = C * g.SZ + 32;
  g.WROW = 2 * C * g.SZ + 32;
  g.OFF_L = (3 * g.M16 + 3 * C) * 4;  // header: bias, dden, cN, cS, sw, a
  g.OFF_2 = g.OFF_L + (g.M16 + 1) * g.TROW;
  return g;
}

size_t image_bytes(int dtype, int C, int MB) {
  const PrepGeo g = prep_geo(dtype, C, 16 * MB, MB);
  return (size_t)g.OFF_2 + (size_t)g.M16 * g.WROW;
}

// Row j of the logits table, dden_j, and (j = M16) the rest of the header;
// thread t: channel t (C <= 256).
template <typename T>
__device__ __forceinline__ void prep_row(const PrepGeo& g, const PrepArgs& p, int j, float* red) {
  char* img = reinterpret_cast<char*>(p.img);
  float* hdr = reinterpret_cast<float*>(img);
  const T* A = reinterpret_cast<const T*>(p.A);
  const T* av = reinterpret_cast<const T*>(p.a);
  const int C = g.C, M = g.M, M16 = g.M16, cr = p.cr, t = threadIdx.x;
  const bool states = p.dS != nullptr && p.pass == kSliceBwd;
  const bool row = j < M16;
  T v = from_f<T>(0.f);
  if (t < cr) {
    if (row && j < M) v = A[(int64_t)t * M + j];
    if (!row && av) v = av[t];
  }
  if (t < C) {
    *reinterpret_cast<T*>(img + g.OFF_L + lds_off(j, t * g.SZ, g.TROW)) = v;
    if (!row) hdr[3 * M16 + 2 * C + t] = to_f<T>(v);
  }
  if (row) {
    const bool on = states && j < M;
    const float dj = on ? p.den[j] : 1.f;
    float s = on && t < cr ? p.dS[j * cr + t] * (p.num[j * cr + t] / dj) : 0.f;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) s += __shfl_xor(s, o);
    if ((t & 63) == 0) red[t >> 6] = s;
    __syncthreads();
    if (t == 0) {
      const float sum = (red[0] + red[1]) + (red[2] + red[3]);
      hdr[M16 + j] = on && dj >= p.eps ? -sum / dj : 0.f;
      // padded slices j >= M get bias -inf: their softmax weight is exactly 0
      hdr[j] = j < M ? (p.b ? p.b[j] : 0.f) : -INFINITY;
    }
  } else if (t < 64) {
    const float wk = t < M ? (states ? fmaxf(p.den[t], 0.f) : 1.f) : 0.f;
    float wsum = wk;  // fixed-order butterfly over the slices
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) wsum += __shfl_xor(wsum, o);
    if (t < M16) hdr[2 * M16 + 2 * C + t] = wk / wsum;
  }
}

// 64 columns of the backward table: lane l column 64 bid + l, wave w the
// slices [w M16 / 4, (w + 1) M16 / 4).
template <typename T>
__device__ __forceinline__ void prep_columns(const PrepGeo& g, const PrepArgs& p, int bid,
                                             float* red) {
  char* img = reinterpret_cast<char*>(p.img);
  float* hdr = reinterpret_cast<float*>(img);
  const int C = g.C, M = g.M, M16 = g.M16, cr = p.cr;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, per = M16 / 4, j0 = wave * per;
  const bool states = p.dS != nullptr && p.pass == kSliceBwd;
  const bool desl = p.Sp != nullptr && p.pass == kSliceBwd;
  const int cc = 64 * bid + lane;  // (2C is a multiple of 64)
  const bool first = cc < C;
  const int c = first ? cc : cc - C;
  // (columns c >= cr are padding: zero rows, centre 0)
  const bool on = (first ? states : desl) && c < cr;
  const float* src = first ? p.dS : p.Sp;
  float v[16], d[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const bool in = k < per && j0 + k < M;
    const int j = in ? j0 + k : 0;
    v[k] = on && in ? src[j * cr + c] : 0.f;
    d[k] = states && in ? p.den[j] : 1.f;
  }
  float wsum = 0.f, sum = 0.f;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    if (k < per && j0 + k < M) {
      const float w = states ? fmaxf(d[k], 0.f) : 1.f;
      if (first) v[k] *= 1.0f / (d[k] >= p.eps ? d[k] : p.eps);  // dnum_j
      wsum += w;
      sum += w * v[k];
    }
  }
  red[64 * wave + lane] = sum;
  red[256 + 64 * wave + lane] = wsum;
  __syncthreads();
  sum = (red[lane] + red[64 + lane]) + (red[128 + lane] + red[192 + lane]);
  wsum = (red[256 + lane] + red[320 + lane]) + (red[384 + lane] + red[448 + lane]);
  const float ctr = on && wsum > 0.f ? sum * (1.0f / wsum) : 0.f;
  if (wave == 0) hdr[2 * M16 + cc] = ctr;  // cN[c] (cc < C), then cS[c]
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (k < per)
      *reinterpret_cast<T*>(img + g.OFF_2 + lds_off(j0 + k, cc * g.SZ, g.WROW)) =
          from_f<T>(on && j0 + k < M ? v[k] - ctr : 0.f);
}

template <typename T>
__global__ void __launch_bounds__(256) k_prep_back(PrepGeo g, PrepArgs p) {
  __shared__ float red[512];
  if (gridDim.y > 1) {
    p.A = head_at(p.A, p.hs_A);
    p.b = head_at(p.b, p.hs_b);
    p.a = head_at(p.a, p.hs_a);
    p.Sp = head_at(p.Sp, p.hs_Sp);
    p.num = head_at(p.num, p.hs_num);
    p.den = head_at(p.den, p.hs_den);
    p.dS = head_at(p.dS, p.hs_dS);
    p.img = head_at(p.img, p.hs_img);
  }
  if ((int)blockIdx.x <= g.M16)
    prep_row<T>(g, p, blockIdx.x, red);
  else
    prep_columns<T>(g, p, blockIdx.x - g.M16 - 1, red);
}

hipError_t launch_prep_back(const PrepArgs& p, hipStream_t st) {
  if (!p.img || !p.A || (p.pass != kSliceBwd && p.pass != kWeightsBwd)) return hipErrorInvalidValue;
  if (p.cr < 16 || p.cr > p.C || p.cr % 16 || p.C > 256 || p.C % 32) return hipErrorInvalidValue;
  if (p.M < 1 || p.M > 16 * p.MB || p.MB > 4) return hipErrorInvalidValue;
  if (p.pass == kSliceBwd && p.dS && (!p.num || !p.den)) return hipErrorInvalidValue;
  if (p.heads < 1 || p.heads > kMaxHeads) return hipErrorInvalidValue;
  const PrepGeo g = prep_geo(p.dtype, p.C, p.M, p.MB);
  const dim3 grid(g.M16 + 1 + 2 * p.C / 64, p.heads);
  if (p.dtype == 1)
    hipLaunchKernelGGL(k_prep_back<bf16>, grid, dim3(256), 0, st, g, p);
  else
    hipLaunchKernelGGL(k_prep_back<float>, grid, dim3(256), 0, st, g, p);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Ordered reduction of partial records (and the states of Eq. 1)
// ---------------------------------------------------------------------------
// Fixed-order sum of the 16 group sums of one column.
__device__ __forceinline__ float group_total(const double* t16) {
  double t[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) t[q] = t16[2 * q] + t16[2 * q + 1];
  return (float)(((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7])));
}

// Bound by latency (8 MB of records at C = 256, M = 32, one block of kRedCols
// columns per CU): 32 record columns x 16 partial groups per block, each
// thread adding every 16th partial with all of a chunk's loads (256 records)
// issued at once.  (Before, with 16 columns and a loop of batches of 8 whose
// remainder ran load by load: 5 to 7 us per call, most of it the remainder
// for fewer than 128 records.)
constexpr int kRedCols = 32;

// Sum over records pg, pg + 16, .. of one column, in that order.
__device__ __forceinline__ void red_chunk(float (&v)[16], const float* col, int64_t rec, int p0,
                                          int pg, int P) {
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    v[u] = 0.f;
    if (p0 + 16 * u < P) {  // (uniform; records past the end: the last one, not added)
      const int p = p0 + 16 * u + pg;
      v[u] = col[(int64_t)(p < P ? p : P - 1) * rec];
    }
  }
}
__device__ __forceinline__ double red_add(double acc, const float (&v)[16], int p0, int pg, int P) {
#pragma unroll
  for (int u = 0; u < 16; ++u) acc += p0 + 16 * u + pg < P ? (double)v[u] : 0.0;
  return acc;
}

__global__ void __launch_bounds__(16 * kRedCols) k_reduce(const float* __restrict__ parts, int P,
                                                          int64_t rec, Segments seg) {
  // The 16 group sums of a column are added in a fixed tree order.  The sums
  // are formed in fp64: the records are signed partial sums (gradients) whose
  // total can be far smaller than the sum of their magnitudes.  Sixteen
  // numerator columns belong to one slice j (16 divides C): their threads also
  // form den_j, in the same order as den_j's own block, for the states.
  __shared__ double sh[kRedCols][17];
  __shared__ double shd[kRedCols / 16][17];
  // head blockIdx.y of a per-head batch (0 otherwise): its records and
  // destinations at the batch's strides, applied where they are used (the
  // argument struct is only read: writing its arrays would copy it to scratch)
  parts = head_at(parts, seg.hs_parts);
  float* const S = head_at(seg.S, seg.hs_S);
  const int kk = threadIdx.x % kRedCols, pg = threadIdx.x / kRedCols, h = kk / 16;
  const int64_t k0 = (int64_t)blockIdx.x * kRedCols, k = k0 + kk;
  const int64_t kc = k < rec ? k : rec - 1;
  const bool states = S != nullptr && k0 < seg.nS;
  const int64_t kd = states ? seg.den_col + (kc < seg.nS ? kc : seg.nS - 1) / seg.C : 0;
  double acc = 0.0, ad = 0.0;
  for (int p0 = 0; p0 < P; p0 += 256) {
    float v[16], w[16];
    red_chunk(v, parts + kc, rec, p0, pg, P);
    if (states) red_chunk(w, parts + kd, rec, p0, pg, P);
    acc = red_add(acc, v, p0, pg, P);
    if (states) ad = red_add(ad, w, p0, pg, P);
  }
  sh[kk][pg] = acc;
  if (states && kk % 16 == 0) shd[h][pg] = ad;
  __syncthreads();
  if (pg == 0 && k < rec) {
    const float tot = group_total(sh[kk]);
    int64_t off = k;
    for (int i = 0; i < seg.n; ++i) {
      if (off < seg.len[i]) {
        if (seg.dst[i]) head_at(seg.dst[i], seg.hs_dst[i])[off] = tot;
        if (seg.dst2[i]) head_at(seg.dst2[i], seg.hs_dst2[i])[off] = tot;
        break;
      }
      off -= seg.len[i];
    }
    if (states && k < seg.nS) {
      const float den = group_total(shd[h]);
      S[k] = tot / (den >= seg.eps ? den : seg.eps);
    }
  }
}

hipError_t launch_reduce(const float* partials, int P, int64_t rec, const Segments& seg,
                         hipStream_t st) {
  if (!partials || P < 1 || rec < 1) return hipErrorInvalidValue;
  if (seg.S && (seg.C < 16 || seg.C % 16 || seg.nS > rec || seg.den_col < 0 ||
                seg.den_col + seg.nS / seg.C > rec))
    return hipErrorInvalidValue;
  const int heads = seg.heads > 1 ? seg.heads : 1;
  if (heads > kMaxHeads) return hipErrorInvalidValue;
  const int blocks = (int)((rec + kRedCols - 1) / kRedCols);
  hipLaunchKernelGGL(k_reduce, dim3(blocks, heads), dim3(16 * kRedCols), 0, st, partials, P, rec, seg);
  return hipGetLastError();
}

}  // namespace pa
