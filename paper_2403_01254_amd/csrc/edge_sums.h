// The per-edge sums of the normal equations: their layout, their reduction from the finalisation's per-block
// partial sums, and their expansion into an edge's 93 values.
#pragma once

#include "block_sort.h"

namespace rkhsba {

// Slots of the per-point products summed per edge (finalisation, pairs.hip).
constexpr int kStA = 0, kStB = 1, kStXBm = 4, kStQB = 7, kStAx = 10, kStAxx = 13, kStAq = 19, kStSzz = 22,
              kStXS = 28, kStWr2 = 37, kStF = 38, kStCnt = 39;

// Running sums: FP64, or FP32 with Kahan compensation (option).
template <typename T>
struct Acc;
template <>
struct Acc<double> {
  double s = 0.0;
  __device__ void add(double v) { s += v; }
  __device__ double value() const { return s; }
};
template <>
struct Acc<float> {
  float s = 0.f, c = 0.f;
  __device__ void add(float v) {
    const float y = v - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
  }
  __device__ float value() const { return s; }
};

// Sums N values over the wavefront, the values spread over the lanes as they are summed: at every step a lane
// keeps one half of its values and hands the other half to the lane o away, so that N values take about N + 6
// exchanges where one butterfly per value takes 6 N.  The additions pair the same lanes in the same order as
// wave_sum's (lanes 32 apart first).  Returns the index of the value whose sum v[0] holds in this lane, or N for
// none (an odd count leaves the upper half of the lanes one value short).
template <int N, typename T>
__device__ __forceinline__ int wave_sum_spread(T (&v)[N]) {
  const int lane = threadIdx.x & 63;
  int idx = 0, held = N;  // this lane's values: idx .. idx + held - 1
  int n = N;              // the most that a lane holds (compile-time after unrolling)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int h = (n + 1) / 2;
    const bool hi = (lane & o) != 0;
#pragma unroll
    for (int k = 0; k < (N + 1) / 2; ++k) {
      if (k >= h) continue;
      const T a = v[k];
      const T b = k + h < n ? v[k + h < N ? k + h : 0] : (T)0;
      v[k] = (hi ? b : a) + __shfl_xor(hi ? a : b, o, 64);
    }
    idx += hi ? h : 0;
    held = hi ? max(held - h, 0) : min(held, h);
    n = h;
  }
  return held > 0 ? idx : N;
}

__device__ __forceinline__ void sym_row_col(int k, int& r, int& c) {  // k-th entry of a 6x6 upper triangle, row-major
  r = 0;
  int len = 6;
  while (k >= len) {
    k -= len;
    --len;
    ++r;
  }
  c = r + k;
}

// Entry (i, j) of the cross-product matrix of a.
template <typename T>
__device__ __forceinline__ T skew_at(const T* a, int i, int j) {
  if (i == j) return (T)0;
  const T v = a[3 - i - j];
  return (j - i + 3) % 3 == 1 ? -v : v;
}

// Value k of an edge (F, b_m, b_n, H_mm, H_nn, H_mn, pairs, sum w r^2; kEdgeVals) from its sums T.  The fused
// multiply-adds are written out: a solve in a direction that the view leaves nearly free multiplies the last bits of H
// and b by 1e8, so their rounding is part of the results and is not left to the compiler.
template <typename TT>
__device__ __forceinline__ double edge_value(const TT* T, const EdgeXf& X, double n_pairs, int k) {
  auto Rmn = [&](int r, int c) { return (TT)X.R[3 * c + r]; };
  const TT A = T[kStA];
  const TT* B = T + kStB;
  // row r of R_mn times a vector
  auto Rmn_dot = [&](int r, TT v0, TT v1, TT v2) { return fma(Rmn(r, 2), v2, fma(Rmn(r, 0), v0, Rmn(r, 1) * v1)); };
  if (k == 0) return (double)T[kStF];
  if (k < 4) return (double)Rmn_dot(k - 1, B[0], B[1], B[2]);
  if (k < 7) return (double)T[kStXBm + k - 4];
  if (k < 10) return (double)-B[k - 7];
  if (k < 13) return (double)-T[kStQB + k - 10];
  if (k == 91) return n_pairs;
  if (k == 92) return (double)T[kStWr2];
  TT S[3];
  for (int i = 0; i < 3; ++i) S[i] = T[kStAq + i] - B[i];
  if (k < 55) {  // H_mm or H_nn: [[A I, -[a]], [[a], tr(Q) I - Q]]
    const bool mm = k < 34;
    const TT* Q = T + (mm ? kStAxx : kStSzz);  // xx, xy, xz, yy, yz, zz
    int r, c;
    sym_row_col(k - (mm ? 13 : 34), r, c);
    if (c < 3) return (double)(r == c ? A : (TT)0);
    if (r < 3) return (double)-(mm ? skew_at(T + kStAx, r, c - 3) : skew_at(S, r, c - 3));
    r -= 3; c -= 3;
    const TT tr = Q[0] + Q[3] + Q[5];
    return (double)((r == c ? tr : (TT)0) - Q[r == 0 ? c : r + c + 1]);
  }
  // H_mn: [[-A R_mn, R_mn [S]], [-[A x] R_mn, sum [x] R_mn [S]]]
  const int r = (k - 55) / 6, c = (k - 55) % 6;
  if (r < 3 && c < 3) return (double)(-A * Rmn(r, c));
  if (r < 3) return (double)Rmn_dot(r, skew_at(S, 0, c - 3), skew_at(S, 1, c - 3), skew_at(S, 2, c - 3));
  TT v = 0;
  if (c < 3) {
    for (int a = 0; a < 3; ++a) v = fma(skew_at(T + kStAx, r - 3, a), Rmn(a, c), v);
    return (double)-v;
  }
  // sum_p [x_p] R_mn [S_p]: the sums of x_i S_j under the two cross products' signs
  for (int a = 2; a >= 0; --a)
    for (int b = 2; b >= 0; --b) {
      const int rr = r - 3, cc = c - 3;
      if (a == rr || b == cc) continue;
      const TT m = T[kStXS + 3 * (3 - rr - a) + (3 - b - cc)];
      const bool neg = ((a - rr + 3) % 3 == 1) != ((cc - b + 3) % 3 == 1);
      v = fma(neg ? -m : m, Rmn(a, b), v);
    }
  return (double)v;
}

template <typename TT>
struct EdgeSums {  // LDS of one wavefront
  TT T[kFinStats];
  double n_pairs;
};

// One wavefront: the edge's sums over its finalisation blocks in block order, expanded into out[kEdgeVals].  The
// values are spread over the lanes: one thread wrote all 93 of them before, 10 us of serial FP64 for 28 edges that
// now take 3.  (Inlined by force, with its helpers, as all that take LDS: block_sort.h.)
template <typename TT>
__device__ __forceinline__ void reduce_edge(const double* __restrict__ partial, const EdgeInfo& ed, const EdgeXf& X,
                                            int mode, EdgeSums<TT>& sh, double* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int ns = mode == MODE_LOSS ? 2 : kFinStats;
  const double* p = partial + (int64_t)ed.fin_off * kFinStats + lane;
  if (lane < kFinStats) {
    // 16 blocks' values in flight at a time, added in block order
    constexpr int U = 16;
    const bool count = lane == ns - 1;  // the pair counts, summed in FP64
    Acc<TT> s;
    double c = 0.0;
    if (lane < ns)
      for (int b = 0; b < ed.n_fin; b += U) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = b + u < ed.n_fin ? p[(int64_t)(b + u) * kFinStats] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (b + u < ed.n_fin) {
            if (count) c += v[u];
            else s.add((TT)v[u]);
          }
      }
    if (count) sh.n_pairs = c;
    sh.T[lane] = count ? (TT)0 : s.value();
  }
  wave_sync();
  for (int k = lane; k < kEdgeVals; k += 64)
    out[k] = mode != MODE_LOSS ? edge_value(sh.T, X, sh.n_pairs, k)  // (sum w r^2 needs the moments)
                               : k == 0 ? (double)sh.T[0] : k == 91 ? sh.n_pairs : 0.0;
  wave_sync();
}

}  // namespace rkhsba
