// Element-wide pieces of the matrix-core operator (N >= 5), shared by its
// kernels and the resident CG: the element's shape and LDS layout, the
// fragments of the derivative matrix, the contractions of a 16-column tile and
// the metric of a straight-edged element.
#pragma once

#include "common.hpp"
#include "mfma_16x16x4.hpp"

namespace sem {

// Wavefronts per element and waves per SIMD (register budget) by order and
// bytes of T.  The waves are the most that do not spill (a spill of ten
// registers costs 40-80 % here: N = 9 FP64 at five waves 173 us against 97 at
// three), few wavefronts of several points each beat many of one (N = 5: one
// wavefront per element 87 us, four 122 us), and with the budget stated the
// results of the products stay out of the accumulation registers, from which
// each would be moved.
constexpr int ax_waves(int N, int bytes) {
  return N == 5 ? 1 : N == 6 ? (bytes == 8 ? 2 : 3) : N == 10 ? 8 : 4;
}
constexpr int ax_min_waves(int N, int bytes, int geo) {
  if (geo) return N == 7 ? 5 : N == 5 || N == 9 ? 3 : 4;
  return bytes == 8 ? (N == 5 || N == 9 ? 3 : N == 7 ? 6 : 4)
                    : (N == 5 || N == 9 ? 5 : N == 6 || N == 7 ? 8 : 7);
}
// Shape of the operator kernel: NW wavefronts per element, each lane with the
// points t, t + 64 NW, ... (coalesced factor loads at every order).
template <int N, typename T>
struct LShape {
  static constexpr int n1 = N + 1;
  static constexpr int P2 = n1 * n1;
  static constexpr int P = P2 * n1;
  static constexpr int NW = ax_waves(N, sizeof(T));
  static constexpr int TPB = 64 * NW;
  static constexpr int PPT = (P + TPB - 1) / TPB;    // points per lane
  static constexpr int NT = (P2 + 15) / 16;          // 16-column tiles per direction
  static constexpr int TPW = (NT + NW - 1) / NW;     // tiles per wavefront and direction
  static constexpr int KS = (n1 + 3) / 4;            // products per tile
  static constexpr int LS = n1 == 8 ? 9 : n1;        // LDS row stride (n1 = 8: 16 rows of 8
                                                     // would meet in a quarter of the banks)
  static constexpr int PS = n1 * LS;                 // LDS layer stride
};

// LDS place of point q of the element
template <int N, typename T>
__device__ __forceinline__ int lds_point(int q) {
  using S = LShape<N, T>;
  return S::LS == S::n1 ? q : (q / S::n1) * S::LS + q % S::n1;
}

// Fragments of D (forward) and D^T.  In both precisions the row of result r in
// lane group kk is kk + 4 r, and step s contracts the columns kk + 4 s, so
// every lane has KS result rows (FP32 results of 16x16x4 products come in rows
// 4 kk + r, so the rows of the operand are taken in that order).
// BLK (FP64): products of four 4x4x4 blocks, whose blocks are the four column
// groups of a tile (A[i][k] of every block in lane i + 4 b + 16 k, B[k][j] and
// the result's row k, column 4 b + j in lane 16 k + 4 b + j): KS x KS of them
// cover 4 KS rows, where the 16x16x4 form always computes 16 (N = 7: 8 used) at
// the same rate.  The straight-edged operator, which computes more than it
// streams, gains by them (8 million points, N = 7: 73 -> 64 us); the streaming
// one loses by their larger number (82 -> 87 us).
template <int N, typename T, bool BLK>
struct DFrag {
  static_assert(!BLK || sizeof(T) == 8, "4x4x4 blocks are FP64");
  static constexpr int n1 = N + 1, KS = LShape<N, T>::KS, R = BLK ? KS : 1;
  T m[R][KS];
  DFrag() = default;
  __device__ __forceinline__ DFrag(const T* __restrict__ D, int lane, bool trans) {
    const int i = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = BLK ? 4 * r + (i & 3) : sizeof(T) == 8 ? i : (i >> 2) + 4 * (i & 3);
      const int rc = min(row, n1 - 1);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int l = 4 * s + kk, lc = min(l, n1 - 1);
        const T v = trans ? D[lc * n1 + rc] : D[rc * n1 + lc];
        m[r][s] = row < n1 && l < n1 ? v : T(0);
      }
    }
  }
  // out[r] = rows kk + 4 r of the matrix times the tile with operands x[s]
  __device__ __forceinline__ void mul(const T (&x)[KS], T (&out)[KS]) const {
    if constexpr (BLK) {
#pragma unroll
      for (int r = 0; r < KS; ++r) out[r] = 0.0;
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int r = 0; r < KS; ++r)
          out[r] = __builtin_amdgcn_mfma_f64_4x4x4f64(m[r][s], x[s], out[r], 0, 0, 0);
    } else {
      typename Mm<T>::V acc = {T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int s = 0; s < KS; ++s) acc = Mm<T>::mma(m[0][s], x[s], acc);
#pragma unroll
      for (int r = 0; r < KS; ++r) out[r] = acc[r];
    }
  }
};

// The three contractions of one 16-column tile: along i from si, along j
// from sj, along k from sk (element blocks in LDS), results to ri, rj, rk at
// the same lines (in place allowed).  No access but the last rows' stores is
// predicated: columns past the last one repeat it (the same values to the same
// places) and contraction indices past n1 repeat the last one against zero
// fragments.
template <int N, typename T, bool BLK>
__device__ __forceinline__ void contract_tile(int tile, int lane, const DFrag<N, T, BLK>& m,
                                              const T* si, const T* sj, const T* sk, T* ri,
                                              T* rj, T* rk) {
  using S = LShape<N, T>;
  constexpr int n1 = S::n1, KS = S::KS, LS = S::LS, PS = S::PS;
  const int kk = lane >> 4;
  const int col = min(tile * 16 + (lane & 15), S::P2 - 1);
  const int cq = col / n1, cr = col % n1;
  const int bi = cq * PS + cr * LS, bj = cq * PS + cr, bk = cq * LS + cr;
  T xi[KS], xj[KS], xk[KS], ai[KS], aj[KS], ak[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int l = 4 * s + 3 < n1 ? kk + 4 * s : min(kk + 4 * s, n1 - 1);
    xi[s] = si[bi + l];
    xj[s] = sj[bj + l * LS];
    xk[s] = sk[bk + l * PS];
  }
  m.mul(xi, ai);
  m.mul(xj, aj);
  m.mul(xk, ak);
#pragma unroll
  for (int r = 0; r < KS; ++r) {
    const int row = kk + 4 * r;
    if (4 * r + 3 < n1 || row < n1) {
      ri[bi + row] = ai[r];
      rj[bj + row * LS] = aj[r];
      rk[bk + row * PS] = ak[r];
    }
  }
}

// Metric of a straight-edged element (the trilinear image of its corners) at
// the point (r, s, t) with quadrature weight wq, from the element's seven
// coefficient vectors c = (x_r, x_s, x_t, x_rs, x_rt, x_st, x_rst): g =
// (rr, rs, rt, ss, st, tt) as stored factors hold them, and B.  In FP64 also
// where the operator runs in FP32, so that its factors round as the stored ones.
typedef const double __attribute__((address_space(4))) * UniformD;  // read by scalar loads
__device__ __forceinline__ void straight_metric(UniformD c, double r, double s, double t,
                                                double wq, double (&g)[6], double& B) {
  double xr[3], xs[3], xt[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double rs = c[9 + d], rt = c[12 + d], st = c[15 + d], rst = c[18 + d];
    const double a = st + rst * r;
    xr[d] = (c[d] + rs * s) + (rt + rst * s) * t;
    xs[d] = (c[3 + d] + rs * r) + a * t;
    xt[d] = (c[6 + d] + rt * r) + a * s;
  }
  double A[3][3];  // detJ grad r, grad s, grad t
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int e = (d + 1) % 3, f = (d + 2) % 3;
    A[0][d] = xs[e] * xt[f] - xs[f] * xt[e];
    A[1][d] = xt[e] * xr[f] - xt[f] * xr[e];
    A[2][d] = xr[e] * xs[f] - xr[f] * xs[e];
  }
  const double det = xr[0] * A[0][0] + xr[1] * A[0][1] + xr[2] * A[0][2];
  // 1 / det by two Newton steps on the hardware's estimate (a full division
  // also handles what a determinant checked positive cannot be)
  double rd = __builtin_amdgcn_rcp(det);
  rd = rd * (2.0 - det * rd);
  rd = rd * (2.0 - det * rd);
  const double sc = wq * rd;
  B = wq * det;
  g[0] = sc * (A[0][0] * A[0][0] + A[0][1] * A[0][1] + A[0][2] * A[0][2]);
  g[1] = sc * (A[0][0] * A[1][0] + A[0][1] * A[1][1] + A[0][2] * A[1][2]);
  g[2] = sc * (A[0][0] * A[2][0] + A[0][1] * A[2][1] + A[0][2] * A[2][2]);
  g[3] = sc * (A[1][0] * A[1][0] + A[1][1] * A[1][1] + A[1][2] * A[1][2]);
  g[4] = sc * (A[1][0] * A[2][0] + A[1][1] * A[2][1] + A[1][2] * A[2][2]);
  g[5] = sc * (A[2][0] * A[2][0] + A[2][1] * A[2][1] + A[2][2] * A[2][2]);
}

}  // namespace sem
