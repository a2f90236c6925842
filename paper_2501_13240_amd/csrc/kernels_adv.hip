// Convective term C_e(u) f on every element (the advection terms of the
// Boussinesq equations, Sec. 4.1).
//
// Over-integrated rule (M = floor(3(N+1)/2) Gauss points per direction):
//   1. each velocity component u_d is interpolated to the M^3 points,
//      (J x J x J) u_d, and folded into V_a = sum_d G_ad u_d (a = r, s, t);
//      the nine factors G_ad = w detJ dr_a/dx_d are streamed from HBM once;
//   2. the reference derivatives of f at the points, (J x J x JD) f,
//      (J x JD x J) f and (JD x J x J) f with JD = J D, give
//      c = sum_a V_a df/dr_a;
//   3. the test functions project back: out = (J^T x J^T x J^T) c.
// The factors at the set-up come from the same stages of the coordinates, as
// batches of 16-column tiles of 16x16x4 MFMA products.
//
// Collocation (the GLL nodes themselves): one thread per node, derivative
// sums over LDS.
#include <type_traits>

#include "advection.hpp"
#include "ax_tiles.hpp"

namespace sem {
namespace {

// dst = A src along direction DIR of an [S2][S1][S0] array (index 0
// fastest); the extent along DIR changes from NI to NO.  A is NO x NI,
// passed as this lane's fragments a[s] = A[lane % 16][4 s + lane / 16].
// The columns of the product are the points of the other two directions,
// in storage order.
template <typename T, int S2, int S1, int S0, int NO, int DIR>
struct Ct {
  typedef typename Mm<T>::V V;
  static constexpr int NI = DIR == 0 ? S0 : DIR == 1 ? S1 : S2;
  static constexpr int NC = S2 * S1 * S0 / NI;
  static constexpr int NT = (NC + 15) / 16;
  static constexpr int KS = (NI + 3) / 4;
  static_assert(NI <= 16 && NO <= 16, "one MFMA tile per matrix");
  // address of (column c, index l along DIR) with extent L along DIR
  template <int L>
  static __device__ __forceinline__ int addr(int c, int l) {
    if constexpr (DIR == 0) return c * L + l;
    else if constexpr (DIR == 1) return (c / S0) * (L * S0) + l * S0 + c % S0;
    else return l * (S1 * S0) + c;
  }
  static __device__ __forceinline__ V tile(const T* __restrict__ src, const T* a, int t,
                                           int lane) {
    const int col = t * 16 + (lane & 15);
    const bool cv = col < NC;
    const int kk = lane >> 4;
    V acc = {T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int l = 4 * s + kk;
      const T b = (cv && l < NI) ? src[addr<NI>(cv ? col : 0, l)] : T(0);
      acc = Mm<T>::mma(a[s], b, acc);
    }
    return acc;
  }
  static __device__ __forceinline__ void store(T* __restrict__ dst, V acc, int t, int lane) {
    const int col = t * 16 + (lane & 15);
    if (col >= NC) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = Mm<T>::row(lane, r);
      if (row < NO) dst[addr<NO>(col, row)] = acc[r];
    }
  }
};

// this lane's fragments of the NO x NI row-major matrix A
template <typename T, int NO, int NI>
__device__ __forceinline__ void fragments(const T* __restrict__ A, T* a, int lane) {
  constexpr int KS = (NI + 3) / 4;
  const int row = lane & 15;
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int l = 4 * s + (lane >> 4);
    a[s] = (row < NO && l < NI) ? A[row * NI + l] : T(0);
  }
}

constexpr int kAdvWaves = 4;
constexpr int kAdvThreads = 64 * kAdvWaves;

// The interpolation stages of an order-N element to M points per direction.
template <int N, int M, typename T>
struct Stages {
  static constexpr int n = N + 1, P = n * n * n, Q = M * M * M;
  typedef Ct<T, n, n, n, M, 0> I0;  // (n,n,n) -> (n,n,M)
  typedef Ct<T, n, n, M, M, 1> I1;  // (n,n,M) -> (n,M,M)
  typedef Ct<T, n, M, M, M, 2> I2;  // (n,M,M) -> (M,M,M)
  static constexpr int KN = I0::KS;
  // LDS: the input block and the two first-stage outputs (later the M^3
  // array c and the (n,n,M) back-projection stage), and one (n,M,M) array
  static constexpr int IX = P + 2 * n * n * M;
  static constexpr int YS = n * M * M;
  static_assert(Q <= IX && P <= YS, "LDS regions");
};

// ------------------------------------------------- the over-integrated rule

// One 1-D transform y = A x of a line held in registers, A (NO x NI) with
// A[NO-1-i][NI-1-j] = A[i][j] (interpolation, projection) or = -A[i][j] (ANTI,
// differentiation, whose rows also sum to zero): the mirror symmetry of the
// nodes.  With the even and odd parts e_j = x_j + x_{NI-1-j}, o_j = x_j -
// x_{NI-1-j}, half of the outputs are a + b and the mirrored ones a - b (ANTI:
// b - a), a = ce e, b = co o: 68 operations for 8 -> 12 points instead of 96.
// ANTI takes the e_j less the innermost one, so a constant line gives exact
// zeros and one product per output goes.
//
// The coefficients, row by row (HI of ce, NI / 2 of co), are uniform over the
// wavefront and come through scalar registers, which cannot hold a matrix:
// each chunk of rows is requested while the one before it is used (left to the
// compiler's order, which waits for each: four FP64 fields on the 32x32x16, N =
// 7 box 1081 against 640 us).
template <int NI, int NO, bool ANTI, typename T>
struct Eo {
  static constexpr int HI = (NI + 1) / 2, NH = NI / 2, HO = (NO + 1) / 2, SZ = HO * NI;
  static constexpr int kRow = NI * (int)sizeof(T) / 4;            // scalar registers per row
  // rows per chunk: about 32 registers; single rows measured faster at rows of
  // 12 and 18 (four FP64 fields: N = 5 361 -> 318 us, N = 8 379 -> 331 us, where
  // N = 7 and N = 9 lose 8-11 % by them)
  static constexpr int RC = kRow >= 24 || kRow == 12 || kRow == 18 ? 1 : kRow >= 12 ? 2 : 4;
  static constexpr int NC = (HO + RC - 1) / RC;
  T e[HI], o[NH == 0 ? 1 : NH];
  template <typename F>
  __device__ __forceinline__ explicit Eo(F&& x) {
#pragma unroll
    for (int j = 0; j < NH; ++j) {
      const T p = x(j), q = x(NI - 1 - j);
      e[j] = p + q;
      o[j] = p - q;
    }
    if constexpr (NI & 1) e[NH] = x(NH);
    if constexpr (ANTI) {
      const T c = (NI & 1) ? e[NH] + e[NH] : e[HI - 1];
#pragma unroll
      for (int j = 0; j < HI - 1; ++j) e[j] -= c;
    }
  }
  template <typename F>
  __device__ __forceinline__ void apply(const T* __restrict__ coef, F&& put) const {
    typedef const T __attribute__((address_space(4))) * Uniform;  // read by scalar loads
    int anew = 0;
    asm volatile("" : "+s"(anew));  // for every line: the reads are not kept over the kernel
    Uniform c = (Uniform)(uintptr_t)coef + anew;
    T buf[2][RC * NI];
    auto fetch = [&](int k) {
#pragma unroll
      for (int x = 0; x < RC * NI; ++x)
        if (k * RC * NI + x < SZ) buf[k & 1][x] = c[k * RC * NI + x];
    };
    fetch(0);
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (k + 1 < NC) fetch(k + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < RC; ++r) {
        const int i = k * RC + r;
        if (i >= HO) break;
        const T* row = buf[k & 1] + r * NI;
        constexpr int ne = ANTI ? HI - 1 : HI;
        const bool mid = (NO & 1) && i == HO - 1;
        T a = T(0), b = T(0);
        if (!(mid && ANTI))
#pragma unroll
          for (int j = 0; j < ne; ++j) a = j == 0 ? row[j] * e[j] : a + row[j] * e[j];
        if (!(mid && !ANTI))
#pragma unroll
          for (int j = 0; j < NH; ++j) b = j == 0 ? row[HI + j] * o[j] : b + row[HI + j] * o[j];
        if (mid) {
          put(i, ANTI ? b : a);
        } else {
          put(i, a + b);
          put(NO - 1 - i, ANTI ? b - a : a - b);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// Shape of the dealiased kernel: n nodes and M points per direction.
template <int N, typename T>
struct AdvShape {
  static constexpr int n = N + 1, M = (3 * n) / 2, P = n * n * n, Q = M * M * M;
  static constexpr int n2 = n * n, nM = n * M, M2 = M * M;
  static constexpr int TPB = ((M2 + 63) / 64) * 64;
  // LDS rows (k, jq) of n or M values along i, an odd number apart (a line per
  // lane then meets every bank)
  static constexpr int SA = n | 1, SY = M | 1;
  static constexpr int A = nM * SA, Y = nM * SY;
  // three line arrays at once (u components, derivative directions) up to 40
  // KB, else one after another, with more barriers and more workgroups per CU
  // (four fields, FP64: N = 6, 30 KB, 364 against 402 us; N = 7, 51 KB, 399
  // against 363 us)
  static constexpr int NY = (3 * A + 3 * Y) * (int)sizeof(T) <= 40 * 1024 ? 3 : 1;
  static constexpr int NA = NY == 3 ? 3 : 2;
  typedef Eo<n, M, false, T> J;
  typedef Eo<n, M, true, T> JD;
  typedef Eo<M, n, false, T> JT;
  static_assert(2 * A >= Y && 3 * n2 <= 3 * TPB, "regions");
};

// Factors w adj_ad, a = 0, 1, 2, of velocity component d along the line (r, s, z)
// of an element with the coefficient vectors g = (x_r, x_s, x_t, x_rs, x_rt,
// x_st, x_rst): c0 + c1 z, c2 + c3 z and c4 + c5 z + c6 z^2, the components of
// x_s x x_t, x_t x x_r and x_r x x_s, where x_r = a0 + a1 z and x_s = b0 + b1 z,
// and x_t = h is the same all along it.  Formed in FP64, rounded to T once.
template <typename T>
__device__ __forceinline__ void line_factors(UniformD g, int d, double r, double s, double w,
                                             T (&c)[7]) {
  const int e = (d + 1) % 3, f = (d + 2) % 3;
  double a0[2], a1[2], b0[2], b1[2], h[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int x = i ? f : e;
    a0[i] = g[x] + g[9 + x] * s;
    a1[i] = g[12 + x] + g[18 + x] * s;
    b0[i] = g[3 + x] + g[9 + x] * r;
    b1[i] = g[15 + x] + g[18 + x] * r;
    h[i] = (g[6 + x] + g[12 + x] * r) + (g[15 + x] + g[18 + x] * r) * s;
  }
  auto cross = [](const double (&p)[2], const double (&q)[2]) { return p[0] * q[1] - p[1] * q[0]; };
  c[0] = (T)(w * cross(b0, h));
  c[1] = (T)(w * cross(b1, h));
  c[2] = (T)(w * cross(h, a0));
  c[3] = (T)(w * cross(h, a1));
  c[4] = (T)(w * cross(a0, b0));
  c[5] = (T)(w * (cross(a0, b1) + cross(a1, b0)));
  c[6] = (T)(w * cross(a1, b1));
}

// Over-integrated rule, one element per workgroup; a thread transforms one
// line at a time in registers:
//   u_d:  along j from memory, along i through LDS, along k into the M^3
//         points, where V_a += G_ad u_d (the thread's (jq, iq) line of points;
//         the nine factors are streamed once);
//   f:    J f and J' f along j; J, J' and J along i; J, J, J' along k give the
//         three derivatives at the thread's points, c = sum_a V_a df/dr_a;
//   out:  J^T along k from registers, along i through LDS, along j to memory.
// V stays in registers and serves every field.
//
// FP64 vector and matrix products run at the same rate on gfx950, and the
// matrix form of these stages used 12 of 16 rows in the interpolations and 8 of
// 16 in the projections (and a branch per predicated access).  What bounds this
// form is its stream with one field (the nine factors; 5.5 TB/s in FP64 at N =
// 7) and its vector instructions with several.  Boxes of 4 million points, us
// for one / four fields, matrix form -> this form:
//   N      FP64                          FP32
//   3      366/816 -> 226/311            243/521 -> 107/142
//   5      293/614 -> 225/318            239/504 -> 111/151
//   7      270/500 -> 212/322            160/295 -> 107/169
//   9      354/694 -> 281/423            219/442 -> 116/173
//   10     282/558 -> 194/304            252/510 -> 87/146
// (Requesting a component's factors ahead into registers, as that form did,
// costs occupancy here: 774 against 322 us.)
//
// GEO 1 (every element straight-edged): the factors along the thread's point
// line are polynomials of its coordinate (line_factors), evaluated in place of
// nine streamed values.  The same boxes, stored -> formed:
//   N      FP64                          FP32
//   3      225/311 -> 113/258            111/139 -> 71/136
//   5      226/326 -> 113/233            111/152 -> 63/122
//   7      211/326 -> 111/250            107/163 -> 63/134
//   9      274/423 -> 129/295            117/173 -> 65/140
//   10     194/302 -> 105/235            89/145 -> 55/122
// bound by its vector instructions throughout.  (N = 7, FP64: 171 registers
// leave two waves per SIMD, 167/379 us, hence the budget of three.)
template <int N, typename T, int GEO>
__global__ __launch_bounds__((AdvShape<N, T>::TPB))
    __attribute__((amdgpu_waves_per_eu((N == 8 || (N == 7 && GEO)) && sizeof(T) == 8 ? 3 : 1))) void adv_dealias_kernel(
    int nf, const T* __restrict__ coef, const T* __restrict__ G, const double* __restrict__ geo,
    const double* __restrict__ pts, const T* __restrict__ u, int64_t ustride,
    const T* __restrict__ f, T* __restrict__ out) {
  typedef AdvShape<N, T> S;
  typedef typename S::J J;
  typedef typename S::JD JD;
  typedef typename S::JT JT;
  constexpr int n = S::n, M = S::M, P = S::P, Q = S::Q, n2 = S::n2, nM = S::nM, M2 = S::M2,
                TPB = S::TPB, SA = S::SA, SY = S::SY, NY = S::NY;
  __shared__ T sA[S::NA * S::A];
  __shared__ T sY[NY * S::Y];
  const T* cJ = coef;
  const T* cJD = coef + J::SZ;
  const T* cJT = cJD + JD::SZ;
  const T* cP = cJT + JT::SZ;  // points, weights
  (void)cP;
  const int t = threadIdx.x;
  const int64_t eP = (int64_t)blockIdx.x * P;
  const T* Ge = G + (int64_t)blockIdx.x * 9 * Q;
  (void)Ge;
  // this thread's node line along j (p = k n + i), its row of lines along i
  // and its point line along k
  const bool own_j = t < n2, own_k = t < M2;
  const int jbase = (t / n) * n2 + t % n;             // node (k, 0, i)
  const int abase = (t / n) * M * SA + t % n;         // sA place (k, jq = 0, i)
  const int ybase = (t / M) * SY + t % M;             // sY place (k = 0, jq, iq)

  // The line of the next field.  It is taken less the field's value at the
  // element's first node: the derivatives do not see a constant, and the
  // interpolations then round the field's variation over the element instead
  // of its values.
  T xf[n], f0;
  auto fetch_f = [&](const T* __restrict__ fe) {
    f0 = fe[0];
#pragma unroll
    for (int j = 0; j < n; ++j) xf[j] = own_j ? fe[jbase + j * n] : T(0);
  };
  fetch_f(f + eP);

  T V[3][M];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int q = 0; q < M; ++q) V[a][q] = T(0);
  auto lines_j = [&](int d, int p, T* __restrict__ dst) {
    const T* ud = u + d * ustride + eP + (p / n) * n2 + p % n;
    T* w = dst + (p / n) * M * SA + p % n;
    J([&](int j) { return ud[j * n]; }).apply(cJ, [&](int q, T y) { w[q * SA] = y; });
  };
  auto lines_i = [&](const T* __restrict__ src, T* __restrict__ dst, int r) {
    J([&](int i) { return src[r * SA + i]; }).apply(cJ, [&](int q, T y) { dst[r * SY + q] = y; });
  };
  auto add_v = [&](int d, const T* __restrict__ src) {
    auto line = [&](int k) { return src[ybase + k * M * SY]; };
    if constexpr (GEO == 1) {
      T c[7];
      line_factors<T>((UniformD)(uintptr_t)(geo + (int64_t)blockIdx.x * 21), d, pts[t % M],
                      pts[t / M], pts[M + t % M] * pts[M + t / M], c);
      J(line).apply(cJ, [&](int q, T y) {
        const T z = cP[q], wy = cP[M + q] * y;
        V[0][q] += (c[0] + c[1] * z) * wy;
        V[1][q] += (c[2] + c[3] * z) * wy;
        V[2][q] += (c[4] + (c[5] + c[6] * z) * z) * wy;
      });
    } else {
      const T* g = Ge + d * Q + t;
      J(line).apply(cJ, [&](int q, T y) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
          V[a][q] += __builtin_nontemporal_load(g + 3 * a * Q + q * M2) * y;
      });
    }
  };
  if constexpr (NY == 3) {
    for (int p = t; p < 3 * n2; p += TPB) lines_j(p / n2, p % n2, sA + (p / n2) * S::A);
    __syncthreads();
    for (int r = t; r < 3 * nM; r += TPB)
      lines_i(sA + (r / nM) * S::A, sY + (r / nM) * S::Y, r % nM);
    __syncthreads();
    if (own_k)
#pragma unroll
      for (int d = 0; d < 3; ++d) add_v(d, sY + d * S::Y);
  } else {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      if (own_j) lines_j(d, t, sA);
      __syncthreads();
      if (t < nM) lines_i(sA, sY, t);
      __syncthreads();
      if (own_k) add_v(d, sY);
    }
  }

  for (int m = 0; m < nf; ++m) {
    if (own_j) {
      auto x = [&](int j) { return xf[j] - f0; };
      J(x).apply(cJ, [&](int q, T y) { sA[abase + q * SA] = y; });
      JD(x).apply(cJD, [&](int q, T y) { sA[S::A + abase + q * SA] = y; });
    }
    // the next field's line is on its way during this field
    if (m + 1 < nf) fetch_f(f + (m + 1) * ustride + eP);
    __syncthreads();
    T c[M];
#pragma unroll
    for (int q = 0; q < M; ++q) c[q] = T(0);
    // derivative a at this thread's points from its (jq, iq) lines
    auto add_c = [&](auto dir, const T* __restrict__ src) {
      constexpr int a = decltype(dir)::value;
      auto x = [&](int k) { return src[ybase + k * M * SY]; };
      auto put = [&](int q, T y) { c[q] += V[a][q] * y; };
      if constexpr (a == 2) JD(x).apply(cJD, put);
      else J(x).apply(cJ, put);
    };
    if constexpr (NY == 3) {
      for (int r = t; r < 2 * nM; r += TPB) {
        const int row = r % nM;
        if (r < nM) {
          auto x = [&](int i) { return sA[row * SA + i]; };
          JD(x).apply(cJD, [&](int q, T y) { sY[row * SY + q] = y; });
          J(x).apply(cJ, [&](int q, T y) { sY[2 * S::Y + row * SY + q] = y; });
        } else {
          lines_i(sA + S::A, sY + S::Y, row);
        }
      }
      __syncthreads();
      if (own_k) {
        add_c(std::integral_constant<int, 0>(), sY);
        add_c(std::integral_constant<int, 1>(), sY + S::Y);
        add_c(std::integral_constant<int, 2>(), sY + 2 * S::Y);
      }
    } else {
      if (t < nM) {
        JD([&](int i) { return sA[t * SA + i]; }).apply(cJD, [&](int q, T y) { sY[t * SY + q] = y; });
      }
      __syncthreads();
      if (own_k) add_c(std::integral_constant<int, 0>(), sY);
      __syncthreads();
      if (t < nM) lines_i(sA + S::A, sY, t);
      __syncthreads();
      if (own_k) add_c(std::integral_constant<int, 1>(), sY);
      __syncthreads();
      if (t < nM) lines_i(sA, sY, t);
      __syncthreads();
      if (own_k) add_c(std::integral_constant<int, 2>(), sY);
    }
    // project: along k (to the first region, whose lines are used up) ...
    if (own_k) {
      JT([&](int q) { return c[q]; })
          .apply(cJT, [&](int k, T y) { sA[ybase + k * M * SY] = y; });
    }
    __syncthreads();
    // ... along i ...
    if (t < nM) {
      JT([&](int q) { return sA[t * SY + q]; })
          .apply(cJT, [&](int i, T y) { sY[t * SA + i] = y; });
    }
    __syncthreads();
    // ... along j
    if (own_j) {
      T* w = out + m * ustride + eP + jbase;
      JT([&](int q) { return sY[abase + q * SA]; })
          .apply(cJT, [&](int j, T y) { w[j * n] = y; });
    }
  }
}

// Collocation rule, one element per workgroup, a thread per node.  Bound by its
// stream with stored factors (GEO 0) and by the derivative sums' LDS reads with
// straight-edged ones, which it forms at its nodes (GEO 1; boxes of 4 million
// points, one / four fields in FP64, us: N = 3 101/173 -> 58/156, 7 85/140 ->
// 39/115, 10 103/192 -> 49/167).
template <int N, typename T, int GEO>
__global__ __launch_bounds__(kAdvThreads) void adv_colloc_kernel(
    int nf, const T* __restrict__ D, const T* __restrict__ G, const double* __restrict__ geo,
    const double* __restrict__ pts, const T* __restrict__ u, int64_t ustride,
    const T* __restrict__ f, T* __restrict__ out) {
  constexpr int n = N + 1, P = n * n * n, PT = (P + kAdvThreads - 1) / kAdvThreads;
  __shared__ T sF[P];
  __shared__ T sD[n * n];
  const int64_t e = blockIdx.x;
  for (int q = threadIdx.x; q < n * n; q += kAdvThreads) sD[q] = D[q];
  // V_a = sum_d G_ad u_d at this thread's nodes
  const T* Ge = G + e * 9 * P;
  T V[PT][3];
#pragma unroll
  for (int j = 0; j < PT; ++j) {
    const int q = threadIdx.x + j * kAdvThreads;
#pragma unroll
    for (int a = 0; a < 3; ++a) V[j][a] = T(0);
    if (q < P) {
      const int i = q % n, jj = (q / n) % n, kk = q / (n * n);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const T ud = u[d * ustride + e * P + q];
        if constexpr (GEO == 1) {
          const double z = pts[kk];
          double cd[7];
          line_factors<double>((UniformD)(uintptr_t)(geo + e * 21), d, pts[i], pts[jj],
                               pts[n + i] * pts[n + jj] * pts[n + kk], cd);
          V[j][0] += (T)(cd[0] + cd[1] * z) * ud;
          V[j][1] += (T)(cd[2] + cd[3] * z) * ud;
          V[j][2] += (T)(cd[4] + (cd[5] + cd[6] * z) * z) * ud;
        } else {
#pragma unroll
          for (int a = 0; a < 3; ++a) V[j][a] += Ge[(3 * a + d) * P + q] * ud;
        }
      }
    }
  }
  for (int k = 0; k < nf; ++k) {
    if (k > 0) __syncthreads();  // the previous field's sums are done with sF
    for (int q = threadIdx.x; q < P; q += kAdvThreads) sF[q] = f[k * ustride + e * P + q];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      const int q = threadIdx.x + j * kAdvThreads;
      if (q >= P) continue;
      const int i = q % n, jj = (q / n) % n, kk = q / (n * n);
      T fr = T(0), fs = T(0), ft = T(0);
#pragma unroll
      for (int l = 0; l < n; ++l) {
        fr += sD[i * n + l] * sF[(kk * n + jj) * n + l];
        fs += sD[jj * n + l] * sF[(kk * n + l) * n + i];
        ft += sD[kk * n + l] * sF[(l * n + jj) * n + i];
      }
      out[k * ustride + e * P + q] = V[j][0] * fr + V[j][1] * fs + V[j][2] * ft;
    }
  }
}

// dX[e][3 c + a] = dx_c/dr_a at the rule's points: the reference gradient of
// each coordinate, by the same stages as f in the dealiased kernel
template <int N, int M>
__global__ __launch_bounds__(kAdvThreads) void adv_metric_kernel(const double* __restrict__ mats,
                                                                 const double* __restrict__ xyz,
                                                                 double* __restrict__ dX) {
  typedef Stages<N, M, double> S;
  constexpr int n = S::n, P = S::P, Q = S::Q;
  __shared__ double sIX[S::IX];
  __shared__ double sY[S::YS];
  double* sIn = sIX;
  double* sX0 = sIX + P;
  double* sX1 = sX0 + n * n * M;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t e = blockIdx.x;
  double aJ[S::KN], aJD[S::KN];
  fragments<double, M, n>(mats, aJ, lane);
  fragments<double, M, n>(mats + M * n, aJD, lane);
  for (int cc = 0; cc < 3; ++cc) {
    for (int q = threadIdx.x; q < P; q += kAdvThreads) sIn[q] = xyz[(e * P + q) * 3 + cc];
    __syncthreads();
    for (int t = wv; t < S::I0::NT; t += kAdvWaves) {
      S::I0::store(sX0, S::I0::tile(sIn, aJ, t, lane), t, lane);
      S::I0::store(sX1, S::I0::tile(sIn, aJD, t, lane), t, lane);
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double* src = a == 0 ? sX1 : sX0;
      const double* a1 = a == 1 ? aJD : aJ;
      const double* a2 = a == 2 ? aJD : aJ;
      for (int t = wv; t < S::I1::NT; t += kAdvWaves)
        S::I1::store(sY, S::I1::tile(src, a1, t, lane), t, lane);
      __syncthreads();
      double* dst = dX + (e * 9 + 3 * cc + a) * Q;
      for (int t = wv; t < S::I2::NT; t += kAdvWaves)
        S::I2::store(dst, S::I2::tile(sY, a2, t, lane), t, lane);
      __syncthreads();
    }
  }
}

// G_ad = w detJ dr_a/dx_d = w adj(dx/dr)_ad in place of dx_c/dr_a, per point
__global__ void adv_metric_finish(int64_t E, int q1, const double* __restrict__ w1,
                                  double* __restrict__ G, float* __restrict__ G32,
                                  int* __restrict__ bad) {
  const int64_t Q = (int64_t)q1 * q1 * q1;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= E * Q) return;
  const int64_t e = idx / Q, q = idx % Q;
  const int i = (int)(q % q1), j = (int)((q / q1) % q1), k = (int)(q / ((int64_t)q1 * q1));
  double* g = G + e * 9 * Q + q;
  double m[3][3];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int a = 0; a < 3; ++a) m[c][a] = g[(3 * c + a) * Q];
  double adj[3][3];  // adj[a][d] = det * (dr_a/dx_d)
  adj[0][0] = m[1][1] * m[2][2] - m[1][2] * m[2][1];
  adj[0][1] = m[0][2] * m[2][1] - m[0][1] * m[2][2];
  adj[0][2] = m[0][1] * m[1][2] - m[0][2] * m[1][1];
  adj[1][0] = m[1][2] * m[2][0] - m[1][0] * m[2][2];
  adj[1][1] = m[0][0] * m[2][2] - m[0][2] * m[2][0];
  adj[1][2] = m[0][2] * m[1][0] - m[0][0] * m[1][2];
  adj[2][0] = m[1][0] * m[2][1] - m[1][1] * m[2][0];
  adj[2][1] = m[0][1] * m[2][0] - m[0][0] * m[2][1];
  adj[2][2] = m[0][0] * m[1][1] - m[0][1] * m[1][0];
  const double det = m[0][0] * adj[0][0] + m[0][1] * adj[1][0] + m[0][2] * adj[2][0];
  if (!(det > 0.0)) atomicAdd(bad, 1);
  const double W = w1[i] * w1[j] * w1[k];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double v = W * adj[a][d];
      g[(3 * a + d) * Q] = v;
      if (G32) G32[e * 9 * Q + (3 * a + d) * Q + q] = (float)v;
    }
}

template <int N, typename T>
hipError_t run_advect(const sem_mesh* m, const AdvRule& R, int rule, int nf, const T* D,
                      const T* u, const T* f, T* out, hipStream_t s) {
  const int64_t ustride = m->E * (int64_t)m->P;
  const T* G = nullptr;
  const T* eo = nullptr;
  if constexpr (sizeof(T) == 8) {
    G = R.G64.as<double>();
    eo = R.eo64.as<double>();
  } else {
    G = R.G32.as<float>();
    eo = R.eo32.as<float>();
  }
  const double* geo = R.geo.as<double>();
  const double* pts = R.pts64.as<double>();
  const dim3 grid((unsigned)m->E);
  // straight-edged: from N = 3 on (box of 4 million points, one / four fields, us,
  // stored -> formed: N = 2 FP64 259/358 -> 166/373, FP32 97/193 -> 119/212;
  // N = 3 FP64 223/309 -> 113/258, FP32 108/146 -> 71/136), collocation always
  constexpr int kFrom = 3;
#define SEM_ADV(KERNEL, TPB, MAT, FROM)                                                        \
  do {                                                                                         \
    if (N >= FROM && R.straight)                                                               \
      hipLaunchKernelGGL((KERNEL<N, T, (N >= FROM ? 1 : 0)>), grid, dim3(TPB), 0, s, nf, MAT, G, geo, pts, u,    \
                         ustride, f, out);                                                     \
    else                                                                                       \
      hipLaunchKernelGGL((KERNEL<N, T, 0>), grid, dim3(TPB), 0, s, nf, MAT, G, geo, pts, u,    \
                         ustride, f, out);                                                     \
  } while (0)
  if (rule == 0) SEM_ADV(adv_colloc_kernel, kAdvThreads, D, 1);
  else SEM_ADV(adv_dealias_kernel, (AdvShape<N, T>::TPB), eo, kFrom);
#undef SEM_ADV
  return hipGetLastError();
}

template <int N>
hipError_t run_metric(const sem_mesh* m, int q1, const double* mats, const double* xyz,
                      double* dX, hipStream_t s) {
  constexpr int Md = (3 * (N + 1)) / 2;
  if (q1 == N + 1)
    hipLaunchKernelGGL((adv_metric_kernel<N, N + 1>), dim3((unsigned)m->E), dim3(kAdvThreads), 0,
                       s, mats, xyz, dX);
  else if (q1 == Md)
    hipLaunchKernelGGL((adv_metric_kernel<N, Md>), dim3((unsigned)m->E), dim3(kAdvThreads), 0, s,
                       mats, xyz, dX);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_adv_geometry(const sem_mesh* m, int q1, const double* mats, const double* w1,
                               const double* xyz, double* G, float* G32, int* bad,
                               hipStream_t s) {
  hipError_t err;
  switch (m->N) {
    case 1: err = run_metric<1>(m, q1, mats, xyz, G, s); break;
    case 2: err = run_metric<2>(m, q1, mats, xyz, G, s); break;
    case 3: err = run_metric<3>(m, q1, mats, xyz, G, s); break;
    case 4: err = run_metric<4>(m, q1, mats, xyz, G, s); break;
    case 5: err = run_metric<5>(m, q1, mats, xyz, G, s); break;
    case 6: err = run_metric<6>(m, q1, mats, xyz, G, s); break;
    case 7: err = run_metric<7>(m, q1, mats, xyz, G, s); break;
    case 8: err = run_metric<8>(m, q1, mats, xyz, G, s); break;
    case 9: err = run_metric<9>(m, q1, mats, xyz, G, s); break;
    case 10: err = run_metric<10>(m, q1, mats, xyz, G, s); break;
    default: return hipErrorInvalidValue;
  }
  if (err != hipSuccess) return err;
  const int64_t total = m->E * (int64_t)q1 * q1 * q1;
  const int64_t blocks = (total + 255) / 256;
  hipLaunchKernelGGL(adv_metric_finish, dim3((unsigned)blocks), dim3(256), 0, s, m->E, q1, w1, G,
                     G32, bad);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_advect(const sem_mesh* m, const AdvRule& R, int rule, int nf, const T* D,
                         const T* u, const T* f, T* out, hipStream_t s) {
  if (nf <= 0) return hipSuccess;
  switch (m->N) {
    case 1: return run_advect<1, T>(m, R, rule, nf, D, u, f, out, s);
    case 2: return run_advect<2, T>(m, R, rule, nf, D, u, f, out, s);
    case 3: return run_advect<3, T>(m, R, rule, nf, D, u, f, out, s);
    case 4: return run_advect<4, T>(m, R, rule, nf, D, u, f, out, s);
    case 5: return run_advect<5, T>(m, R, rule, nf, D, u, f, out, s);
    case 6: return run_advect<6, T>(m, R, rule, nf, D, u, f, out, s);
    case 7: return run_advect<7, T>(m, R, rule, nf, D, u, f, out, s);
    case 8: return run_advect<8, T>(m, R, rule, nf, D, u, f, out, s);
    case 9: return run_advect<9, T>(m, R, rule, nf, D, u, f, out, s);
    case 10: return run_advect<10, T>(m, R, rule, nf, D, u, f, out, s);
    default: return hipErrorInvalidValue;
  }
}
template hipError_t launch_advect<double>(const sem_mesh*, const AdvRule&, int, int,
                                          const double*, const double*, const double*, double*,
                                          hipStream_t);
template hipError_t launch_advect<float>(const sem_mesh*, const AdvRule&, int, int, const float*,
                                         const float*, const float*, float*, hipStream_t);

}  // namespace sem
