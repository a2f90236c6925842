// Fast-diagonalisation local solves of the overlapping Schwarz smoother.
//
// Per element the residual is gathered into the (N+3)^3 box through its
// subdomain map (0 at points outside the subdomain), transformed by S_r^T,
// S_s^T, S_t^T along the three directions, divided by l_r,i + l_s,j + l_t,k,
// transformed back by S_r, S_s, S_t, and written to the box buffer; a
// segmented sum over the box points of each free node completes
// z = sum_e R_e^T A~_e^{-1} R_e r.  Each 1-D transform of the box is a batch
// of 16-column tiles C = M X on the matrix cores (16x16x4 MFMA in FP64 or
// FP32) with M = S or S^T of this element.
#include <algorithm>

#include "mfma_16x16x4.hpp"
#include "schwarz.hpp"

namespace sem {
namespace {

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Addressing of the box [k][j][i] by tiles of 16 columns along direction DIR
// (columns enumerate the other two indices, the lower one fastest).  No load
// or store is predicated per access (a branch each kept every LDS read in a
// block of its own: 223 mask changes per element at n = 10), and tile, step and row enter as constants added to one lane
// base per direction, so they become the instructions' offsets.  Columns past
// the last one repeat it (they compute and store the same values), contraction
// indices past n repeat the last one against zero fragments of M, and result
// rows past n are left out for all tiles at once.
template <int n>
struct BoxLane {
  static constexpr int P2 = n * n, NT = (P2 + 15) / 16, KS = (n + 3) / 4;
  int c16, kk;
  int clast;     // column of the last tile
  int b1[NT];    // DIR 1: place of each tile's column
  __device__ __forceinline__ explicit BoxLane(int lane) : c16(lane & 15), kk(lane >> 4) {
    clast = min(16 * (NT - 1) + c16, P2 - 1);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int c = col(t);
      b1[t] = (c / n) * P2 + c % n;
    }
  }
  __device__ __forceinline__ int col(int t) const { return t < NT - 1 ? c16 + 16 * t : clast; }
  // contraction index of step s
  __device__ __forceinline__ int at_step(int s) const {
    return 4 * s + 3 < n ? kk + 4 * s : min(kk + 4 * s, n - 1);
  }
  template <int DIR>
  __device__ __forceinline__ int place(int t, int l) const {
    if constexpr (DIR == 0) return t < NT - 1 ? c16 * n + l + 16 * n * t : clast * n + l;
    else if constexpr (DIR == 1) return b1[t] + l * n;
    else return t < NT - 1 ? l * P2 + c16 + 16 * t : l * P2 + clast;
  }
};

// this lane's fragments of M = S^T (trans) or S, one per step of four columns
template <int n, typename T>
__device__ __forceinline__ void fdm_frag(const T* __restrict__ S, bool trans,
                                         const BoxLane<n>& q, T (&af)[BoxLane<n>::KS]) {
  const int mrow = min(q.c16, n - 1);
#pragma unroll
  for (int s = 0; s < BoxLane<n>::KS; ++s) {
    const int l = q.at_step(s);
    const T v = trans ? S[l * n + mrow] : S[mrow * n + l];
    af[s] = (q.c16 < n && 4 * s + q.kk < n) ? v : T(0);
  }
}

// acc = M times every tile of the box along DIR
template <int n, typename T, int DIR>
__device__ __forceinline__ void fdm_mul(const T* __restrict__ box, const T (&af)[BoxLane<n>::KS],
                                        const BoxLane<n>& q,
                                        typename Mm<T>::V (&acc)[BoxLane<n>::NT]) {
  constexpr int NT = BoxLane<n>::NT, KS = BoxLane<n>::KS;
  T b[NT][KS];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s) b[t][s] = box[q.template place<DIR>(t, q.at_step(s))];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    acc[t] = typename Mm<T>::V{T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int s = 0; s < KS; ++s) acc[t] = Mm<T>::mma(af[s], b[t][s], acc[t]);
  }
}

// the result tiles back to the box (any memory) along DIR
template <int n, typename T, int DIR>
__device__ __forceinline__ void fdm_put(T* __restrict__ box, const BoxLane<n>& q, int lane,
                                        const typename Mm<T>::V (&acc)[BoxLane<n>::NT]) {
  constexpr int dr = sizeof(T) == 8 ? 4 : 1;  // rows between a lane's result registers
  const int row0 = Mm<T>::row(lane, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (row0 + r * dr < n)
#pragma unroll
      for (int t = 0; t < BoxLane<n>::NT; ++t)
        box[q.template place<DIR>(t, row0 + r * dr)] = acc[t][r];
}

// One wavefront per element: its LDS operations complete in program order, so
// no stage waits for a barrier, and the wavefronts of a CU overlap each
// other's latencies.  Measured on the 32x32x16, N = 7 box in FP32 (mean of the
// launches of a solve): 56 us, against 82 us of a persistent workgroup of four
// wavefronts per element with six LDS round trips and nine barriers; 114
// against 142 us in FP64.  The 218 MB of the FP32 form stream in 44 us; what
// bounds it is issue (31 us of vector instructions, a quarter of them the
// divisions, and 28 us of matrix products).
// The stages are ordered so that little goes through LDS: the t-direction
// comes first, straight from the gathered registers, and last, straight to
// memory (its tile columns are 16 consecutive points); the forward and
// backward s-transforms with the division between them stay in registers (a
// result tile's rows are the contraction index of the next product).  Every
// tile reads and writes only its own 16 lines, so the box is transformed in
// place.
constexpr int fdm_waves(int n) { return n <= 8 ? 4 : 1; }  // elements per workgroup

// Wavefronts per SIMD asked for: with a budget of at most 128 registers the
// compiler keeps the products' results in the ordinary registers (in the
// accumulation registers each costs a move before its store).
template <typename T>
constexpr int fdm_min_waves(int n) {
  return sizeof(T) == 4 ? (n <= 8 ? 7 : n <= 10 ? 5 : n <= 12 ? 4 : 3)
                        : (n <= 6 ? 5 : n <= 8 ? 4 : n <= 10 ? 3 : 2);
}

template <int n, typename T>
__global__ __launch_bounds__(64 * fdm_waves(n))
    __attribute__((amdgpu_waves_per_eu(fdm_min_waves<T>(n)))) void fdm_kernel(
    int64_t E, const int32_t* __restrict__ xmap, const T* __restrict__ S,
    const T* __restrict__ lam, const T* __restrict__ r, T* __restrict__ out,
    const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int P2 = n * n, P3 = P2 * n, NT = BoxLane<n>::NT, KS = BoxLane<n>::KS;
  constexpr int NF = 3 * P2 + 3 * n;  // S then lam of one element
  constexpr int FPT = (NF + 63) / 64, NWG = fdm_waves(n);
  __shared__ T sA[NWG][P3];
  __shared__ T sF[NWG][NF];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  T* A = sA[w];
  T* F = sF[w];
  const int64_t e = (int64_t)blockIdx.x * NWG + w;
  if (e >= E) return;  // the whole wavefront (no workgroup barrier follows)
  const BoxLane<n> q(lane);
  typename Mm<T>::V acc[NT];
  T af[KS];
  {
    const int32_t* xm = xmap + e * P3;
    const T* Se = S + e * 3 * P2;
    const T* Le = lam + e * 3 * n;
    int32_t gi[NT][KS];
    T rv[NT][KS], fv[FPT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int s = 0; s < KS; ++s) gi[t][s] = xm[q.template place<2>(t, q.at_step(s))];
#pragma unroll
    for (int s = 0; s < FPT; ++s) {
      const int f = min(lane + 64 * s, NF - 1);
      const T* at = f < 3 * P2 ? Se + f : Le + (f - 3 * P2);
      fv[s] = *at;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const T v = r[max(gi[t][s], 0)];
        rv[t][s] = gi[t][s] >= 0 ? v : T(0);
      }
#pragma unroll
    for (int s = 0; s < FPT; ++s) F[min(lane + 64 * s, NF - 1)] = fv[s];
    wave_sync();
    fdm_frag<n, T>(F + 2 * P2, true, q, af);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc[t] = typename Mm<T>::V{T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int s = 0; s < KS; ++s) acc[t] = Mm<T>::mma(af[s], rv[t][s], acc[t]);
    }
  }
  fdm_put<n, T, 2>(A, q, lane, acc);
  wave_sync();
  fdm_frag<n, T>(F, true, q, af);
  fdm_mul<n, T, 0>(A, af, q, acc);
  fdm_put<n, T, 0>(A, q, lane, acc);
  wave_sync();
  fdm_frag<n, T>(F + P2, true, q, af);
  fdm_mul<n, T, 1>(A, af, q, acc);
  {
    const T* L = F + 3 * P2;
    T ab[4], ls[4];  // S_s and l_s in the order of a result tile's rows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int l = Mm<T>::row(lane, i), lc = min(l, n - 1);
      const T v = F[P2 + min(q.c16, n - 1) * n + lc];
      ab[i] = (q.c16 < n && l < n) ? v : T(0);
      ls[i] = L[n + lc];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int c = q.col(t);
      const T lrt = L[c % n] + L[2 * n + c / n];
      typename Mm<T>::V back = {T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int i = 0; i < 4; ++i)  // rows past n: 0 divided by a sum that is there
        back = Mm<T>::mma(ab[i], acc[t][i] / (lrt + ls[i]), back);
      acc[t] = back;
    }
  }
  fdm_put<n, T, 1>(A, q, lane, acc);
  wave_sync();
  fdm_frag<n, T>(F, false, q, af);
  fdm_mul<n, T, 0>(A, af, q, acc);
  fdm_put<n, T, 0>(A, q, lane, acc);
  wave_sync();
  fdm_frag<n, T>(F + 2 * P2, false, q, af);
  fdm_mul<n, T, 2>(A, af, q, acc);
  fdm_put<n, T, 2>(out + e * P3, q, lane, acc);
}

template <int n, typename T>
hipError_t run_fdm(int64_t E, const int32_t* xmap, const T* S, const T* lam, const T* r, T* out,
                   const int32_t* skip, hipStream_t s) {
  constexpr int NWG = fdm_waves(n);
  const int64_t grid = (E + NWG - 1) / NWG;
  hipLaunchKernelGGL((fdm_kernel<n, T>), dim3((unsigned)grid), dim3(64 * NWG), 0, s, E, xmap, S,
                     lam, r, out, skip);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_fdm(const SchwarzDev& X, int64_t E, const T* r, T* box_out,
                      const int32_t* skip, hipStream_t s) {
  const int32_t* xm = X.xmap.as<int32_t>();
  const T* S = sizeof(T) == 8 ? (const T*)X.S64.p : (const T*)X.S32.p;
  const T* L = sizeof(T) == 8 ? (const T*)X.L64.p : (const T*)X.L32.p;
  switch (X.nx) {
    case 5: return run_fdm<5, T>(E, xm, S, L, r, box_out, skip, s);
    case 6: return run_fdm<6, T>(E, xm, S, L, r, box_out, skip, s);
    case 7: return run_fdm<7, T>(E, xm, S, L, r, box_out, skip, s);
    case 8: return run_fdm<8, T>(E, xm, S, L, r, box_out, skip, s);
    case 9: return run_fdm<9, T>(E, xm, S, L, r, box_out, skip, s);
    case 10: return run_fdm<10, T>(E, xm, S, L, r, box_out, skip, s);
    case 11: return run_fdm<11, T>(E, xm, S, L, r, box_out, skip, s);
    case 12: return run_fdm<12, T>(E, xm, S, L, r, box_out, skip, s);
    case 13: return run_fdm<13, T>(E, xm, S, L, r, box_out, skip, s);
    default: return hipErrorInvalidValue;
  }
}
template hipError_t launch_fdm<double>(const SchwarzDev&, int64_t, const double*, double*,
                                       const int32_t*, hipStream_t);
template hipError_t launch_fdm<float>(const SchwarzDev&, int64_t, const float*, float*,
                                      const int32_t*, hipStream_t);

}  // namespace sem
