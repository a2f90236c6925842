// Element operator kernels for gfx950 (wave64).
//
// A_L(k) u = sum_ab D_a^T diag(k G_ab) D_b u + h2 B u on every element: the
// matrix-free tensor-product operator of Sec. 2.2, whose leading work is
// dense (N+1)x(N+1) contractions identical for all elements.
//
// Mapping: one thread per local point (two for N = 10), one element (or a
// few small ones) per workgroup.  Every thread issues all of its global loads
// -- u (or its gather through the free numbering), the six geometric factors
// and k -- before the first barrier, so a workgroup has its whole element in
// flight at once; the streamed arrays are read and w written with
// nontemporal hints (each byte is touched once).  The in-solve form's
// shared-copy outputs are plain stores instead when the local array is small
// enough: the segmented sum reads them right after and finds most of them in
// the memory-side cache (28 -> 22 us per iteration on the 32x32x16, N = 7
// box, against 2 us more for the operator).  The element
// block and D live in LDS; the reference-gradient phase and the transposed
// phase are separated by one barrier.  For N = 7 a wavefront is exactly one k-plane,
// so the t-direction coefficients D[k][l] are wave-uniform and come from
// scalar loads instead of LDS.
//
// For larger N the scalar contractions make the kernel LDS-bound (each
// point reads 2 (N+1) values per direction per phase from LDS).  There the
// contractions run on the matrix cores instead (ax_line_kernel): each
// direction is a batch of 16-column tiles C = D X (or D^T X) with X gathered
// from the element block in LDS, 16x16x4 MFMAs in FP64 or FP32, so every LDS
// value feeds a whole tile column instead of one output.
//
// Per local point the FP64 apply streams u (8 B), six geometric factors
// (48 B, planar layout [E][6][P]) and w (8 B): 64 B.
//
// Inside the CG (N >= 5) the matrix-core kernel also splits its output: the
// nodes with a single local copy are finished by the element itself, so it
// stores w there straight into the free vector (with the sums of p w, and
// with a null space of w, over its copies), and only the shared copies go through the
// segmented sum, from the element's surface slots.
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include <hip/hip_ext.h>

#include "ax_tiles.hpp"
#include "common.hpp"

namespace sem {
namespace {

// elements per workgroup and points per thread, chosen so that the workgroup
// fills whole wavefronts with little idle work and stays within 1024 threads
constexpr int pick_epb(int P) {
  return P <= 8 ? 32 : P <= 27 ? 9 : P <= 64 ? 4 : P <= 343 ? 2 : 1;
}

template <int N>
struct Shape {
  static constexpr int n1 = N + 1;
  static constexpr int P2 = n1 * n1;
  static constexpr int P = P2 * n1;
  static constexpr int PPT = P > 1024 ? 2 : 1;          // points per thread
  static constexpr int TPE = (P + PPT - 1) / PPT;       // threads per element
  static constexpr int EPB = pick_epb(P);
  static constexpr int BT = ((EPB * TPE + 63) / 64) * 64;
  static constexpr bool kUniform = (P2 == 64 && PPT == 1);  // a wavefront = one k-plane
};

template <typename T>
__device__ __forceinline__ T ld_stream(const T* p) {
  return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ __forceinline__ void st_stream(T v, T* p) {
  __builtin_nontemporal_store(v, p);
}

template <int N, typename T, bool GATHER>
__global__ __launch_bounds__(Shape<N>::BT) void ax_kernel(
    const T* __restrict__ u, const int32_t* __restrict__ lmap, T* __restrict__ w,
    const T* __restrict__ kf, const T h2, const T* __restrict__ G, const T* __restrict__ B,
    const T* __restrict__ D, const int64_t E, const int32_t* __restrict__ skip) {
  using S = Shape<N>;
  constexpr int n1 = S::n1, P2 = S::P2, P = S::P, EPB = S::EPB, PPT = S::PPT, TPE = S::TPE;
  if (skip && *skip) return;  // uniform over the grid
  __shared__ T su[EPB][P];
  __shared__ T sv[EPB][3][P];
  __shared__ T sD[n1 * n1];

  const int t = threadIdx.x;
  const int slot = t / TPE;
  const int tl = t - slot * TPE;
  const int64_t e = xcd_block(blockIdx.x, gridDim.x) * EPB + slot;
  const bool ok_e = slot < EPB && e < E;
  const int ss = slot < EPB ? slot : 0;
  const bool use_k = kf != nullptr;
  const bool use_h2 = h2 != T(0);

  // Idle threads (tail of the last workgroup, padding lanes) load from a
  // clamped valid address and discard the values, so every load below is
  // unconditional and issued back to back.
  const int64_t ec = ok_e ? e : E - 1;
  for (int a = t; a < n1 * n1; a += S::BT) sD[a] = D[a];
  T uq[PPT], gq[PPT][6], kq[PPT];
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int qr = tl + s * TPE;
    const int q = qr < P ? qr : P - 1;
    const int64_t idx = ec * P + q;
    T v;
    if constexpr (GATHER) {
      const int32_t lm = ld_stream(lmap + idx);
      v = u[lm >= 0 ? lm : 0];
      v = lm >= 0 ? v : T(0);
    } else {
      v = ld_stream(u + idx);
    }
    uq[s] = ok_e ? v : T(0);
    const T* g = G + ec * 6 * P + q;
#pragma unroll
    for (int c = 0; c < 6; ++c) gq[s][c] = ld_stream(g + c * P);
    kq[s] = use_k ? ld_stream(kf + idx) : T(1);
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = tl + s * TPE;
    if (slot < EPB && q < P) su[ss][q] = uq[s];
  }
  __syncthreads();

  // reference gradient, metric, conductivity
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = tl + s * TPE;
    if (slot < EPB && q < P) {
      const int i = q % n1, j = (q / n1) % n1;
      const int k = S::kUniform ? __builtin_amdgcn_readfirstlane(q / P2) : q / P2;
      const T* uk = &su[ss][k * P2];
      T ur = T(0), us = T(0), ut = T(0);
#pragma unroll
      for (int l = 0; l < n1; ++l) {
        ur += sD[i * n1 + l] * uk[j * n1 + l];
        us += sD[j * n1 + l] * uk[l * n1 + i];
        const T dkl = S::kUniform ? D[k * n1 + l] : sD[k * n1 + l];
        ut += dkl * su[ss][l * P2 + j * n1 + i];
      }
      const T* gc = gq[s];
      T vr = gc[0] * ur + gc[1] * us + gc[2] * ut;
      T vs = gc[1] * ur + gc[3] * us + gc[4] * ut;
      T vt = gc[2] * ur + gc[4] * us + gc[5] * ut;
      if (use_k) {
        vr *= kq[s];
        vs *= kq[s];
        vt *= kq[s];
      }
      sv[ss][0][q] = vr;
      sv[ss][1][q] = vs;
      sv[ss][2][q] = vt;
    }
  }
  __syncthreads();

  // transposed contractions (+ mass term)
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = tl + s * TPE;
    if (ok_e && q < P) {
      const int i = q % n1, j = (q / n1) % n1;
      const int k = S::kUniform ? __builtin_amdgcn_readfirstlane(q / P2) : q / P2;
      const T* vr = &sv[ss][0][k * P2];
      const T* vs = &sv[ss][1][k * P2];
      T acc = T(0);
#pragma unroll
      for (int l = 0; l < n1; ++l) {
        acc += sD[l * n1 + i] * vr[j * n1 + l];
        acc += sD[l * n1 + j] * vs[l * n1 + i];
        const T dlk = S::kUniform ? D[l * n1 + k] : sD[l * n1 + k];
        acc += dlk * sv[ss][2][l * P2 + j * n1 + i];
      }
      const int64_t idx = e * P + q;
      if (use_h2) acc += h2 * ld_stream(B + idx) * uq[s];
      st_stream(acc, w + idx);
    }
  }
}


// ------------------------------------------------------------ matrix cores

typedef _Float16 v4h_t __attribute__((ext_vector_type(4)));
typedef __bf16 v4bf_t __attribute__((ext_vector_type(4)));

// 16x16x16 MFMA with 16-bit operands and FP32 accumulation (products of two
// 16-bit values are exact in FP32): A[i][k] in lane i + 16 (k / 4), vector
// element k % 4; B[k][j] in lane j + 16 (k / 4), element k % 4; result laid
// out as in the FP32 16x16x4 form (checked on the device).  One instruction
// covers a whole contraction: K = 16 >= N + 1, the rest padded with zeros.
// LP = 1: bfloat16 operands; LP = 2: IEEE half operands.  Conversions round
// to nearest, ties to even.
template <int LP>
struct Mfma16;
template <>
struct Mfma16<1> {
  typedef v4bf_t V;
  static __device__ __forceinline__ __bf16 cvt(float x) { return (__bf16)x; }
  static __device__ __forceinline__ v4f_t mma(V a, V b, v4f_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma16<2> {
  typedef v4h_t V;
  static __device__ __forceinline__ _Float16 cvt(float x) { return (_Float16)x; }
  static __device__ __forceinline__ v4f_t mma(V a, V b, v4f_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
  }
};

// One 16-column tile of a contraction along direction DIR of the element
// block src ([k][j][i], n1 per direction): out[.., row, ..] = sum_l A[row][l]
// src[.., l, ..], A = D (forward) or D^T (transposed), given as this lane's
// fragment.  Columns enumerate the two other indices: DIR 0 (along i):
// col = k n1 + j; DIR 1 (along j): col = k n1 + i; DIR 2 (along k): col =
// j n1 + i.  ACC adds into dst instead of storing.  Each source value is
// multiplied by the block scale `sc` (a power of two, exact) before rounding,
// and each result by `inv` = 1 / sc after accumulation.
template <int n1, int LP, int DIR, bool ACC>
__device__ __forceinline__ void contract_tile16(const float* __restrict__ src,
                                                float* __restrict__ dst,
                                                typename Mfma16<LP>::V afrag, int tile, int lane,
                                                float sc, float inv) {
  constexpr int P2 = n1 * n1;
  const int col = tile * 16 + (lane & 15);
  const int kk = lane >> 4;
  const bool cval = col < P2;
  const int c1 = cval ? col / n1 : 0, c0 = cval ? col % n1 : 0;
  typename Mfma16<LP>::V b;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int l = 4 * kk + e;
    float x = 0.0f;
    if (cval && l < n1) {
      const int a = DIR == 0 ? c1 * P2 + c0 * n1 + l : DIR == 1 ? c1 * P2 + l * n1 + c0 : l * P2 + col;
      x = src[a];
    }
    b[e] = Mfma16<LP>::cvt(x * sc);
  }
  v4f_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
  acc = Mfma16<LP>::mma(afrag, b, acc);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * (lane >> 4) + r;
    if (cval && row < n1) {
      const int a =
          DIR == 0 ? c1 * P2 + c0 * n1 + row : DIR == 1 ? c1 * P2 + row * n1 + c0 : row * P2 + col;
      if (ACC) dst[a] += acc[r] * inv;
      else dst[a] = acc[r] * inv;
    }
  }
}

// Power-of-two scale that puts a block maximum m in [2^14, 2^15) (IEEE half
// keeps all its bits there and cannot overflow), with the exponent kept in
// FP32's normal range; 1 for zero or non-finite m.
__device__ __forceinline__ float half_block_scale(float m) {
  if (!(m > 0.0f) || !(m <= 3.402823466e38f)) return 1.0f;
  int ex;
  (void)frexpf(m, &ex);
  const int k = min(max(15 - ex, -126), 126);
  return ldexpf(1.0f, k);
}


__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// Shape of the 16-bit operand kernel
template <int N>
struct MShape {
  static constexpr int n1 = N + 1;
  static constexpr int P2 = n1 * n1;
  static constexpr int P = P2 * n1;
  // threads per element (= per workgroup)
  static constexpr int TPB =
      P <= 64 ? 64 : P <= 128 ? 128 : P <= 1000 ? 256 : 512;
  static constexpr int PPT = (P + TPB - 1) / TPB;    // points per thread
  static constexpr int NT = (P2 + 15) / 16;          // 16-column tiles per direction
  static constexpr int NW = TPB / 64;                // wavefronts
};

// -------------------------------------- matrix-core operator (FP64, FP32)

// Operator with matrix-core contractions in T, one element per workgroup:
//   loads, u to LDS | D along i, j, k | metric and k | D^T along i, j, k, in
//   place | sum of the three, store                          (| = barrier).
// Bound by its stream: 64 B per point in FP64, 32 B in FP32 (+ 4 B of routing
// codes and the gathers in the solve).  Measured on boxes of 8 million points,
// us per apply, against the form whose tile accesses each sat behind a branch
// and whose three transposed contractions ran one after another:
//   N           5        6        7        8        9       10
//   FP64    122->88  105->94   83->82  118->92  116->97  106->97
//   FP32     84->58   76->53   53->43   63->48   59->51   62->50
// (A form that kept each wavefront's points in the products' result layout, so
// that the k contractions need no LDS, loads the factors in runs of 16: as fast
// at N = 7, 158 us at N = 8.)
//
// MODE 0: u and w local [E][P].  MODE 1: u gathered from a free vector
// through lmap.  MODE 2 (in-solve split): lmap holds v >= 0 for a free node v
// with one local copy, -(v + 2) for a shared free node v, -1 for a Dirichlet
// copy; single-copy results go straight to the free vector wf[v], shared
// copies' results to w (local, at the element's surface slots, for the
// segmented sum), and epart[a E + e] receives each element's sums
// of p w and of w over all its free copies (p = the gathered input; over the
// copies of a shared node they add up to p_g w_g and w_g), reduced in a fixed
// order.  MODE 3: MODE 2 with nontemporal shared-copy stores (for local arrays
// larger than the memory-side cache).  MODE 4 / 5: MODE 2 / 3 without the
// sums (a Chebyshev pass needs none).  MODE 6 / 7: MODE 2 / 3 with
// p w only (sum(w) serves the null-space projection alone).
//
// GEO 0: factors from G and B.  GEO 1 (every element of the mesh is straight-
// edged; FP64 only): formed per point from the element's coefficients (geo, 21
// per element; pts: the GLL nodes and weights): 16 B per point.  In FP32 the
// same arithmetic costs more than the 24 B it saves (N = 7: 53 against 43 us).
// FP64 with k and h2 on 8 million points, stored -> straight-edged, us:
//   N = 5 106 -> 88, 6 118 -> 85, 7 99 -> 74, 8 108 -> 88, 9 107 -> 84, 10 112 -> 92;
// bound by its FP64 operations (about 150 per point, products and vector
// instructions in the same units) and LDS passes.
template <int N, typename T, int MODE, int GEO>
__global__ __launch_bounds__((LShape<N, T>::TPB))
    __attribute__((amdgpu_waves_per_eu(ax_min_waves(N, sizeof(T), GEO)))) void ax_line_kernel(
        const T* __restrict__ u, const int32_t* __restrict__ lmap, T* __restrict__ w,
        const T* __restrict__ kf, const T h2, const T* __restrict__ G, const T* __restrict__ B,
        const T* __restrict__ D, const double* __restrict__ geo,
        const double* __restrict__ pts, const int32_t* __restrict__ skip, T* __restrict__ wf,
        double* __restrict__ epart) {
  using S = LShape<N, T>;
  constexpr int n1 = S::n1, P = S::P, KS = S::KS, PPT = S::PPT, TPB = S::TPB, NW = S::NW,
                NT = S::NT, TPW = S::TPW, SZ = n1 * S::PS;
  constexpr int kSums = (MODE == 2 || MODE == 3) ? 2 : (MODE == 6 || MODE == 7) ? 1 : 0;
  constexpr bool kNtShared = (MODE == 3 || MODE == 5 || MODE == 7);
  if (skip && *skip) return;  // uniform over the grid
  __shared__ T su[SZ];
  __shared__ T sa[3][SZ];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t e = blockIdx.x;
  const bool use_k = kf != nullptr;
  const bool use_h2 = h2 != T(0);
  const T* Ge = G + e * 6 * P;
  const int64_t eP = e * P;
  // point s of this lane (past the element's last: the last one again)
  auto point = [&](int s) -> uint32_t {
    return (s + 1) * TPB <= P ? t + s * TPB : min(t + s * TPB, P - 1);
  };
  auto in_element = [&](int s) { return (s + 1) * TPB <= P || t + s * TPB < P; };

  // all of the element's loads are issued before the first use: routing codes
  // first, the factors before the gathers that wait for the codes
  T uq[PPT], gq[PPT][6], kq[PPT], bq[PPT];
  int32_t code[PPT];
  (void)code;
  if constexpr (MODE >= 1) {
#pragma unroll
    for (int s = 0; s < PPT; ++s) code[s] = ld_stream(lmap + eP + point(s));
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const uint32_t q = point(s);
    if constexpr (MODE == 0) uq[s] = ld_stream(u + eP + q);
    kq[s] = use_k ? ld_stream(kf + eP + q) : T(1);
    if constexpr (GEO == 0) {
#pragma unroll
      for (int c = 0; c < 6; ++c) gq[s][c] = ld_stream(Ge + c * P + q);
      bq[s] = use_h2 ? ld_stream(B + eP + q) : T(0);
    }
  }
  // the straight-edged form's D^T is fetched behind the forward contractions
  const DFrag<N, T, GEO == 1> af(D, lane, false);
  DFrag<N, T, GEO == 1> at;
  if constexpr (GEO == 0) at = DFrag<N, T, GEO == 1>(D, lane, true);
  __shared__ double sp[GEO == 1 ? 2 * n1 : 1];  // nodes and weights
  if constexpr (GEO == 1)
    if (t < 2 * n1) sp[t] = pts[t];
  if constexpr (MODE >= 1) {
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
      const int32_t cd = code[s];
      const int32_t g = MODE >= 2 ? (cd >= 0 ? cd : cd <= -2 ? -(cd + 2) : -1) : cd;
      const T v = u[max(g, 0)];
      uq[s] = g >= 0 ? v : T(0);
    }
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s) su[lds_point<N, T>(point(s))] = uq[s];
  __syncthreads();
#pragma unroll
  for (int x = 0; x < TPW; ++x) {
    const int tile = wv + x * NW;
    if ((x + 1) * NW <= NT || tile < NT)
      contract_tile<N, T, GEO == 1>(tile, lane, af, su, su, su, sa[0], sa[1], sa[2]);
  }
  if constexpr (GEO == 1) at = DFrag<N, T, true>(D, lane, true);
  __syncthreads();
  // metric and k
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = lds_point<N, T>(point(s));
    if constexpr (GEO == 1) {
      const int p = (int)point(s), i = p % n1, j = (p / n1) % n1, k = p / (n1 * n1);
      straight_metric((UniformD)(uintptr_t)(geo + e * 21), sp[i], sp[j], sp[k],
                      sp[n1 + i] * sp[n1 + j] * sp[n1 + k], gq[s], bq[s]);
    }
    const T ur = sa[0][q], us = sa[1][q], ut = sa[2][q];
    const T* gc = gq[s];
    T vr = gc[0] * ur + gc[1] * us + gc[2] * ut;
    T vs = gc[1] * ur + gc[3] * us + gc[4] * ut;
    T vt = gc[2] * ur + gc[4] * us + gc[5] * ut;
    if (use_k) {
      vr *= kq[s];
      vs *= kq[s];
      vt *= kq[s];
    }
    if (in_element(s)) {
      sa[0][q] = vr;
      sa[1][q] = vs;
      sa[2][q] = vt;
    }
    // the straight-edged form's factors live for one point
    if constexpr (GEO == 1) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < TPW; ++x) {
    const int tile = wv + x * NW;
    if ((x + 1) * NW <= NT || tile < NT)
      contract_tile<N, T, GEO == 1>(tile, lane, at, sa[0], sa[1], sa[2], sa[0], sa[1], sa[2]);
  }
  __syncthreads();
  double ps[2] = {0.0, 0.0};
  (void)ps;
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = (int)point(s), ql = lds_point<N, T>(q);
    T acc = (sa[0][ql] + sa[1][ql]) + sa[2][ql];
    if (use_h2) acc += h2 * bq[s] * uq[s];
    if (!in_element(s)) continue;
    if constexpr (MODE >= 2) {
      const int32_t cd = code[s];
      if (cd >= 0) {
        st_stream(acc, wf + cd);
      } else if (cd <= -2) {
        // shared copy: at its surface slot of the element's block
        T* dst = w + eP + surface_rank(q % n1, (q / n1) % n1, q / (n1 * n1), N);
        if constexpr (kNtShared)
          st_stream(acc, dst);
        else
          *dst = acc;
      }
      if constexpr (kSums > 0) {
        if (cd != -1) {  // free copies only
          ps[0] += (double)uq[s] * (double)acc;
          if constexpr (kSums == 2) ps[1] += (double)acc;
        }
      }
    } else {
      st_stream(acc, w + eP + q);
    }
  }
  // the element's sums, in a fixed order; the barrier waits for LDS only, not
  // for the stores on their way
  if constexpr (kSums > 0) {
    __shared__ double spw[NW][2];
#pragma unroll
    for (int a = 0; a < kSums; ++a) {
      const double x = wave_sum_d(ps[a]);
      if (lane == 0) spw[wv][a] = x;
    }
    if constexpr (NW > 1) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    } else {
      __syncthreads();
    }
    if (t < kSums) {
      double x = spw[0][t];
#pragma unroll
      for (int a = 1; a < NW; ++a) x += spw[a][t];
      epart[(int64_t)t * gridDim.x + e] = x;
    }
  }
}

// The same operator with 16-bit contraction operands (FP32 data): D, the u
// block and each v_a block rounded to bfloat16 (LP = 1) or IEEE half (LP = 2;
// each block scaled by its power-of-two block scale, whose maxima are reduced
// before the barriers the phases already have), FP32 accumulation.  MODE 0: u
// and w local; MODE 1: u gathered from a free vector through lmap.  Phases:
// loads -> forward contractions (3 NT tiles over the wavefronts) -> pointwise
// metric and k -> transposed contractions accumulated direction by direction
// into the (now free) input block -> stores.
template <int N, int MODE, int LP>
__global__ __launch_bounds__(MShape<N>::TPB) void ax_mfma16_kernel(
    const float* __restrict__ u, const int32_t* __restrict__ lmap, float* __restrict__ w,
    const float* __restrict__ kf, const float h2, const float* __restrict__ G,
    const float* __restrict__ B, const float* __restrict__ D, const int32_t* __restrict__ skip) {
  using S = MShape<N>;
  constexpr int n1 = S::n1, P = S::P, TPB = S::TPB, PPT = S::PPT, NT = S::NT, NW = S::NW;
  constexpr bool kScale = LP == 2;
  if (skip && *skip) return;  // uniform over the grid
  __shared__ float su[P];
  __shared__ float sa[3][P];
  __shared__ float smax[4][NW];  // block maxima of u, v_r, v_s, v_t per wavefront (LP = 2)
  float* so = su;  // output accumulator, reuses the input block after the forward phase
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t e = blockIdx.x;
  const bool use_k = kf != nullptr;
  const bool use_h2 = h2 != 0.0f;

  float uq[PPT], gq[PPT][6], kq[PPT];
  int32_t lvq[PPT];
  (void)lvq;
  if constexpr (MODE >= 1) {
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
      const int qr = t + s * TPB;
      lvq[s] = ld_stream(lmap + e * P + (qr < P ? qr : P - 1));
    }
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int qr = t + s * TPB;
    const int q = qr < P ? qr : P - 1;
    const float* g = G + e * 6 * P + q;
#pragma unroll
    for (int c = 0; c < 6; ++c) gq[s][c] = ld_stream(g + c * P);
    kq[s] = use_k ? ld_stream(kf + e * P + q) : 1.0f;
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int qr = t + s * TPB;
    const int q = qr < P ? qr : P - 1;
    if constexpr (MODE >= 1) {
      const int32_t lm = lvq[s];
      const float v = u[lm >= 0 ? lm : 0];
      uq[s] = lm >= 0 ? v : 0.0f;
    } else {
      uq[s] = ld_stream(u + e * P + q);
    }
  }
  // derivative-matrix fragments: forward A = D, transposed A = D^T
  typename Mfma16<LP>::V af16, at16;
  {
    const int row = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int l = 4 * kk + x;
      const bool ok = row < n1 && l < n1;
      af16[x] = Mfma16<LP>::cvt(ok ? D[row * n1 + l] : 0.0f);
      at16[x] = Mfma16<LP>::cvt(ok ? D[l * n1 + row] : 0.0f);
    }
  }
  if constexpr (kScale) {
    float mu = 0.0f;
#pragma unroll
    for (int s = 0; s < PPT; ++s) mu = fmaxf(mu, fabsf(uq[s]));
    mu = wave_max(mu);
    if (lane == 0) smax[0][wv] = mu;
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = t + s * TPB;
    if (q < P) su[q] = uq[s];
  }
  __syncthreads();
  {
    float sc = 1.0f;
    if constexpr (kScale) {
      float m = 0.0f;
#pragma unroll
      for (int x = 0; x < NW; ++x) m = fmaxf(m, smax[0][x]);
      sc = half_block_scale(m);
    }
    const float inv = 1.0f / sc;
    for (int job = wv; job < 3 * NT; job += NW) {
      const int dir = job / NT, tile = job - dir * NT;
      if (dir == 0) contract_tile16<n1, LP, 0, false>(su, sa[0], af16, tile, lane, sc, inv);
      else if (dir == 1) contract_tile16<n1, LP, 1, false>(su, sa[1], af16, tile, lane, sc, inv);
      else contract_tile16<n1, LP, 2, false>(su, sa[2], af16, tile, lane, sc, inv);
    }
  }
  __syncthreads();
  float mv[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = t + s * TPB;
    if (q < P) {
      const float ur = sa[0][q], us = sa[1][q], ut = sa[2][q];
      const float* gc = gq[s];
      float vr = gc[0] * ur + gc[1] * us + gc[2] * ut;
      float vs = gc[1] * ur + gc[3] * us + gc[4] * ut;
      float vt = gc[2] * ur + gc[4] * us + gc[5] * ut;
      if (use_k) {
        vr *= kq[s];
        vs *= kq[s];
        vt *= kq[s];
      }
      sa[0][q] = vr;
      sa[1][q] = vs;
      sa[2][q] = vt;
      if constexpr (kScale) {
        mv[0] = fmaxf(mv[0], fabsf(vr));
        mv[1] = fmaxf(mv[1], fabsf(vs));
        mv[2] = fmaxf(mv[2], fabsf(vt));
      }
    }
  }
  if constexpr (kScale) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float m = wave_max(mv[d]);
      if (lane == 0) smax[1 + d][wv] = m;
    }
  }
  __syncthreads();
  {
    float sc[3] = {1.0f, 1.0f, 1.0f};
    if constexpr (kScale) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        float m = 0.0f;
#pragma unroll
        for (int x = 0; x < NW; ++x) m = fmaxf(m, smax[1 + d][x]);
        sc[d] = half_block_scale(m);
      }
    }
    for (int tile = wv; tile < NT; tile += NW)
      contract_tile16<n1, LP, 0, false>(sa[0], so, at16, tile, lane, sc[0], 1.0f / sc[0]);
    __syncthreads();
    for (int tile = wv; tile < NT; tile += NW)
      contract_tile16<n1, LP, 1, true>(sa[1], so, at16, tile, lane, sc[1], 1.0f / sc[1]);
    __syncthreads();
    for (int tile = wv; tile < NT; tile += NW)
      contract_tile16<n1, LP, 2, true>(sa[2], so, at16, tile, lane, sc[2], 1.0f / sc[2]);
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = t + s * TPB;
    if (q < P) {
      float acc = so[q];
      if (use_h2) acc += h2 * ld_stream(B + e * P + q) * uq[s];
      st_stream(acc, w + e * P + q);
    }
  }
}

// The matrix-core kernel exists from N = 5 on (below that a 16-wide tile
// wastes most of its lanes).  Which kernel serves a launch: the environment
// variable SEM_AX_KERNEL = scalar | mfma forces one (read once per process),
// otherwise the measured default of prefer_mfma.
constexpr bool has_mfma(int N) { return N >= 5; }
enum class AxChoice { Auto, Scalar, Mfma };
AxChoice ax_choice() {
  static const AxChoice c = [] {
    const char* e = std::getenv("SEM_AX_KERNEL");
    if (e && std::strcmp(e, "scalar") == 0) return AxChoice::Scalar;
    if (e && std::strcmp(e, "mfma") == 0) return AxChoice::Mfma;
    return AxChoice::Auto;
  }();
  return c;
}
bool prefer_mfma(int N, bool gather, bool fp32) {
  (void)gather;
  (void)fp32;
  return N >= 5;
}

// Both gradients of w = A_L(k) u for a cotangent wbar in one pass, one element
// per workgroup (the phases of ax_line_kernel with u carried through the
// forward contractions as well): ubar = A_L(k) wbar and kbar = sum_ab (D_a wbar)
// G_ab (D_b u).  One read of the factors serves both (88 B per point instead
// of 152 with k and h2; 40 B on straight-edged elements): 8 million points, N =
// 7, 190 -> 110 us (straight-edged 84 us).
template <int N, int GEO>
__global__ __launch_bounds__((LShape<N, double>::TPB))
    __attribute__((amdgpu_waves_per_eu(N == 7 ? 5 : N == 10 ? 4 : 3))) void ax_backward_kernel(
    const double* __restrict__ u, const double* __restrict__ wbar, const double* __restrict__ kf,
    const double h2, const double* __restrict__ G, const double* __restrict__ B,
    const double* __restrict__ D, const double* __restrict__ geo, const double* __restrict__ pts,
    double* __restrict__ ubar, double* __restrict__ kbar) {
  typedef double T;
  using S = LShape<N, T>;
  constexpr int n1 = S::n1, P = S::P, KS = S::KS, PPT = S::PPT, TPB = S::TPB, NW = S::NW,
                NT = S::NT, TPW = S::TPW, SZ = n1 * S::PS;
  __shared__ T su[SZ];
  __shared__ T sa[3][SZ];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t e = blockIdx.x;
  const bool use_k = kf != nullptr;
  const bool use_h2 = h2 != 0.0;
  const T* Ge = G + e * 6 * P;
  const int64_t eP = e * P;
  auto point = [&](int s) -> uint32_t {
    return (s + 1) * TPB <= P ? t + s * TPB : min(t + s * TPB, P - 1);
  };
  auto in_element = [&](int s) { return (s + 1) * TPB <= P || t + s * TPB < P; };
  T wq[PPT], uq[PPT], gq[PPT][6], kq[PPT], bq[PPT];
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const uint32_t q = point(s);
    wq[s] = ld_stream(wbar + eP + q);
    uq[s] = ld_stream(u + eP + q);
    kq[s] = use_k ? ld_stream(kf + eP + q) : T(1);
    if constexpr (GEO == 0) {
#pragma unroll
      for (int c = 0; c < 6; ++c) gq[s][c] = ld_stream(Ge + c * P + q);
      bq[s] = use_h2 ? ld_stream(B + eP + q) : T(0);
    }
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s) su[lds_point<N, T>(point(s))] = uq[s];
  const DFrag<N, T, GEO == 1> af(D, lane, false);
  __shared__ double sp[GEO == 1 ? 2 * n1 : 1];
  if constexpr (GEO == 1)
    if (t < 2 * n1) sp[t] = pts[t];
  __syncthreads();
  auto forward = [&](const T* src) {
#pragma unroll
    for (int x = 0; x < TPW; ++x) {
      const int tile = wv + x * NW;
      if ((x + 1) * NW <= NT || tile < NT)
        contract_tile<N, T, GEO == 1>(tile, lane, af, src, src, src, sa[0], sa[1], sa[2]);
    }
    __syncthreads();
  };
  // the gradient of u at this lane's points first, then that of wbar
  T ud[PPT][3];
  forward(su);
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = lds_point<N, T>(point(s));
#pragma unroll
    for (int d = 0; d < 3; ++d) ud[s][d] = sa[d][q];
    su[q] = wq[s];
  }
  __syncthreads();
  forward(su);
  const DFrag<N, T, GEO == 1> at(D, lane, true);
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = lds_point<N, T>(point(s));
    if constexpr (GEO == 1) {
      const int p = (int)point(s), i = p % n1, j = (p / n1) % n1, k = p / (n1 * n1);
      straight_metric((UniformD)(uintptr_t)(geo + e * 21), sp[i], sp[j], sp[k],
                      sp[n1 + i] * sp[n1 + j] * sp[n1 + k], gq[s], bq[s]);
    }
    const T wr = sa[0][q], ws = sa[1][q], wt = sa[2][q];
    const T* gc = gq[s];
    T vr = gc[0] * wr + gc[1] * ws + gc[2] * wt;
    T vs = gc[1] * wr + gc[3] * ws + gc[4] * wt;
    T vt = gc[2] * wr + gc[4] * ws + gc[5] * wt;
    const T kb = ud[s][0] * vr + ud[s][1] * vs + ud[s][2] * vt;
    if (use_k) {
      vr *= kq[s];
      vs *= kq[s];
      vt *= kq[s];
    }
    if (in_element(s)) {
      st_stream(kb, kbar + eP + point(s));
      sa[0][q] = vr;
      sa[1][q] = vs;
      sa[2][q] = vt;
    }
    if constexpr (GEO == 1) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < TPW; ++x) {
    const int tile = wv + x * NW;
    if ((x + 1) * NW <= NT || tile < NT)
      contract_tile<N, T, GEO == 1>(tile, lane, at, sa[0], sa[1], sa[2], sa[0], sa[1], sa[2]);
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const uint32_t q = point(s);
    const int ql = lds_point<N, T>(q);
    T acc = (sa[0][ql] + sa[1][ql]) + sa[2][ql];
    if (use_h2) acc += h2 * bq[s] * wq[s];
    if (in_element(s)) st_stream(acc, ubar + eP + q);
  }
}

// kbar_q = sign sum_ab (D_a wbar)_q G_ab,q (D_b u)_q: the derivative of the
// operator in k contracted with a cotangent (same mapping, 72 B per point);
// sign = -1 gives the gradient of a solve (exact negation).
template <int N>
__global__ __launch_bounds__(Shape<N>::BT) void kbar_kernel(
    const double* __restrict__ u, const double* __restrict__ wb, double* __restrict__ kbar,
    const double* __restrict__ G, const double* __restrict__ D, const int64_t E,
    const double sign) {
  using S = Shape<N>;
  constexpr int n1 = S::n1, P2 = S::P2, P = S::P, EPB = S::EPB, PPT = S::PPT, TPE = S::TPE;
  __shared__ double su[EPB][P];
  __shared__ double sw[EPB][P];
  __shared__ double sD[n1 * n1];
  const int t = threadIdx.x;
  const int slot = t / TPE;
  const int tl = t - slot * TPE;
  const int64_t e = (int64_t)blockIdx.x * EPB + slot;
  const bool ok_e = slot < EPB && e < E;
  const int ss = slot < EPB ? slot : 0;
  const int64_t ec = ok_e ? e : E - 1;
  double gq[PPT][6];
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int qr = tl + s * TPE;
    const int q = qr < P ? qr : P - 1;
    const double* g = G + ec * 6 * P + q;
#pragma unroll
    for (int c = 0; c < 6; ++c) gq[s][c] = ld_stream(g + c * P);
    const double uv = ld_stream(u + ec * P + q), wv = ld_stream(wb + ec * P + q);
    if (slot < EPB && qr < P) {
      su[ss][q] = ok_e ? uv : 0.0;
      sw[ss][q] = ok_e ? wv : 0.0;
    }
  }
  for (int a = t; a < n1 * n1; a += S::BT) sD[a] = D[a];
  __syncthreads();
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = tl + s * TPE;
    if (ok_e && q < P) {
      const int i = q % n1, j = (q / n1) % n1, k = q / P2;
      double ur = 0, us = 0, ut = 0, wr = 0, ws = 0, wt = 0;
#pragma unroll
      for (int l = 0; l < n1; ++l) {
        const double dil = sD[i * n1 + l], djl = sD[j * n1 + l], dkl = sD[k * n1 + l];
        const int qr = k * P2 + j * n1 + l, qs = k * P2 + l * n1 + i, qt = l * P2 + j * n1 + i;
        ur += dil * su[ss][qr];
        us += djl * su[ss][qs];
        ut += dkl * su[ss][qt];
        wr += dil * sw[ss][qr];
        ws += djl * sw[ss][qs];
        wt += dkl * sw[ss][qt];
      }
      const double* gc = gq[s];
      const double vr = gc[0] * ur + gc[1] * us + gc[2] * ut;
      const double vs = gc[1] * ur + gc[3] * us + gc[4] * ut;
      const double vt = gc[2] * ur + gc[4] * us + gc[5] * ut;
      st_stream(sign * (wr * vr + ws * vs + wt * vt), kbar + e * P + q);
    }
  }
}

template <typename T>
__global__ void mass_kernel(int64_t n, const T* __restrict__ B, const T* __restrict__ u,
                            T* __restrict__ w) {
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n;
       q += (int64_t)gridDim.x * blockDim.x)
    w[q] = B[q] * u[q];
}

// A launch that, when ev0 / ev1 are given, has the runtime stamp them with the
// kernel's own start and end (the solve's operator timing): an event recorded
// before the launch would also count the dispatch latency.
#define SEM_LAUNCH(ev0, ev1, kernel, grid, block, stream, ...)                           \
  do {                                                                                 \
    if ((ev0) != nullptr || (ev1) != nullptr)                                          \
      hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, ev0, ev1, 0, __VA_ARGS__); \
    else                                                                               \
      hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);                 \
  } while (0)

template <int N, int LP>
hipError_t run_ax_mfma16(const sem_mesh* m, const float* u, const int32_t* lmap, float* w,
                         const float* k, float h2, const float* G, const float* B, const float* D,
                         hipStream_t s, const int32_t* skip, hipEvent_t ev0, hipEvent_t ev1) {
  const dim3 grid((unsigned)m->E), block(MShape<N>::TPB);
  if (lmap)
    SEM_LAUNCH(ev0, ev1, (ax_mfma16_kernel<N, 1, LP>), grid, block, s, u, lmap, w, k, h2, G, B, D,
               skip);
  else
    SEM_LAUNCH(ev0, ev1, (ax_mfma16_kernel<N, 0, LP>), grid, block, s, u, lmap, w, k, h2, G, B, D,
               skip);
  return hipGetLastError();
}

// the nodes and weights behind D in the FP64 buffer (see sem_setup_mesh)
inline const double* gll_points(const sem_mesh* m) {
  return m->D64.as<double>() + m->n1 * m->n1 + m->n1;
}

#define SEM_AX_LINE(MD, lm, wfree, ep)                                                          \
  do {                                                                                         \
    constexpr int kGeo = sizeof(T) == 8 ? 1 : 0;                                               \
    if (kGeo && m->straight)                                                                   \
      SEM_LAUNCH(ev0, ev1, (ax_line_kernel<N, T, MD, kGeo>), grid, block, s, u, lm, w, k, h2, G, \
                 B, D, m->geo.as<double>(), gll_points(m), skip, wfree, ep);                   \
    else                                                                                       \
      SEM_LAUNCH(ev0, ev1, (ax_line_kernel<N, T, MD, 0>), grid, block, s, u, lm, w, k, h2, G, B, \
                 D, (const double*)nullptr, (const double*)nullptr, skip, wfree, ep);          \
  } while (0)

template <int N, typename T>
hipError_t run_ax_line(const sem_mesh* m, const T* u, const int32_t* lmap, T* w, const T* k, T h2,
                       const T* G, const T* B, const T* D, hipStream_t s, const int32_t* skip,
                       hipEvent_t ev0, hipEvent_t ev1) {
  const dim3 grid((unsigned)m->E), block(LShape<N, T>::TPB);
  if (lmap)
    SEM_AX_LINE(1, lmap, (T*)nullptr, (double*)nullptr);
  else
    SEM_AX_LINE(0, lmap, (T*)nullptr, (double*)nullptr);
  return hipGetLastError();
}

template <int N, typename T>
hipError_t run_ax(const sem_mesh* m, const T* u, const int32_t* lmap, T* w, const T* k, T h2,
                  const T* G, const T* B, const T* D, hipStream_t s, const int32_t* skip, int lp,
                  hipEvent_t ev0, hipEvent_t ev1) {
  if constexpr (std::is_same<T, float>::value) {
    if (lp == 1) return run_ax_mfma16<N, 1>(m, u, lmap, w, k, h2, G, B, D, s, skip, ev0, ev1);
    if (lp == 2) return run_ax_mfma16<N, 2>(m, u, lmap, w, k, h2, G, B, D, s, skip, ev0, ev1);
  }
  if (lp != 0) return hipErrorInvalidValue;
  if constexpr (has_mfma(N)) {
    const AxChoice c = ax_choice();
    const bool mfma = c == AxChoice::Auto ? prefer_mfma(N, lmap != nullptr, sizeof(T) == 4)
                                          : c == AxChoice::Mfma;
    if (mfma) return run_ax_line<N, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, ev0, ev1);
  }
  using S = Shape<N>;
  const int64_t grid = (m->E + S::EPB - 1) / S::EPB;
  if (lmap)
    SEM_LAUNCH(ev0, ev1, (ax_kernel<N, T, true>), dim3((unsigned)grid), dim3(S::BT), s, u, lmap,
               w, k, h2, G, B, D, m->E, skip);
  else
    SEM_LAUNCH(ev0, ev1, (ax_kernel<N, T, false>), dim3((unsigned)grid), dim3(S::BT), s, u, lmap,
               w, k, h2, G, B, D, m->E, skip);
  return hipGetLastError();
}

template <int N>
hipError_t run_kbar(const sem_mesh* m, const double* u, const double* wb, double* kbar,
                    double sign, hipStream_t s) {
  using S = Shape<N>;
  const int64_t grid = (m->E + S::EPB - 1) / S::EPB;
  hipLaunchKernelGGL((kbar_kernel<N>), dim3((unsigned)grid), dim3(S::BT), 0, s, u, wb, kbar,
                     m->G64.as<double>(), m->D64.as<double>(), m->E, sign);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_ax(const sem_mesh* m, const T* u, const int32_t* lmap, T* w, const T* k, T h2,
                     const T* G, const T* B, const T* D, hipStream_t s, const int32_t* skip,
                     int lp, hipEvent_t ev0, hipEvent_t ev1) {
  switch (m->N) {
    case 1: return run_ax<1, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 2: return run_ax<2, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 3: return run_ax<3, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 4: return run_ax<4, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 5: return run_ax<5, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 6: return run_ax<6, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 7: return run_ax<7, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 8: return run_ax<8, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 9: return run_ax<9, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    case 10: return run_ax<10, T>(m, u, lmap, w, k, h2, G, B, D, s, skip, lp, ev0, ev1);
    default: return hipErrorInvalidValue;
  }
}
template hipError_t launch_ax<double>(const sem_mesh*, const double*, const int32_t*, double*,
                                      const double*, double, const double*, const double*,
                                      const double*, hipStream_t, const int32_t*, int, hipEvent_t,
                                      hipEvent_t);
template hipError_t launch_ax<float>(const sem_mesh*, const float*, const int32_t*, float*,
                                     const float*, float, const float*, const float*,
                                     const float*, hipStream_t, const int32_t*, int, hipEvent_t,
                                     hipEvent_t);

namespace {
template <int N, typename T>
hipError_t run_ax_split(const sem_mesh* m, const T* u, T* wf, T* w, double* epart, bool mean_sums,
                        const T* k, T h2, const T* G, const T* B, const T* D, hipStream_t s,
                        const int32_t* skip, hipEvent_t ev0, hipEvent_t ev1) {
  if constexpr (has_mfma(N)) {
    // shared-copy results stay in the memory-side cache for the segmented
    // sum when the local array fits well inside it (256 MB): plain stores up
    // to m->ax_nt_bytes, 128 MB by default (the 32x32x16, N = 7 box: 67 MB,
    // 1.1 % faster per iteration), nontemporal above (the 32^3, N = 9 cube:
    // 262 MB, 2.2 %) (a run-time switch in the kernel cost what the
    // nontemporal stores save).  Sums: p w and sum(w) (MODE 2 / 3) when the
    // solve projects out the constants, p w alone (MODE 6 / 7) otherwise,
    // none without epart (MODE 4 / 5).
    const bool plain = m->nL * (int64_t)sizeof(T) <= m->ax_nt_bytes;
    const int mode = !epart ? (plain ? 4 : 5) : mean_sums ? (plain ? 2 : 3) : (plain ? 6 : 7);
    const dim3 grid((unsigned)m->E), block(LShape<N, T>::TPB);
    const int32_t* lm = m->lmap2.as<int32_t>();
#define SEM_SPLIT_CASE(MD) \
  case MD:                 \
    SEM_AX_LINE(MD, lm, wf, epart); \
    break;
    switch (mode) {
      SEM_SPLIT_CASE(2)
      SEM_SPLIT_CASE(3)
      SEM_SPLIT_CASE(4)
      SEM_SPLIT_CASE(5)
      SEM_SPLIT_CASE(6)
      SEM_SPLIT_CASE(7)
    }
#undef SEM_SPLIT_CASE
    return hipGetLastError();
  } else {
    return hipErrorNotSupported;
  }
}
}  // namespace

bool ax_split_available(const sem_mesh* m) {
  // SEM_AX_SPLIT=0 (read once) keeps the gather form in the solve
  static const bool enabled = [] {
    const char* e = std::getenv("SEM_AX_SPLIT");
    return !(e && std::strcmp(e, "0") == 0);
  }();
  if (!enabled || !has_mfma(m->N) || !m->lmap2.p || !m->split_ok) return false;
  const AxChoice c = ax_choice();
  return c == AxChoice::Auto ? prefer_mfma(m->N, true, false) : c == AxChoice::Mfma;
}

template <typename T>
hipError_t launch_ax_split(const sem_mesh* m, const T* u, T* wf, T* wL, double* epart,
                           bool mean_sums, const T* k, T h2, const T* G, const T* B, const T* D,
                           hipStream_t s, const int32_t* skip, hipEvent_t ev0, hipEvent_t ev1) {
  if (!ax_split_available(m)) return hipErrorNotSupported;
  switch (m->N) {
    case 5: return run_ax_split<5, T>(m, u, wf, wL, epart, mean_sums, k, h2, G, B, D, s, skip,
                                           ev0, ev1);
    case 6: return run_ax_split<6, T>(m, u, wf, wL, epart, mean_sums, k, h2, G, B, D, s, skip,
                                           ev0, ev1);
    case 7: return run_ax_split<7, T>(m, u, wf, wL, epart, mean_sums, k, h2, G, B, D, s, skip,
                                           ev0, ev1);
    case 8: return run_ax_split<8, T>(m, u, wf, wL, epart, mean_sums, k, h2, G, B, D, s, skip,
                                           ev0, ev1);
    case 9: return run_ax_split<9, T>(m, u, wf, wL, epart, mean_sums, k, h2, G, B, D, s, skip,
                                           ev0, ev1);
    case 10: return run_ax_split<10, T>(m, u, wf, wL, epart, mean_sums, k, h2, G, B, D, s, skip,
                                           ev0, ev1);
    default: return hipErrorNotSupported;
  }
}
template hipError_t launch_ax_split<double>(const sem_mesh*, const double*, double*, double*,
                                            double*, bool, const double*, double, const double*,
                                            const double*, const double*, hipStream_t,
                                            const int32_t*, hipEvent_t, hipEvent_t);
template hipError_t launch_ax_split<float>(const sem_mesh*, const float*, float*, float*, double*,
                                           bool, const float*, float, const float*, const float*,
                                           const float*, hipStream_t, const int32_t*, hipEvent_t,
                                           hipEvent_t);

hipError_t launch_ax_kbar(const sem_mesh* m, const double* u, const double* wbar, double* kbar,
                          double sign, hipStream_t s) {
  switch (m->N) {
    case 1: return run_kbar<1>(m, u, wbar, kbar, sign, s);
    case 2: return run_kbar<2>(m, u, wbar, kbar, sign, s);
    case 3: return run_kbar<3>(m, u, wbar, kbar, sign, s);
    case 4: return run_kbar<4>(m, u, wbar, kbar, sign, s);
    case 5: return run_kbar<5>(m, u, wbar, kbar, sign, s);
    case 6: return run_kbar<6>(m, u, wbar, kbar, sign, s);
    case 7: return run_kbar<7>(m, u, wbar, kbar, sign, s);
    case 8: return run_kbar<8>(m, u, wbar, kbar, sign, s);
    case 9: return run_kbar<9>(m, u, wbar, kbar, sign, s);
    case 10: return run_kbar<10>(m, u, wbar, kbar, sign, s);
    default: return hipErrorInvalidValue;
  }
}

namespace {
template <int N>
hipError_t run_backward(const sem_mesh* m, const double* u, const double* wbar, const double* k,
                        double h2, double* ubar, double* kbar, hipStream_t s) {
  const dim3 grid((unsigned)m->E), block(LShape<N, double>::TPB);
  const double *G = m->G64.as<double>(), *B = m->B64.as<double>(), *D = m->D64.as<double>();
  if (m->straight)
    hipLaunchKernelGGL((ax_backward_kernel<N, 1>), grid, block, 0, s, u, wbar, k, h2, G, B, D,
                       m->geo.as<double>(), gll_points(m), ubar, kbar);
  else
    hipLaunchKernelGGL((ax_backward_kernel<N, 0>), grid, block, 0, s, u, wbar, k, h2, G, B, D,
                       (const double*)nullptr, (const double*)nullptr, ubar, kbar);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_ax_backward(const sem_mesh* m, const double* u, const double* wbar,
                              const double* k, double h2, double* ubar, double* kbar,
                              hipStream_t s) {
  // the matrix-core form writes ubar and kbar element by element after reading
  // u and wbar there; forced scalar operators (and N < 5) run the two apart
  if (has_mfma(m->N) && ax_choice() != AxChoice::Scalar) {
    switch (m->N) {
      case 5: return run_backward<5>(m, u, wbar, k, h2, ubar, kbar, s);
      case 6: return run_backward<6>(m, u, wbar, k, h2, ubar, kbar, s);
      case 7: return run_backward<7>(m, u, wbar, k, h2, ubar, kbar, s);
      case 8: return run_backward<8>(m, u, wbar, k, h2, ubar, kbar, s);
      case 9: return run_backward<9>(m, u, wbar, k, h2, ubar, kbar, s);
      case 10: return run_backward<10>(m, u, wbar, k, h2, ubar, kbar, s);
      default: break;
    }
  }
  const hipError_t e = launch_ax<double>(m, wbar, nullptr, ubar, k, h2, m->G64.as<double>(),
                                         m->B64.as<double>(), m->D64.as<double>(), s);
  return e != hipSuccess ? e : launch_ax_kbar(m, u, wbar, kbar, 1.0, s);
}

template <typename T>
hipError_t launch_mass(int64_t n, const T* B, const T* u, T* w, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>((n + kVecBlock - 1) / kVecBlock, 8192);
  hipLaunchKernelGGL((mass_kernel<T>), dim3((unsigned)std::max<int64_t>(blocks, 1)),
                     dim3(kVecBlock), 0, s, n, B, u, w);
  return hipGetLastError();
}
template hipError_t launch_mass<double>(int64_t, const double*, const double*, double*,
                                        hipStream_t);
template hipError_t launch_mass<float>(int64_t, const float*, const float*, float*, hipStream_t);

}  // namespace sem
