// p-multigrid V-cycle on the device.
//
// V_l(r):  x = Cheb_l(r)                       pre-smoothing (fourth kind, Jacobi)
//          x += P_l V_{l+1}(P_l^T (r - A_l x))  coarse correction
//          x += Cheb_l(r - A_l x)               post-smoothing
// and a fixed number of Jacobi-PCG iterations on the coarsest level (Sec. 2.2
// names p-multigrid with Chebyshev-accelerated smoothing as the default
// pressure preconditioner).  Vectors are free-unique per level; P_l
// interpolates element blocks (tensor product of the 1-D interpolation J_l)
// and averages the copies of each fine node, P_l^T divides each fine value by
// its number of copies, applies J_l^T per element and sums the copies of each
// coarse node (on conforming meshes both through a node's first copy alone, which
// is the same: k_transfer).  Every launch returns at once when the enclosing flexible CG
// has finished, so overshooting iterations cost nothing.
#include <type_traits>

#include "pmg.hpp"

namespace sem {
namespace {

constexpr int kN1 = kMaxOrder + 1;
constexpr int kP3 = kN1 * kN1 * kN1;
constexpr int kInterpThreads = 256;

#define GRID_STRIDE(idx, n)                                                        \
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < (n); \
       idx += (int64_t)gridDim.x * blockDim.x)

// out_L = (M x M x M) in, one element per workgroup; the three contractions
// (along i, then j, then k) go through LDS
template <typename T, int MODE>
__global__ __launch_bounds__(kInterpThreads) void interp_kernel(
    int n_in, int n_out, const T* __restrict__ M, const T* __restrict__ in,
    const int32_t* __restrict__ lmap, const int32_t* __restrict__ seg, T* __restrict__ out,
    const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ T sM[kN1 * kN1];
  __shared__ T A[kP3];
  __shared__ T B[kP3];
  const int64_t e = blockIdx.x;
  const int t = threadIdx.x, nt = blockDim.x;
  const int p_in = n_in * n_in * n_in, p_out = n_out * n_out * n_out;
  for (int a = t; a < n_out * n_in; a += nt) sM[a] = M[a];
  for (int q = t; q < p_in; q += nt) {
    const int64_t idx = e * p_in + q;
    T v;
    if constexpr (MODE == 0) {
      v = in[idx];
    } else {
      const int32_t g = lmap[idx];
      v = g >= 0 ? in[g] : T(0);
      if constexpr (MODE == 2) {
        if (g >= 0) v = v / (T)(seg[g + 1] - seg[g]);
      }
    }
    A[q] = v;
  }
  __syncthreads();
  for (int o = t; o < n_in * n_in * n_out; o += nt) {  // along i
    const int a = o % n_out, kj = o / n_out;
    T s = T(0);
    for (int i = 0; i < n_in; ++i) s += sM[a * n_in + i] * A[kj * n_in + i];
    B[o] = s;
  }
  __syncthreads();
  for (int o = t; o < n_in * n_out * n_out; o += nt) {  // along j
    const int a = o % n_out, b = (o / n_out) % n_out, k = o / (n_out * n_out);
    T s = T(0);
    for (int j = 0; j < n_in; ++j) s += sM[b * n_in + j] * B[(k * n_in + j) * n_out + a];
    A[o] = s;
  }
  __syncthreads();
  const int n2 = n_out * n_out;
  for (int o = t; o < p_out; o += nt) {  // along k
    const int ba = o % n2, c = o / n2;
    T s = T(0);
    for (int k = 0; k < n_in; ++k) s += sM[c * n_in + k] * A[k * n2 + ba];
    out[e * p_out + o] = s;
  }
}

// The same transfers where the copies of a fine node interpolate to one value
// (a conforming mesh, checked at the set-up), one wavefront per element and
// sizes known at compile time.  Only a node's first copy (omap, else -1) takes
// part: PROLONG adds the interpolated value to x there (x: the free vector of
// the fine level), the restriction reads the residual there and counts it as
// zero at the other copies, whose interpolation weights are the same.  Bound by
// the fine level's map and gathers.  32x32x16 elements, FP32, N = 7 -> 3 and 3
// -> 1: prolongation 17 and 8 us (with every copy stored, then averaged: 88
// together), restriction 13 and 6 us (every copy read and divided by their
// number: 55 together).
template <typename T, int NI, int NO, bool PROLONG>
__global__ __launch_bounds__(64) void k_transfer(const T* __restrict__ M, const T* __restrict__ in,
                                                 const int32_t* __restrict__ map_in,
                                                 const int32_t* __restrict__ omap,
                                                 T* __restrict__ out,
                                                 const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int PI = NI * NI * NI, PO = NO * NO * NO, S1 = NI * NI * NO, S2 = NI * NO * NO;
  constexpr int QI = (PI + 63) / 64, QO = (PO + 63) / 64;
  __shared__ T sM[NO * NI];
  __shared__ T A[PI > S2 ? PI : S2];
  __shared__ T B[S1];
  const int64_t e = blockIdx.x;
  const int t = threadIdx.x;
  int32_t gi[QI], go[QO];
  T xo[QO];
  const int32_t* mi = (PROLONG ? map_in : omap) + e * PI;
#pragma unroll
  for (int a = 0; a < QI; ++a) gi[a] = t + 64 * a < PI ? mi[t + 64 * a] : -1;
  if constexpr (PROLONG) {
#pragma unroll
    for (int a = 0; a < QO; ++a) go[a] = t + 64 * a < PO ? omap[e * PO + t + 64 * a] : -1;
  }
  for (int a = t; a < NO * NI; a += 64) sM[a] = M[a];
  T v[QI];
#pragma unroll
  for (int a = 0; a < QI; ++a) v[a] = gi[a] >= 0 ? in[gi[a]] : T(0);
  if constexpr (PROLONG) {
#pragma unroll
    for (int a = 0; a < QO; ++a) xo[a] = go[a] >= 0 ? out[go[a]] : T(0);
  }
#pragma unroll
  for (int a = 0; a < QI; ++a)
    if (t + 64 * a < PI) A[t + 64 * a] = v[a];
  __syncthreads();
#pragma unroll
  for (int o = t; o < S1; o += 64) {  // along i
    const int a = o % NO, kj = o / NO;
    T s = T(0);
#pragma unroll
    for (int i = 0; i < NI; ++i) s += sM[a * NI + i] * A[kj * NI + i];
    B[o] = s;
  }
  __syncthreads();
#pragma unroll
  for (int o = t; o < S2; o += 64) {  // along j
    const int a = o % NO, b = (o / NO) % NO, k = o / (NO * NO);
    T s = T(0);
#pragma unroll
    for (int j = 0; j < NI; ++j) s += sM[b * NI + j] * B[(k * NI + j) * NO + a];
    A[o] = s;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < QO; ++q) {  // along k
    const int o = t + 64 * q;
    if (o >= PO) break;
    const int ba = o % (NO * NO), c = o / (NO * NO);
    T s = T(0);
#pragma unroll
    for (int k = 0; k < NI; ++k) s += sM[c * NI + k] * A[k * NO * NO + ba];
    if constexpr (PROLONG) {
      if (go[q] >= 0) out[go[q]] = xo[q] + s;
    } else {
      out[e * PO + o] = s;
    }
  }
}

// omap[q] = the free node of local point q where q is its first copy, else -1
__global__ void k_first_copies(int64_t nL, const int32_t* __restrict__ lmap,
                               const int32_t* __restrict__ seg, const int32_t* __restrict__ perm,
                               int32_t* __restrict__ omap) {
  GRID_STRIDE(q, nL) {
    const int32_t g = lmap[q];
    omap[q] = g >= 0 && perm[seg[g]] == (int32_t)q ? g : -1;
  }
}

// some values in [-1, 1] without a pattern in the node number
__global__ void k_scatter_values(int64_t n, double* __restrict__ x) {
  GRID_STRIDE(g, n) {
    uint32_t h = (uint32_t)g * 2654435761u;
    h ^= h >> 15;
    h *= 2246822519u;
    h ^= h >> 13;
    x[g] = (double)(int32_t)h * (1.0 / 2147483648.0);
  }
}

// counts copies whose value is not that of their node's first copy
__global__ void k_copies_differ(int64_t nL, const int32_t* __restrict__ lmap,
                                const int32_t* __restrict__ seg, const int32_t* __restrict__ perm,
                                const double* __restrict__ vL, int* __restrict__ count) {
  GRID_STRIDE(q, nL) {
    const int32_t g = lmap[q];
    if (g >= 0 && !(fabs(vL[q] - vL[perm[seg[g]]]) <= 1e-10)) atomicAdd(count, 1);
  }
}

// out[g] = sum of the copies of free node g
template <typename T>
__global__ void k_seg_sum(int64_t nf, const int32_t* __restrict__ seg,
                          const int32_t* __restrict__ perm, const T* __restrict__ vL,
                          T* __restrict__ out, const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  GRID_STRIDE(g, nf) out[g] = segment_sum<T>(perm, vL, seg[g], seg[g + 1]);
}

// x[g] += mean of the copies of free node g
template <typename T>
__global__ void k_seg_add_avg(int64_t nf, const int32_t* __restrict__ seg,
                              const int32_t* __restrict__ perm, const T* __restrict__ vL,
                              T* __restrict__ x, const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  GRID_STRIDE(g, nf) {
    const int32_t a = seg[g], b = seg[g + 1];
    x[g] += segment_sum<T>(perm, vL, a, b) / (T)(b - a);
  }
}

// r[g] = b[g] - sum of the copies of free node g
template <typename T>
__global__ void k_seg_sub(int64_t nf, const int32_t* __restrict__ seg,
                          const int32_t* __restrict__ perm, const T* __restrict__ vL,
                          const T* __restrict__ b, T* __restrict__ r,
                          const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  GRID_STRIDE(g, nf) r[g] = b[g] - segment_sum<T>(perm, vL, seg[g], seg[g + 1]);
}

// r[g] -= sum of the copies of free node g (in place)
template <typename T>
__global__ void k_seg_dec(int64_t nf, const int32_t* __restrict__ seg,
                          const int32_t* __restrict__ perm, const T* __restrict__ vL,
                          T* __restrict__ r, const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  GRID_STRIDE(g, nf) r[g] -= segment_sum<T>(perm, vL, seg[g], seg[g + 1]);
}

// The same residuals from the split operator's output (levels of order >= 5
// that carry its routing): w at the single-copy nodes [0, n1) is read from
// wf, contiguous; only the shared nodes [n1, nf) sum their copies, from the
// elements' surface slots.  SUB: r = b - A d; else r -= A d.  A thread takes
// kResSingle nodes of the first range and kResShared of the second: the shared
// nodes' chains (offsets, copy indices, copies) overlap each other and the
// first range's stream.  FP32, 32x32x16 elements, N = 7: 30.3 us (a chunk of each
// range per block, one node at a time) -> 21.1 us, 5.0 TB/s; 24^3 elements, N = 9:
// 45.3 -> 31.5 us.
constexpr int kResSingle = 4, kResShared = 2;
template <typename T, bool SUB>
__global__ __launch_bounds__(kVecBlock) void k_split_res(
    int64_t n1, int64_t nf, const int32_t* __restrict__ seg, const int32_t* __restrict__ perm,
    const T* __restrict__ wf, const T* __restrict__ wL, const T* __restrict__ b,
    T* __restrict__ r, const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  const int64_t g1 = (int64_t)blockIdx.x * (kResSingle * kVecBlock) + threadIdx.x;
  const int64_t g2 = n1 + (int64_t)blockIdx.x * (kResShared * kVecBlock) + threadIdx.x;
  int32_t lo[kResShared], hi[kResShared], idx[kResShared][8];
  T rs[kResShared], r1[kResSingle], w1[kResSingle];
#pragma unroll
  for (int i = 0; i < kResShared; ++i) {
    const int64_t g = g2 + i * kVecBlock;
    const bool in = g < nf;
    lo[i] = in ? seg[g] : 0;
    hi[i] = in ? seg[g + 1] : 0;
    rs[i] = in ? (SUB ? b[g] : r[g]) : T(0);
  }
#pragma unroll
  for (int i = 0; i < kResSingle; ++i) {
    const int64_t g = g1 + i * kVecBlock;
    const bool in = g < n1;
    r1[i] = in ? (SUB ? b[g] : r[g]) : T(0);
    w1[i] = in ? wf[g] : T(0);
  }
#pragma unroll
  for (int i = 0; i < kResShared; ++i)
#pragma unroll
    for (int c = 0; c < 8; ++c) idx[i][c] = lo[i] + c < hi[i] ? perm[lo[i] + c] : -1;
#pragma unroll
  for (int i = 0; i < kResSingle; ++i) {
    const int64_t g = g1 + i * kVecBlock;
    if (g < n1) r[g] = r1[i] - w1[i];
  }
#pragma unroll
  for (int i = 0; i < kResShared; ++i) {
    const int64_t g = g2 + i * kVecBlock;
    T v[8], sum = T(0);
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = idx[i][c] >= 0 ? wL[idx[i][c]] : T(0);
#pragma unroll
    for (int c = 0; c < 8; ++c) sum += v[c];
    for (int32_t c = lo[i] + 8; c < hi[i]; ++c) sum += wL[perm[c]];
    if (g < nf) r[g] = rs[i] - sum;
  }
}

template <typename T>
__global__ void k_vadd(int64_t n, T* __restrict__ x, const T* __restrict__ y,
                       const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  GRID_STRIDE(g, n) x[g] += y[g];
}

unsigned grid_for(int64_t n) {
  const int64_t b = (n + kVecBlock - 1) / kVecBlock;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 16384));
}

template <typename T>
const T* mat(const DevBuf& b64, const DevBuf& b32) {
  if constexpr (sizeof(T) == 8) return b64.as<double>();
  else return b32.as<float>();
}

template <typename T>
const Op<T>& op_of(const PmgLevel& L) {
  if constexpr (sizeof(T) == 8) return L.op64;
  else return L.op32;
}

template <typename T>
const T* dinv_of(const PmgLevel& L) {
  if constexpr (sizeof(T) == 8) return L.dinv64;
  else return L.dinv32;
}

template <typename T>
T* local_scratch(const sem_mesh* m) {
  SolveWork& W = *m->work;
  return W.vec<T>(sizeof(T) == 8 ? W.wL : W.wL32, m->nL);
}

// The additive Schwarz sum fused with the Chebyshev recurrence: q = sum of
// the box copies of free node g (q = S r_k), then at STEP 0 d = ca q, later
// d = ca d + cb q, and z = d_0 + d_1 at step 1 (neither z nor, at step 0, its
// store is needed before), z += d from step 2 on.  `add`: z += all of them
// (z holds the iterate that the smoothing corrects).  LAST: d is not kept.
// Bound by its stream, of which the copies' indices are as much as the copies:
// 29-33 us a step (average of the two smoothing levels of 32x32x16 elements, N =
// 7).  Four steps and the correction pass 12 vectors instead of 17.
constexpr int kSumNodes = 2;  // (one: 5-9 % more time, four: 6-12 %; N = 7 and 9)
template <typename T, int STEP, bool LAST>
__global__ __launch_bounds__(kVecBlock) void k_schw_sum_cheb(int64_t nf, const int32_t* __restrict__ seg,
                                const int32_t* __restrict__ perm, const T* __restrict__ box,
                                T* __restrict__ d, T* __restrict__ z, T ca, T cb, bool add,
                                const int32_t* __restrict__ skip) {
  if (skip && *skip) return;
  // kSumNodes nodes at once: their chains offsets -> indices -> copies overlap
  const int64_t n0 = (int64_t)blockIdx.x * (kSumNodes * kVecBlock) + threadIdx.x;
  int32_t a[kSumNodes], b[kSumNodes], idx[kSumNodes][8];
  T d0[kSumNodes], z0[kSumNodes], q[kSumNodes];
#pragma unroll
  for (int i = 0; i < kSumNodes; ++i) {
    const int64_t g = n0 + i * kVecBlock;
    const bool in = g < nf;
    a[i] = in ? seg[g] : 0;
    b[i] = in ? seg[g + 1] : 0;
    d0[i] = STEP > 0 && in ? d[g] : T(0);
    z0[i] = (STEP > 1 || ((STEP == 1 || LAST) && add)) && in ? z[g] : T(0);
  }
#pragma unroll
  for (int i = 0; i < kSumNodes; ++i)
#pragma unroll
    for (int c = 0; c < 8; ++c) idx[i][c] = a[i] + c < b[i] ? perm[a[i] + c] : -1;
#pragma unroll
  for (int i = 0; i < kSumNodes; ++i) {
    T v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = idx[i][c] >= 0 ? box[idx[i][c]] : T(0);
    q[i] = T(0);
#pragma unroll
    for (int c = 0; c < 8; ++c) q[i] += v[c];
    for (int32_t c = a[i] + 8; c < b[i]; ++c) q[i] += box[perm[c]];
  }
#pragma unroll
  for (int i = 0; i < kSumNodes; ++i) {
    const int64_t g = n0 + i * kVecBlock;
    if (g >= nf) break;
    const T dg = STEP > 0 ? ca * d0[i] + cb * q[i] : ca * q[i];
    if constexpr (!LAST) d[g] = dg;
    if constexpr (STEP > 0 || LAST) z[g] = z0[i] + (STEP == 1 ? d0[i] + dg : dg);
  }
}

template <typename T>
T* box_of(const SchwarzDev& X) {
  if constexpr (sizeof(T) == 8) return X.box64.as<double>();
  else return X.box32.as<float>();
}

// r = b - A d (sub) or r -= A d on one level: the split operator and
// k_split_res where the level carries the split routing (order >= 5: the
// single-copy nodes skip the gather of their copies), else the gather form
// and a segmented sum over all free nodes
template <typename T>
sem_status level_residual(Pmg& P, PmgLevel& L, const Op<T>& op, const T* d, const T* b, T* r,
                          bool sub, const int32_t* skip, hipStream_t s) {
  const sem_mesh* m = L.m;
  SolveWork& W = *m->work;
  const int64_t nf = m->n_free;
  T* wL = local_scratch<T>(m);
  if (!wL) return fail(SEM_ENOMEM, "multigrid work space");
  sem_status st;
  if (op.lp == 0 && ax_split_available(m)) {
    T* wf = P.vec<T>(L, 7);
    if (!wf) return fail(SEM_ENOMEM, "multigrid work space");
    if ((st = apply_op<T>(m, W, op, d, wL, s, false, wf, nullptr))) return st;
    const int32_t* seg = m->fseg.as<int32_t>();
    const int32_t* perm = m->fperm2.as<int32_t>();
    const int64_t per1 = kResSingle * kVecBlock, per2 = kResShared * kVecBlock;
    const dim3 grid((unsigned)std::max((m->n_single + per1 - 1) / per1,
                                       (nf - m->n_single + per2 - 1) / per2));
    if (sub)
      hipLaunchKernelGGL((k_split_res<T, true>), grid, dim3(kVecBlock), 0, s,
                         m->n_single, nf, seg, perm, wf, wL, b, r, skip);
    else
      hipLaunchKernelGGL((k_split_res<T, false>), grid, dim3(kVecBlock), 0, s,
                         m->n_single, nf, seg, perm, wf, wL, b, r, skip);
  } else {
    if ((st = apply_op<T>(m, W, op, d, wL, s, false))) return st;
    const int32_t* seg = m->fseg.as<int32_t>();
    const int32_t* perm = m->fperm.as<int32_t>();
    if (sub)
      hipLaunchKernelGGL((k_seg_sub<T>), dim3(grid_for(nf)), dim3(kVecBlock), 0, s, nf, seg, perm,
                         wL, b, r, skip);
    else
      hipLaunchKernelGGL((k_seg_dec<T>), dim3(grid_for(nf)), dim3(kVecBlock), 0, s, nf, seg, perm,
                         wL, r, skip);
  }
  SEM_CHECK_LAUNCH("level residual");
  return SEM_OK;
}

// z = S r: local fast-diagonalisation solves, then the sum over box copies
template <typename T>
sem_status schwarz_apply(const PmgLevel& L, const T* r, T* z, const int32_t* skip,
                         hipStream_t s) {
  const sem_mesh* m = L.m;
  T* box = box_of<T>(L.sch);
  if (!box) return fail(SEM_EINVAL, "Schwarz factors missing");
  SEM_HIP(launch_fdm<T>(L.sch, m->E, r, box, skip, s));
  hipLaunchKernelGGL((k_seg_sum<T>), dim3(grid_for(m->n_free)), dim3(kVecBlock), 0, s, m->n_free,
                     L.sch.xseg.as<int32_t>(), L.sch.xperm.as<int32_t>(), box, z, skip);
  SEM_CHECK_LAUNCH("Schwarz sum");
  return SEM_OK;
}

// z = p_m(S A) S r (add: z += it) with the fourth-kind coefficients (as the
// Jacobi version).
// Each Schwarz sum carries the recurrence's d and z update (k_schw_sum_cheb),
// and the first residual r_1 = r - A d_0 is formed from r directly.
template <typename T>
sem_status cheb_schwarz(Pmg& P, PmgLevel& L, const T* r, T* z, bool add, const CgScalars* outer,
                        hipStream_t s, int* applies) {
  const sem_mesh* m = L.m;
  const int64_t nf = m->n_free;
  const int32_t* skip = outer ? &outer->done : nullptr;
  T* d = P.vec<T>(L, 5);
  T* rk = P.vec<T>(L, 6);
  T* box = box_of<T>(L.sch);
  if (!d || !rk) return fail(SEM_ENOMEM, "multigrid work space");
  if (!box) return fail(SEM_EINVAL, "Schwarz factors missing");
  Op<T> op = op_of<T>(L);
  op.skip = skip;
  const double lmax = L.rho_hat;
  const int32_t* xseg = L.sch.xseg.as<int32_t>();
  const int32_t* xperm = L.sch.xperm.as<int32_t>();
  sem_status st;
  const dim3 sum_grid((unsigned)((nf + kSumNodes * kVecBlock - 1) / (kSumNodes * kVecBlock)));
  auto sum = [&](int k, double ca, double cb) {
    const bool last = k + 1 == P.smooth_order;
#define SEM_SUM(STEP, LAST)                                                                       \
  hipLaunchKernelGGL((k_schw_sum_cheb<T, STEP, LAST>), sum_grid, dim3(kVecBlock), 0, s,           \
                     nf, xseg, xperm, box, d, z, (T)ca, (T)cb, add, skip)
    if (k == 0 && last) SEM_SUM(0, true);
    else if (k == 0) SEM_SUM(0, false);
    else if (k == 1 && last) SEM_SUM(1, true);
    else if (k == 1) SEM_SUM(1, false);
    else if (last) SEM_SUM(2, true);
    else SEM_SUM(2, false);
#undef SEM_SUM
  };
  SEM_HIP(launch_fdm<T>(L.sch, m->E, r, box, skip, s));
  sum(0, 4.0 / (3.0 * lmax), 0.0);
  for (int k = 1; k < P.smooth_order; ++k) {
    if ((st = level_residual<T>(P, L, op, d, r, rk, k == 1, skip, s))) return st;
    if (applies) ++*applies;
    SEM_HIP(launch_fdm<T>(L.sch, m->E, rk, box, skip, s));
    sum(k, (2.0 * k - 1.0) / (2.0 * k + 3.0), (8.0 * k + 4.0) / ((2.0 * k + 3.0) * lmax));
  }
  SEM_CHECK_LAUNCH("Chebyshev-Schwarz");
  return SEM_OK;
}

// z = the smoothing of r, or z += it (scratch: a free vector for that)
template <typename T>
sem_status smooth(Pmg& P, PmgLevel& L, const T* r, T* z, T* scratch, bool add,
                  const CgScalars* outer, hipStream_t s, int* applies) {
  if (P.smoother == 1) return cheb_schwarz<T>(P, L, r, z, add, outer, s, applies);
  ChebCg c;
  c.skip_sc = outer;
  sem_status st = cheb_apply_dev<T, T>(L.m, *L.m->work, op_of<T>(L), dinv_of<T>(L), r,
                                       add ? scratch : z, P.smooth_order, L.rho_hat, c, s, applies);
  if (st || !add) return st;
  hipLaunchKernelGGL((k_vadd<T>), dim3(grid_for(L.m->n_free)), dim3(kVecBlock), 0, s,
                     L.m->n_free, z, scratch, outer ? &outer->done : nullptr);
  SEM_CHECK_LAUNCH("post-smoothing");
  return SEM_OK;
}

// The single-wavefront transfers between a level of nf^3 points per element and
// one of nc^3; false for pairs of sizes that the default hierarchies do not
// have (k_transfer is compiled for theirs).
template <typename T, bool PROLONG>
bool launch_transfer(int64_t E, int nf, int nc, const T* M, const T* in, const int32_t* map_in,
                     const int32_t* omap, T* out, const int32_t* skip, hipStream_t s) {
#define SEM_PAIR(F, C)                                                                          \
  case 16 * F + C:                                                                              \
    hipLaunchKernelGGL((k_transfer<T, (PROLONG ? C : F), (PROLONG ? F : C), PROLONG>),          \
                       dim3((unsigned)E), dim3(64), 0, s, M, in, map_in, omap, out, skip);      \
    return true
  switch (16 * nf + nc) {
    SEM_PAIR(11, 6);
    SEM_PAIR(10, 5);
    SEM_PAIR(9, 5);
    SEM_PAIR(8, 4);
    SEM_PAIR(7, 4);
    SEM_PAIR(6, 3);
    SEM_PAIR(5, 3);
    SEM_PAIR(4, 2);
    SEM_PAIR(3, 2);
    default: return false;
  }
#undef SEM_PAIR
}

template <typename T>
sem_status vcycle(Pmg& P, int l, const T* r, T* x, const CgScalars* outer, hipStream_t s,
                  int* applies) {
  PmgLevel& L = P.lv[l];
  const sem_mesh* m = L.m;
  SolveWork& W = *m->work;
  const int64_t nf = m->n_free;
  const int32_t* skip = outer ? &outer->done : nullptr;
  const Op<T>& op = op_of<T>(L);
  const T* dinv = dinv_of<T>(L);
  T* t = P.vec<T>(L, 2);
  T* u = P.vec<T>(L, 3);
  T* wL = local_scratch<T>(m);
  if (!t || !u || !wL) return fail(SEM_ENOMEM, "multigrid work space");
  const bool last = (l + 1 == (int)P.lv.size());
  if (last && coarse_fits(L.coarse, sizeof(T) == 8))
    return coarse_cg<T>(L.coarse, m, dinv, r, x, P.coarse_iters, m->nullspace && op.h2 == T(0),
                        outer, s);
  if (last) {
    T* w = P.vec<T>(L, 4);
    if (!w) return fail(SEM_ENOMEM, "multigrid work space");
    return cg_fixed_device<T>(m, W, op, dinv, r, x, t, u, w, wL, P.coarse_iters,
                              m->nullspace && op.h2 == T(0), outer, s);
  }
  Op<T> ops = op;
  ops.skip = skip;
  sem_status st;
  // pre-smoothing
  if ((st = smooth<T>(P, L, r, x, u, false, outer, s, applies))) return st;
  // t = r - A x, restricted to the next level
  if ((st = level_residual<T>(P, L, ops, x, r, t, true, skip, s))) return st;
  if (applies) ++*applies;
  PmgLevel& C = P.lv[l + 1];
  const sem_mesh* mc = C.m;
  T* cL = local_scratch<T>(mc);
  T* rc = P.vec<T>(C, 0);
  T* xc = P.vec<T>(C, 1);
  if (!cL || !rc || !xc) return fail(SEM_ENOMEM, "multigrid work space");
  const int32_t* omap = L.omap.as<int32_t>();
  if (!L.conforming || !launch_transfer<T, false>(m->E, m->n1, mc->n1, mat<T>(L.JT64, L.JT32), t,
                                                  nullptr, omap, cL, skip, s))
    SEM_HIP(launch_interp<T>(m->E, m->n1, mc->n1, mat<T>(L.JT64, L.JT32), 2, t,
                             m->lmap.as<int32_t>(), m->fseg.as<int32_t>(), cL, skip, s));
  hipLaunchKernelGGL((k_seg_sum<T>), dim3(grid_for(mc->n_free)), dim3(kVecBlock), 0, s,
                     mc->n_free, mc->fseg.as<int32_t>(), mc->fperm.as<int32_t>(), cL, rc, skip);
  SEM_CHECK_LAUNCH("restriction");
  if ((st = vcycle<T>(P, l + 1, rc, xc, outer, s, nullptr))) return st;
  // x += P x_c
  if (!L.conforming || !launch_transfer<T, true>(m->E, m->n1, mc->n1, mat<T>(L.J64, L.J32), xc,
                                                 mc->lmap.as<int32_t>(), omap, x, skip, s)) {
    SEM_HIP(launch_interp<T>(m->E, mc->n1, m->n1, mat<T>(L.J64, L.J32), 1, xc,
                             mc->lmap.as<int32_t>(), nullptr, wL, skip, s));
    hipLaunchKernelGGL((k_seg_add_avg<T>), dim3(grid_for(nf)), dim3(kVecBlock), 0, s, nf,
                       m->fseg.as<int32_t>(), m->fperm.as<int32_t>(), wL, x, skip);
  }
  SEM_CHECK_LAUNCH("prolongation");
  // post-smoothing on t = r - A x
  if ((st = level_residual<T>(P, L, ops, x, r, t, true, skip, s))) return st;
  if (applies) ++*applies;
  if ((st = smooth<T>(P, L, t, x, u, true, outer, s, applies))) return st;
  return SEM_OK;
}

}  // namespace

template <typename T>
T* Pmg::vec(PmgLevel& L, int which) {
  DevBuf* b64[8] = {&L.r64, &L.x64, &L.t64, &L.u64, &L.w64, &L.d64, &L.k64v, &L.q64};
  DevBuf* b32[8] = {&L.r32, &L.x32, &L.t32, &L.u32, &L.w32, &L.d32, &L.k32v, &L.q32};
  DevBuf& b = sizeof(T) == 8 ? *b64[which] : *b32[which];
  if (b.ensure((size_t)std::max<int64_t>(L.m->n_free, 1) * sizeof(T)) != SEM_OK) return nullptr;
  return b.as<T>();
}
template double* Pmg::vec<double>(PmgLevel&, int);
template float* Pmg::vec<float>(PmgLevel&, int);

sem_status setup_transfers(Pmg& P, hipStream_t s) {
  const int nt = (int)P.lv.size() - 1;
  if (nt < 1) return SEM_OK;
  // scratch of all levels at once: a count per level, coarse values, copies
  int64_t n_xc = 1, n_v = 1;
  for (int l = 0; l < nt; ++l) {
    n_xc = std::max(n_xc, P.lv[l + 1].m->n_free);
    n_v = std::max(n_v, P.lv[l].m->nL);
  }
  DevBuf tmp;
  sem_status st = tmp.ensure((size_t)(nt + n_xc + n_v) * sizeof(double));
  if (st) return st;
  int* const count = tmp.as<int>();
  double* const x = tmp.as<double>() + nt;
  double* const v = x + n_xc;
  SEM_HIP(launch_fill<int>(count, nt, 0, s));
  for (int l = 0; l < nt; ++l) {
    PmgLevel& L = P.lv[l];
    const sem_mesh* m = L.m;
    const sem_mesh* mc = P.lv[l + 1].m;
    if ((st = L.omap.ensure((size_t)std::max<int64_t>(m->nL, 1) * sizeof(int32_t)))) return st;
    const int32_t* lmap = m->lmap.as<int32_t>();
    const int32_t* seg = m->fseg.as<int32_t>();
    const int32_t* perm = m->fperm.as<int32_t>();
    const dim3 g(grid_for(m->nL)), b(kVecBlock);
    hipLaunchKernelGGL(k_first_copies, g, b, 0, s, m->nL, lmap, seg, perm, L.omap.as<int32_t>());
    hipLaunchKernelGGL(k_scatter_values, dim3(grid_for(mc->n_free)), b, 0, s, mc->n_free, x);
    SEM_HIP(launch_interp<double>(m->E, mc->n1, m->n1, L.J64.as<double>(), 1, x,
                                  mc->lmap.as<int32_t>(), nullptr, v, nullptr, s));
    hipLaunchKernelGGL(k_copies_differ, g, b, 0, s, m->nL, lmap, seg, perm, v, count + l);
    SEM_CHECK_LAUNCH("transfer set-up");
  }
  std::vector<int> n(nt);
  SEM_HIP(hipMemcpyAsync(n.data(), count, nt * sizeof(int), hipMemcpyDeviceToHost, s));
  SEM_HIP(hipStreamSynchronize(s));
  for (int l = 0; l < nt; ++l) {
    P.lv[l].conforming = n[l] == 0;
    if (n[l]) P.lv[l].omap.release();
  }
  return SEM_OK;
}

void pmg_destroy(Pmg* p) {
  if (!p) return;
  for (auto& L : p->lv)
    if (L.owned && L.m) sem_free_mesh(L.m);
  delete p;
}

template <typename T>
hipError_t launch_interp(int64_t E, int n_in, int n_out, const T* M, int mode, const T* in,
                         const int32_t* lmap, const int32_t* seg, T* out_L, const int32_t* skip,
                         hipStream_t s) {
  if (n_in < 1 || n_in > kN1 || n_out < 1 || n_out > kN1 || E < 1) return hipErrorInvalidValue;
  const dim3 g((unsigned)E), b(kInterpThreads);
  if (mode == 0)
    hipLaunchKernelGGL((interp_kernel<T, 0>), g, b, 0, s, n_in, n_out, M, in, lmap, seg, out_L,
                       skip);
  else if (mode == 1)
    hipLaunchKernelGGL((interp_kernel<T, 1>), g, b, 0, s, n_in, n_out, M, in, lmap, seg, out_L,
                       skip);
  else
    hipLaunchKernelGGL((interp_kernel<T, 2>), g, b, 0, s, n_in, n_out, M, in, lmap, seg, out_L,
                       skip);
  return hipGetLastError();
}
template hipError_t launch_interp<double>(int64_t, int, int, const double*, int, const double*,
                                          const int32_t*, const int32_t*, double*,
                                          const int32_t*, hipStream_t);
template hipError_t launch_interp<float>(int64_t, int, int, const float*, int, const float*,
                                         const int32_t*, const int32_t*, float*, const int32_t*,
                                         hipStream_t);

template <typename Tr, typename Tp>
sem_status pmg_precond(const sem_mesh* m, SolveWork& W, const Tr* r, Tr* z, const ChebCg& cg,
                       hipStream_t s, int* applies) {
  (void)W;
  if (!m->pmg || m->pmg->lv.empty() || m->pmg->lv[0].m != m)
    return fail(SEM_EINVAL, "no multigrid hierarchy for this mesh");
  Pmg& P = *m->pmg;
  PmgLevel& L0 = P.lv[0];
  const int64_t nf = m->n_free;
  sem_status st;
  if (cg.sc && (st = launch_cg_gate(cg.check_in, cg.nblk, cg.sc, cg.hist, s))) return st;
  const Tp* r0;
  if constexpr (std::is_same<Tr, Tp>::value) {
    r0 = r;
  } else {
    Tp* rr = P.vec<Tp>(L0, 0);
    if (!rr) return fail(SEM_ENOMEM, "multigrid work space");
    if ((st = launch_convert_skip<Tr, Tp>(nf, r, rr, cg.sc, s))) return st;
    r0 = rr;
  }
  Tp* x0 = P.vec<Tp>(L0, 1);
  if (!x0) return fail(SEM_ENOMEM, "multigrid work space");
  if ((st = vcycle<Tp>(P, 0, r0, x0, cg.sc, s, applies))) return st;
  return launch_flex_dots<Tr, Tp>(nf, x0, z, r, static_cast<const Tr*>(cg.w), cg.part_out, cg.sc,
                                  s);
}
template sem_status pmg_precond<double, double>(const sem_mesh*, SolveWork&, const double*,
                                                double*, const ChebCg&, hipStream_t, int*);
template sem_status pmg_precond<double, float>(const sem_mesh*, SolveWork&, const double*,
                                               double*, const ChebCg&, hipStream_t, int*);
template sem_status pmg_precond<float, float>(const sem_mesh*, SolveWork&, const float*, float*,
                                              const ChebCg&, hipStream_t, int*);

sem_status schwarz_precond(Pmg& P, int level, const double* r, double* z, const ChebCg& cg,
                           hipStream_t s) {
  PmgLevel& L = P.lv[level];
  const int64_t nf = L.m->n_free;
  sem_status st;
  if (cg.sc && (st = launch_cg_gate(cg.check_in, cg.nblk, cg.sc, cg.hist, s))) return st;
  double* q = P.vec<double>(L, 7);
  if (!q) return fail(SEM_ENOMEM, "multigrid work space");
  if ((st = schwarz_apply<double>(L, r, q, cg.sc ? &cg.sc->done : nullptr, s))) return st;
  return launch_flex_dots<double, double>(nf, q, z, r, static_cast<const double*>(cg.w),
                                          cg.part_out, cg.sc, s);
}

}  // namespace sem
