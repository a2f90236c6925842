// Jacobi-PCG of a small mesh as one resident kernel, N >= 5.
//
// A mesh of a few hundred elements at most is bound by launches: an iteration
// of four kernels costs 15-21 us whatever the size, of which the data (all in
// cache) account for about two.  Here a workgroup keeps one element over the
// iterations: x, r, p, S and the metric of its points in registers, the
// contractions in LDS.  Copies of a shared node are kept by every element that
// has one and advance with identical operands, so they stay identical.  An
// iteration is
//   A p on the element, shared copies' results to memory | p.w, sum(w)
//   r -= alpha (w - mean), w summed over the copies in a fixed order | r.r, r.z
//   x += alpha p, p = z + beta p
// with one exchange between the workgroups (gridsync.hpp) at each bar.  The
// copies' values carry the exchange's tag themselves, so they are waited for
// beside the partial sums and not after them, and are shared out evenly over
// the element's lanes (784 values, 64 of them at eight corners, on an element
// of order 7).  Bound by the two exchanges, about 2.5 us each; the operator
// takes 0.8 us.  Iteration, launches -> resident, us:
//   64 elements, N = 5 15.3 -> 6.2, 6 16.1 -> 6.8, 7 15.9 -> 6.9, 8 19.6 -> 8.5,
//   9 20.9 -> 8.4, 10 19.6 -> 9.0; 192 elements, N = 7 16.2 -> 7.4
// and a solve starts without the 250-350 us of a graph's capture: 4x4x4 cube,
// N = 7, to 1e-10 4500 -> 1821 us (values read after the first exchange: 1905).
#include <algorithm>

#include "ax_tiles.hpp"
#include "gridsync.hpp"
#include "resident.hpp"

namespace sem {
namespace {

// Wavefronts per element: one to three points per lane.
template <int N, typename T>
struct RShape : LShape<N, T> {
  using S = LShape<N, T>;
  static constexpr int NW = N <= 8 ? 4 : 8;
  static constexpr int TPB = 64 * NW;
  static constexpr int PPT = (S::P + TPB - 1) / TPB;
  static constexpr int TPW = (S::NT + NW - 1) / NW;
};

constexpr int kBatch = 4;  // values a lane waits for together (an element of order 7: 784 by 256)

__device__ __forceinline__ bool finite(double x) {
  return x == x && fabs(x) <= 1.7976931348623157e308;
}

template <typename T>
struct Dev {
  const T* G;
  const T* B;
  const T* k;
  const T* D;
  T h2;
  T *x, *z, *p;
  const T* dinv;
  const int32_t* lmap2;
  const int32_t* fseg;
  const int32_t* fperm2;
  uint64_t* slots;
  uint64_t* shared;  // [E][P] tagged values: shared copies' results at their surface slots
  uint32_t* epoch;
  CgScalars* sc;
  double *hist, *ahist, *bhist;
  int profile;
};

template <int N, typename T>
__global__ __launch_bounds__((RShape<N, T>::TPB))
    __attribute__((amdgpu_waves_per_eu(2))) void k_resident_cg(const Dev<T> A, int iters) {
  using S = RShape<N, T>;
  constexpr int n1 = S::n1, P = S::P, PPT = S::PPT, TPB = S::TPB, NW = S::NW, NT = S::NT,
                TPW = S::TPW, SZ = n1 * S::PS, CAP = 3 * SZ;
  constexpr bool BLK = sizeof(T) == 8;
  constexpr int KW = kTagWords<T>;
  CgScalars* sc = A.sc;
  if (sc->done) return;  // uniform over the grid
  __shared__ T su[SZ];
  __shared__ T sa[3][SZ];
  __shared__ double red[2 * NW];
  __shared__ int32_t list[CAP];
  __shared__ int nused;
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nblk = gridDim.x;
  const int64_t e = blockIdx.x, eP = e * P;
  const bool first_block = blockIdx.x == 0 && t == 0;
  const uint32_t first = __hip_atomic_load(A.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t tag = first;
  const int it0 = sc->it, max_it = sc->max_it, fixed = sc->fixed, neumann = sc->neumann;
  const double tol2 = sc->tol2, inv_n = sc->inv_n;
  double rho = sc->rho2[it0 & 1], rr = sc->rr, ticks = sc->op_ticks;

  auto point = [&](int s) -> int {
    return (s + 1) * TPB <= P ? t + s * TPB : min(t + s * TPB, P - 1);
  };
  auto in_element = [&](int s) { return (s + 1) * TPB <= P || t + s * TPB < P; };

  // the element's points: metric (times k), h2 B, and the solve's vectors;
  // slot[s]: where a shared copy's result goes, seg[s], cnt[s]: its node's
  // copies (cnt 0: no shared free copy)
  T g[PPT][6], hb[PPT], x[PPT], r[PPT], p[PPT], d[PPT];
  int32_t node[PPT], slot[PPT], seg[PPT], cnt[PPT];
#pragma unroll
  for (int s = 0; s < PPT; ++s) {
    const int q = point(s);
    const int32_t cd = in_element(s) ? A.lmap2[eP + q] : -1;
    node[s] = cd >= 0 ? cd : cd <= -2 ? -(cd + 2) : -1;
    const T kq = A.k ? A.k[eP + q] : T(1);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      g[s][c] = A.G[e * 6 * P + c * P + q];
      if (A.k) g[s][c] *= kq;
    }
    hb[s] = A.h2 != T(0) ? A.h2 * A.B[eP + q] : T(0);
    slot[s] = (int32_t)eP + surface_rank(q % n1, (q / n1) % n1, q / (n1 * n1), N);
    seg[s] = cnt[s] = 0;
    if (cd <= -2) {
      seg[s] = A.fseg[node[s]];
      cnt[s] = A.fseg[node[s] + 1] - seg[s];
    }
    const int32_t at = max(node[s], 0);
    const bool act = node[s] >= 0;
    x[s] = act ? A.x[at] : T(0);
    p[s] = act ? A.p[at] : T(0);
    d[s] = act ? A.dinv[at] : T(0);
    r[s] = act ? A.z[at] / d[s] : T(0);
  }
  // a node's sums are formed, and its vectors written, by its first copy
  bool owner[PPT];
#pragma unroll
  for (int s = 0; s < PPT; ++s)
    owner[s] = node[s] >= 0 && (cnt[s] == 0 || A.fperm2[seg[s]] == slot[s]);
  // the element's list of copies to gather; seg[s] becomes the node's place in
  // it, or ~seg[s] where the list is full
  for (int j = t; j < CAP; j += TPB) list[j] = -1;
  if (t == 0) nused = 0;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < PPT; ++s)
    if (cnt[s]) {
      const int at = atomicAdd(&nused, cnt[s]);
      if (at + cnt[s] <= CAP) {
        for (int c = 0; c < cnt[s]; ++c) list[at + c] = A.fperm2[seg[s] + c];
        seg[s] = at;
      } else {
        seg[s] = ~seg[s];
      }
    }
  __syncthreads();
  const int nlist = min(nused, CAP);
  const DFrag<N, T, BLK> af(A.D, lane, false), at(A.D, lane, true);

  const int last = min(it0 + iters, max_it);
  int it = it0, status = 0;
  bool ok = true, done = false;
  while (!done && it < last) {
    const uint64_t c0 = A.profile ? wall_clock64() : 0;
#pragma unroll
    for (int s = 0; s < PPT; ++s)
      if (in_element(s)) su[lds_point<N, T>(point(s))] = p[s];
    __syncthreads();
#pragma unroll
    for (int y = 0; y < TPW; ++y) {
      const int tile = wv + y * NW;
      if ((y + 1) * NW <= NT || tile < NT)
        contract_tile<N, T, BLK>(tile, lane, af, su, su, su, sa[0], sa[1], sa[2]);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
      const int q = lds_point<N, T>(point(s));
      const T ur = sa[0][q], us = sa[1][q], ut = sa[2][q];
      const T* gc = g[s];
      const T vr = gc[0] * ur + gc[1] * us + gc[2] * ut;
      const T vs = gc[1] * ur + gc[3] * us + gc[4] * ut;
      const T vt = gc[2] * ur + gc[4] * us + gc[5] * ut;
      if (in_element(s)) {
        sa[0][q] = vr;
        sa[1][q] = vs;
        sa[2][q] = vt;
      }
    }
    __syncthreads();
#pragma unroll
    for (int y = 0; y < TPW; ++y) {
      const int tile = wv + y * NW;
      if ((y + 1) * NW <= NT || tile < NT)
        contract_tile<N, T, BLK>(tile, lane, at, sa[0], sa[1], sa[2], sa[0], sa[1], sa[2]);
    }
    __syncthreads();
    T w[PPT];
    double pw = 0.0, sw = 0.0;
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
      const int q = lds_point<N, T>(point(s));
      w[s] = (sa[0][q] + sa[1][q]) + sa[2][q] + hb[s] * p[s];
      if (node[s] >= 0) {
        pw += (double)p[s] * (double)w[s];
        sw += (double)w[s];
        if (cnt[s]) put_tagged<T>(A.shared + (int64_t)slot[s] * KW, w[s], tag + 1);
      }
    }
    if (A.profile) ticks += (double)(wall_clock64() - c0);
    grid_put2<NW>(pw, sw, ++tag, nblk, A.slots, red);
    // all copies of the element's shared nodes, evenly over the lanes, to LDS
    T* const val = sa[0];
    int lost = 0;
    for (int j0 = t; j0 < nlist; j0 += kBatch * TPB) {
      Tagged<T> v[kBatch];
      int32_t from[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        from[i] = list[min(j0 + i * TPB, nlist - 1)];
        if (from[i] >= 0) v[i].load(A.shared + (int64_t)from[i] * KW);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
        if (from[i] >= 0)
          val[min(j0 + i * TPB, nlist - 1)] =
              v[i].get(A.shared + (int64_t)from[i] * KW, tag, lost);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < PPT; ++s)
      if (cnt[s]) {
        T sum = T(0);
        if (seg[s] >= 0) {
          for (int c = 0; c < cnt[s]; ++c) sum += val[seg[s] + c];
        } else {
          for (int c = 0; c < cnt[s]; ++c) {
            const uint64_t* from = A.shared + (int64_t)A.fperm2[~seg[s] + c] * KW;
            Tagged<T> o;
            o.load(from);
            sum += o.get(from, tag, lost);
          }
        }
        w[s] = sum;
      }
    if (!(ok = grid_get2<NW>(pw, sw, tag, nblk, A.slots, red, lost))) break;
    if (!(pw > 0.0) || !finite(pw)) {
      status = 2;
      done = true;
      break;
    }
    const double alpha = rho / pw;
    const T a = (T)alpha, mw = neumann ? (T)(sw * inv_n) : T(0);
    double r2 = 0.0, rz = 0.0;
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
      r[s] -= a * (w[s] - mw);
      if (node[s] < 0) r[s] = T(0);
      if (owner[s]) {
        r2 += (double)r[s] * (double)r[s];
        rz += (double)r[s] * (double)(d[s] * r[s]);
      }
    }
    if (!(ok = grid_sum2<NW>(r2, rz, ++tag, nblk, A.slots, red))) break;
    rr = r2;
#pragma unroll
    for (int s = 0; s < PPT; ++s) x[s] += a * p[s];
    if (first_block) {
      A.ahist[it] = alpha;
      A.hist[it + 1] = sqrt(rr);
    }
    ++it;
    if (!finite(rr)) {
      status = 3;
      done = true;
    } else if (!fixed && rr <= tol2) {
      status = 1;
      done = true;
    } else if (it >= max_it) {
      done = true;
    }
    if (done) break;
    const double beta = rz / rho;
    if (first_block) A.bhist[it - 1] = beta;
    rho = rz;
    const T b = (T)beta;
#pragma unroll
    for (int s = 0; s < PPT; ++s) p[s] = d[s] * r[s] + b * p[s];
  }
#pragma unroll
  for (int s = 0; s < PPT; ++s)
    if (owner[s]) {
      A.x[node[s]] = x[s];
      A.p[node[s]] = p[s];
      A.z[node[s]] = d[s] * r[s];
    }
  if (!ok && t == 0) {
    sc->gave_up = 1;
    sc->done = 1;
  }
  if (first_block) {  // every workgroup has read them: an exchange of all lies behind
    sc->it = it;
    sc->rr = rr;
    sc->rho2[it & 1] = rho;
    sc->status = status;
    sc->op_ticks = ticks;
    if (done) sc->done = 1;
    __hip_atomic_store(A.epoch, first + 2u * (uint32_t)iters, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <int N, typename T>
hipError_t launch(const Dev<T>& A, int64_t E, int iters, hipStream_t s) {
  hipLaunchKernelGGL((k_resident_cg<N, T>), dim3((unsigned)E), dim3(RShape<N, T>::TPB), 0, s, A,
                     iters);
  return hipGetLastError();
}

// All workgroups have to be resident together, beside those of other streams:
// at most a quarter of the workgroups that the chip holds (in FP64 192
// elements up to N = 7, 128 at N = 8, 64 above; up to 256 in FP32).
// Within that the resident form is the faster one at every size.
template <int N, typename T>
bool fits(const sem_mesh* m) {
  static const int per_cu = [] {
    int n = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_resident_cg<N, T>,
                                                        RShape<N, T>::TPB, 0) == hipSuccess ? n : 0;
  }();
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, m->device) != hipSuccess)
    return false;
  return m->E <= (int64_t)per_cu * cus / 4;
}

}  // namespace

template <typename T>
bool resident_fits(const sem_mesh* m) {
  if (!ax_split_available(m) || m->nL > INT32_MAX) return false;
  switch (m->N) {
    case 5: return fits<5, T>(m);
    case 6: return fits<6, T>(m);
    case 7: return fits<7, T>(m);
    case 8: return fits<8, T>(m);
    case 9: return fits<9, T>(m);
    case 10: return fits<10, T>(m);
  }
  return false;
}
template bool resident_fits<double>(const sem_mesh*);
template bool resident_fits<float>(const sem_mesh*);

static int64_t sync_words(const sem_mesh* m) { return 2 * m->E * kGridWords; }

// tag (one word) | slots | tagged values
sem_status resident_begin(const sem_mesh* m, SolveWork& W, hipStream_t s) {
  const int64_t words = 1 + sync_words(m) + 2 * m->nL;
  sem_status st = W.rsync.ensure((size_t)words * sizeof(uint64_t));
  if (st) return st;
  SEM_HIP(launch_fill<double>(W.rsync.as<double>(), words, 0.0, s));
  return SEM_OK;
}

template <typename T>
sem_status resident_run(const sem_mesh* m, SolveWork& W, const ResidentArgs<T>& a, int iters,
                        hipStream_t s) {
  Dev<T> A;
  A.G = a.op.G;
  A.B = a.op.B;
  A.k = a.op.k;
  A.D = a.op.D;
  A.h2 = a.op.h2;
  A.x = a.x;
  A.z = a.z;
  A.p = a.p;
  A.dinv = a.dinv;
  A.lmap2 = m->lmap2.as<int32_t>();
  A.fseg = m->fseg.as<int32_t>();
  A.fperm2 = m->fperm2.as<int32_t>();
  A.epoch = W.rsync.as<uint32_t>();
  A.slots = W.rsync.as<uint64_t>() + 1;
  A.shared = A.slots + sync_words(m);
  A.sc = W.sc.as<CgScalars>();
  A.hist = W.hist.as<double>();
  A.ahist = W.ahist.as<double>();
  A.bhist = W.bhist.as<double>();
  A.profile = a.profile ? 1 : 0;
  hipError_t e = hipErrorInvalidValue;
  switch (m->N) {
    case 5: e = launch<5, T>(A, m->E, iters, s); break;
    case 6: e = launch<6, T>(A, m->E, iters, s); break;
    case 7: e = launch<7, T>(A, m->E, iters, s); break;
    case 8: e = launch<8, T>(A, m->E, iters, s); break;
    case 9: e = launch<9, T>(A, m->E, iters, s); break;
    case 10: e = launch<10, T>(A, m->E, iters, s); break;
  }
  if (e != hipSuccess) return hip_fail(e, "resident CG");
  return SEM_OK;
}
template sem_status resident_run<double>(const sem_mesh*, SolveWork&, const ResidentArgs<double>&,
                                         int, hipStream_t);
template sem_status resident_run<float>(const sem_mesh*, SolveWork&, const ResidentArgs<float>&,
                                        int, hipStream_t);

}  // namespace sem
