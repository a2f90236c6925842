// The coarsest multigrid level of order 1 as one resident kernel.
//
// Its Jacobi-PCG runs a fixed number of iterations on a few thousand to a few
// ten thousand unknowns.  As four launches per iteration (operator, segmented
// sum, two vector updates of 3.4-5.7 us each) it was bound by launches: 505 us
// per V-cycle on the 32x32x16 box (15,360 unknowns, 30 iterations), 17 % of
// the cycle.  Here the level's matrix is assembled once per (k, h2) -- at
// most 27 columns per row on a hexahedral mesh whose vertices join at most
// eight elements -- and a thread keeps one row, its 27 columns' direction
// values and its entries of x, r, p in registers over all iterations.  Each
// iteration is two exchanges between the workgroups (p.Ap; r.z together with
// z at the neighbours), about 2.5 us each at 60 workgroups (see gridsync.hpp):
// 160 us per V-cycle on that box, the p-multigrid solve to 1e-12 there 52.7
// -> 47.9 ms with it alone.  (Reading z after the exchange, all 27 columns by
// every row, took 214 us; 140 unknowns in one workgroup took 96 us that way, 45
// with z in LDS.)
#include <algorithm>
#include <vector>

#include "gridsync.hpp"
#include "pmg.hpp"

namespace sem {
namespace {

constexpr int kCW = kCoarseWidth;
constexpr int kCT = 256;      // threads (= rows) per workgroup
constexpr int kCN = kCT / 64;  // wavefronts

#define GRID_STRIDE(idx, n)                                                        \
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < (n); \
       idx += (int64_t)gridDim.x * blockDim.x)

// u = 1 at local point b of every element, 0 elsewhere (8 points per element)
__global__ void k_unit_points(int64_t nL, int b, double* __restrict__ u) {
  GRID_STRIDE(q, nL) u[q] = (q & 7) == b ? 1.0 : 0.0;
}

// entry j of row g: the sum of its element-matrix contributions
__global__ void k_assemble_rows(int64_t nf, const int32_t* __restrict__ cseg,
                                const int32_t* __restrict__ cperm, const double* __restrict__ w,
                                double* __restrict__ v64, float* __restrict__ v32) {
  GRID_STRIDE(i, nf * kCW) {
    const int64_t g = i / kCW, j = i - g * kCW;
    const double s = segment_sum<double>(cperm, w, cseg[i], cseg[i + 1]);
    v64[j * nf + g] = s;
    v32[j * nf + g] = (float)s;
  }
}

__device__ __forceinline__ bool finite(double x) {
  return x == x && fabs(x) <= 1.7976931348623157e308;
}

// `iters` Jacobi-PCG iterations from x = 0 for b (minus its mean when
// `neumann`), the recurrences of cg_fixed_device: p = z + beta p is formed by
// the owner of a row and, with the same operands, by every row that has it as
// a column.  A workgroup's columns (its list, each once) come to LDS as tagged
// values, waited for beside the partial sums; a single workgroup has them there
// already.  A breakdown ends the iterations with the last x, a wait that gave up
// (gridsync.hpp) writes NaN.
template <typename T>
__global__ __launch_bounds__(kCT)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3))) void k_coarse_cg(
    int nf, const T* __restrict__ val, const int32_t* __restrict__ col,
    const int32_t* __restrict__ list, const int32_t* __restrict__ nlist,
    const T* __restrict__ dinv, const T* __restrict__ b, T* __restrict__ x,
    uint64_t* __restrict__ zx, int iters, int neumann, double inv_n,
    uint64_t* __restrict__ slots, uint32_t* __restrict__ epoch,
    const CgScalars* __restrict__ outer) {
  if (outer && outer->done) return;  // uniform over the grid
  constexpr int KW = kTagWords<T>;
  constexpr int kBatch = 4;  // values a lane waits for together
  __shared__ double red[2 * kCN];
  __shared__ T zl[kCT * kCW];
  const int nblk = gridDim.x;
  const int g = blockIdx.x * kCT + threadIdx.x;
  const bool act = g < nf;
  const uint32_t first = __hip_atomic_load(epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t tag = first;
  const int32_t* const mine = list + (int64_t)blockIdx.x * (kCT * kCW);
  const int nl = nlist[blockIdx.x];
  T v[kCW], pn[kCW];
  int32_t c[kCW];  // places of the columns in zl
#pragma unroll
  for (int j = 0; j < kCW; ++j) {
    v[j] = act ? val[(int64_t)j * nf + g] : T(0);
    c[j] = act ? col[(int64_t)j * nf + g] : 0;
  }
  const T d = act ? dinv[g] : T(0);
  T rg = act ? b[g] : T(0);
  T xg = T(0);
  // s0, s1 <- their sums over all rows, and the columns' z in zl; false when a
  // wait gave up
  const auto exchange = [&](T z, double& s0, double& s1) -> bool {
    ++tag;
    if (nblk == 1) {
      zl[threadIdx.x] = z;
      group_sum2<kCN>(s0, s1, red);
      return true;
    }
    if (act) put_tagged<T>(zx + (int64_t)g * KW, z, tag);
    grid_put2<kCN>(s0, s1, tag, nblk, slots, red);
    int lost = 0;
    for (int j0 = threadIdx.x; j0 < nl; j0 += kBatch * kCT) {
      Tagged<T> w[kBatch];
      const uint64_t* from[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        from[i] = zx + (int64_t)mine[min(j0 + i * kCT, nl - 1)] * KW;
        w[i].load(from[i]);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) zl[min(j0 + i * kCT, nl - 1)] = w[i].get(from[i], tag, lost);
    }
    return grid_get2<kCN>(s0, s1, tag, nblk, slots, red, lost);
  };
  bool ok = true;
  if (neumann) {
    double s = (double)rg, s1 = 0.0;
    ok = grid_sum2<kCN>(s, s1, ++tag, nblk, slots, red);
    rg -= act ? (T)(s * inv_n) : T(0);
  }
  T pg = d * rg;
  double rho = (double)rg * (double)pg, unused = 0.0;
  if (ok) ok = exchange(pg, rho, unused);
  if (ok && rho > 0.0 && finite(rho)) {
#pragma unroll
    for (int j = 0; j < kCW; ++j) pn[j] = zl[c[j]];
    for (int it = 0; it < iters; ++it) {
      T w = T(0);
#pragma unroll
      for (int j = 0; j < kCW; ++j) w += v[j] * pn[j];
      double pw = (double)pg * (double)w, sw = (double)w;
      if (!(ok = grid_sum2<kCN>(pw, sw, ++tag, nblk, slots, red))) break;
      if (!(pw > 0.0) || !finite(pw)) break;
      const double alpha = rho / pw;
      const T a = (T)alpha, mw = neumann && act ? (T)(sw * inv_n) : T(0);
      xg += a * pg;
      if (it + 1 == iters) break;
      rg -= a * (w - mw);
      const T zg = d * rg;
      double rr = (double)rg * (double)rg, rz = rr * (double)d;
      if (!(ok = exchange(zg, rr, rz))) break;
      if (!finite(rr)) break;
      const T bt = (T)(rz / rho);
      rho = rz;
      pg = zg + bt * pg;
#pragma unroll
      for (int j = 0; j < kCW; ++j) pn[j] = zl[c[j]] + bt * pn[j];
    }
  }
  if (act) x[g] = ok ? xg : (T)__builtin_nan("");
  if (g == 0)  // every workgroup has read it: an exchange of all lies behind
    __hip_atomic_store(epoch, first + 2u * (uint32_t)iters + 2u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

unsigned vblocks(int64_t n) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192));
}

}  // namespace

// Host: the rows' columns and where their entries' contributions lie.  Entry
// (g, j) sums w[b nL + 8 e + a] over the elements e that hold row g as local
// point a and the column as local point b (w[b nL + .] = A_L applied to the
// unit vector of point b).  False when a row has more than kCoarseWidth columns.
static bool coarse_pattern(const HostNumbering& hn, int64_t nL, std::vector<int32_t>& col,
                           std::vector<int32_t>& cseg, std::vector<int32_t>& cperm) {
  const int64_t nf = hn.n_free;
  col.assign((size_t)(nf * kCW), 0);
  cseg.assign((size_t)(nf * kCW + 1), 0);
  cperm.clear();
  struct Ent {
    int32_t col, at;
  };
  std::vector<Ent> ent;
  for (int64_t g = 0; g < nf; ++g) {
    ent.clear();
    for (int32_t a = hn.fseg[g]; a < hn.fseg[g + 1]; ++a) {
      const int64_t q = hn.fperm[a], e8 = q & ~int64_t(7);
      for (int b = 0; b < 8; ++b) {
        const int32_t cc = hn.lmap[e8 + b];
        if (cc >= 0) ent.push_back({cc, (int32_t)(b * nL + q)});
      }
    }
    std::stable_sort(ent.begin(), ent.end(),
                     [](const Ent& a, const Ent& b) { return a.col < b.col; });
    int j = -1;
    for (size_t i = 0; i < ent.size(); ++i) {
      if (i == 0 || ent[i].col != ent[i - 1].col) {
        if (++j >= kCW) return false;
        col[(size_t)(j * nf + g)] = ent[i].col;
        cseg[(size_t)(g * kCW + j)] = (int32_t)cperm.size();
      }
      cperm.push_back(ent[i].at);
    }
    for (++j; j < kCW; ++j) {  // empty entries: value 0, the row itself
      col[(size_t)(j * nf + g)] = (int32_t)g;
      cseg[(size_t)(g * kCW + j)] = (int32_t)cperm.size();
    }
  }
  cseg[(size_t)(nf * kCW)] = (int32_t)cperm.size();
  return true;
}

static sem_status put(DevBuf& d, const std::vector<int32_t>& h, hipStream_t s) {
  sem_status st = d.ensure(std::max<size_t>(h.size(), 1) * sizeof(int32_t));
  if (st) return st;
  SEM_HIP(hipMemcpyAsync(d.p, h.data(), h.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
  return SEM_OK;
}

sem_status setup_coarse(CoarseDev& C, const sem_mesh* m, const int64_t* gid,
                        const uint8_t* dirichlet, hipStream_t s) {
  C.on = false;
  const int64_t nf = m->n_free, nL = m->nL;
  if (m->N != 1 || nf < 1 || nf > (int64_t)3 * kCoarseCus / 4 * kCT || nL > INT32_MAX / 8) return SEM_OK;
  HostNumbering hn;
  sem_status st = build_numbering(1, m->E, gid, dirichlet, hn);
  if (st) return st;
  std::vector<int32_t> col, cseg, cperm;
  if (!coarse_pattern(hn, nL, col, cseg, cperm)) return SEM_OK;
  const size_t nv = (size_t)(nf * kCW);
  C.nblk = (int)((nf + kCT - 1) / kCT);
  // 32-bit words: the tag (two), the slots, up to two 64-bit words of z per row
  C.n_sync = 2 + 2 * ((int64_t)2 * C.nblk * kGridWords + 2 * nf);
  // every workgroup's columns, each once, and the places of its rows' columns
  // in that list; one workgroup has the rows themselves
  std::vector<int32_t> list((size_t)C.nblk * kCT * kCW), nlist(C.nblk), place(col.size());
  std::vector<int32_t> at(nf), in(nf, -1);
  for (int w = 0; w < C.nblk; ++w) {
    int n = 0;
    const int64_t hi = std::min<int64_t>(nf, (int64_t)(w + 1) * kCT);
    for (int64_t g = (int64_t)w * kCT; g < hi; ++g)
      for (int j = 0; j < kCW; ++j) {
        const int32_t cc = col[(size_t)(j * nf + g)];
        if (in[cc] != w) {
          in[cc] = w;
          list[(size_t)w * kCT * kCW + n] = cc;
          at[cc] = C.nblk == 1 ? cc : n;
          ++n;
        }
        place[(size_t)(j * nf + g)] = at[cc];
      }
    nlist[w] = n;
  }
  if ((st = put(C.place, place, s)) || (st = put(C.list, list, s)) ||
      (st = put(C.nlist, nlist, s)) || (st = put(C.cseg, cseg, s)) || (st = put(C.cperm, cperm, s)) ||
      (st = C.v64.ensure(nv * sizeof(double))) || (st = C.v32.ensure(nv * sizeof(float))) ||
      (st = C.u.ensure((size_t)nL * sizeof(double))) ||
      (st = C.w.ensure((size_t)(8 * nL) * sizeof(double))) ||
      (st = C.sync.ensure((size_t)C.n_sync * sizeof(int32_t))))
    return st;
  SEM_HIP(hipStreamSynchronize(s));  // host vectors go out of scope
  C.on = true;
  C.valid = false;
  return SEM_OK;
}

sem_status prepare_coarse(CoarseDev& C, const sem_mesh* m, const double* k, double h2,
                          hipStream_t s) {
  if (!C.on) return SEM_OK;
  SEM_HIP(launch_fill<int>(C.sync.as<int>(), C.n_sync, 0, s));
  if (!k && C.valid && C.h2 == h2) return SEM_OK;
  const int64_t nL = m->nL;
  double* u = C.u.as<double>();
  double* w = C.w.as<double>();
  for (int b = 0; b < 8; ++b) {
    hipLaunchKernelGGL(k_unit_points, dim3(vblocks(nL)), dim3(256), 0, s, nL, b, u);
    SEM_HIP(launch_ax<double>(m, u, nullptr, w + b * nL, k, h2, m->G64.as<double>(),
                              m->B64.as<double>(), m->D64.as<double>(), s));
  }
  hipLaunchKernelGGL(k_assemble_rows, dim3(vblocks(m->n_free * kCW)), dim3(256), 0, s, m->n_free,
                     C.cseg.as<int32_t>(), C.cperm.as<int32_t>(), w, C.v64.as<double>(),
                     C.v32.as<float>());
  SEM_CHECK_LAUNCH("coarse matrix");
  C.valid = k == nullptr;
  C.h2 = h2;
  return SEM_OK;
}

bool coarse_fits(const CoarseDev& C, bool f64) {
  return C.on && C.nblk <= (f64 ? 2 : 3) * kCoarseCus / 4;
}

template <typename T>
sem_status coarse_cg(CoarseDev& C, const sem_mesh* m, const T* dinv, const T* b, T* x, int iters,
                     bool neumann, const CgScalars* outer, hipStream_t s) {
  const T* val = nullptr;
  if constexpr (sizeof(T) == 8) val = C.v64.as<double>();
  else val = C.v32.as<float>();
  uint64_t* const slots = C.sync.as<uint64_t>() + 1;
  hipLaunchKernelGGL((k_coarse_cg<T>), dim3(C.nblk), dim3(kCT), 0, s, (int)m->n_free, val,
                     C.place.as<int32_t>(), C.list.as<int32_t>(), C.nlist.as<int32_t>(), dinv, b, x, slots + (int64_t)2 * C.nblk * kGridWords,
                     iters, neumann ? 1 : 0, 1.0 / (double)m->n_free, slots,
                     C.sync.as<uint32_t>(), outer);
  SEM_CHECK_LAUNCH("coarse CG");
  return SEM_OK;
}
template sem_status coarse_cg<double>(CoarseDev&, const sem_mesh*, const double*, const double*,
                                      double*, int, bool, const CgScalars*, hipStream_t);
template sem_status coarse_cg<float>(CoarseDev&, const sem_mesh*, const float*, const float*,
                                     float*, int, bool, const CgScalars*, hipStream_t);

}  // namespace sem
