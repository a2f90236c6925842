// p-multigrid hierarchy (internal).
//
// Sec. 2.2 names the default preconditioner of the pressure solve: p-multigrid
// with fourth-kind Chebyshev acceleration of the smoother, most of it in FP32.
// Levels are orders N_0 = N > N_1 > ... > N_L on the same hexahedra; each
// coarse level is a mesh of its own (coordinates interpolated from the fine
// element maps, unknowns identified through the fine global ids), so every
// level runs the same operator, Jacobi and Chebyshev code as the fine one.
#pragma once

#include <vector>

#include "common.hpp"
#include "schwarz.hpp"
#include "solver.hpp"

namespace sem {

// The coarsest level's assembled matrix and exchange buffers (coarse.hip)
constexpr int kCoarseWidth = 27;  // columns of a row: a vertex and its neighbours in 8 hexahedra
constexpr int kCoarseCus = 256;   // compute units; each holds 3 (FP32) or 2 (FP64) workgroups
struct CoarseDev {
  bool on = false;         // the level qualifies (order 1, rows and row lengths within the limits)
  bool valid = false;      // the matrix of (k == NULL, h2) is there
  double h2 = 0.0;
  int nblk = 0;
  int64_t n_sync = 0;      // 32-bit words of `sync`: running tag, exchange slots, tagged z
  DevBuf place, list, nlist, cseg, cperm, v64, v32, u, w, sync;
};

struct PmgLevel {
  sem_mesh* m = nullptr;  // level mesh (level 0: the fine mesh, not owned)
  bool owned = false;
  int N = 0;
  // interpolation from level l+1 to level l, (N_l+1) x (N_{l+1}+1) row-major,
  // and its transpose (restriction), in both precisions
  DevBuf J64, J32, JT64, JT32;
  // every copy of a node of this level interpolates to the same value, and the
  // free node of each first copy (-1 at the others; see k_transfer)
  bool conforming = false;
  DevBuf omap;
  // free vectors of this level: r (input), x (output), t, u, w (scratch),
  // d, rk, q (Chebyshev-Schwarz smoothing)
  DevBuf r64, x64, t64, u64, w64, d64, k64v, q64, r32, x32, t32, u32, w32, d32, k32v, q32;
  CoarseDev coarse;        // coarsest level only
  SchwarzDev sch;          // Schwarz factors (levels that smooth, Schwarz smoother only)
  double sch_rho = 0.0;    // cached bound of the Schwarz-preconditioned operator (k == NULL)
  double sch_rho_h2 = -1.0;
  DevBuf Ik64;  // interpolation from level 0's GLL points to this level's (levels >= 1)
  DevBuf k64;   // k interpolated to this level (levels >= 1, per solve)
  // per solve
  Op<double> op64;
  Op<float> op32;
  const double* dinv64 = nullptr;
  const float* dinv32 = nullptr;
  double rho_hat = 0.0;  // Chebyshev bound of this level
};

struct Pmg {
  std::vector<PmgLevel> lv;
  int smooth_order = 4;
  int coarse_iters = 30;
  int smoother = 1;  // 0 Jacobi, 1 overlapping Schwarz
  template <typename T>
  T* vec(PmgLevel& L, int which);  // 0 r, 1 x, 2 t, 3 u, 4 w, 5 d, 6 rk, 7 q
};

void pmg_destroy(Pmg* p);
// `conforming` and `omap` of every level but the coarsest (meshes and J64 are
// there); blocks
sem_status setup_transfers(Pmg& P, hipStream_t s);

// host: 1-D Lagrange interpolation from the order-n_from GLL nodes to the
// order-n_to GLL nodes, M is (n_to+1) x (n_from+1) row-major
sem_status host_interp_matrix(int n_from, int n_to, double* M);
// host: coordinates, global ids and Dirichlet flags of the order-Nc mesh on
// the hexahedra of an order-N mesh (dir / dir_c may be null together)
sem_status host_coarse_mesh(int N, int64_t E, const int64_t* gid, const uint8_t* dir,
                            const double* xyz, int Nc, int64_t* gid_c, uint8_t* dir_c,
                            double* xyz_c);

// device: out_L = (M x M x M) applied to each element block (M: n_out x n_in,
// element blocks of n_in^3 and n_out^3 points).  mode 0: the input is a
// local vector in_L; mode 1: gathered from the free vector in_f through
// lmap (0 at Dirichlet copies); mode 2: as 1, divided by the number of local
// copies of the free node (taken from seg).
template <typename T>
hipError_t launch_interp(int64_t E, int n_in, int n_out, const T* M, int mode, const T* in,
                         const int32_t* lmap, const int32_t* seg, T* out_L, const int32_t* skip,
                         hipStream_t s);

// host: columns and contribution tables of the coarsest level (`on` stays
// false when it does not qualify; the cycle then runs cg_fixed_device)
sem_status setup_coarse(CoarseDev& C, const sem_mesh* m, const int64_t* gid,
                        const uint8_t* dirichlet, hipStream_t s);
// per solve: the matrix for (k, h2) and cleared exchange slots
sem_status prepare_coarse(CoarseDev& C, const sem_mesh* m, const double* k, double h2,
                          hipStream_t s);
// the launch fills at most a quarter of the chip (gridsync.hpp)
bool coarse_fits(const CoarseDev& C, bool f64);
// `iters` Jacobi-PCG iterations from x = 0 (as cg_fixed_device) in one launch
template <typename T>
sem_status coarse_cg(CoarseDev& C, const sem_mesh* m, const T* dinv, const T* b, T* x, int iters,
                     bool neumann, const CgScalars* outer, hipStream_t s);

// One V-cycle z = V(r) on free vectors of level 0 (Tr: the caller's vector
// type, Tp: the arithmetic of the cycle).  Coupled to an enclosing flexible CG
// through `cg` exactly as the Chebyshev preconditioner is (convergence gate
// first, z.r and z.(w - mean_w) partials last); a stand-alone call passes an
// empty ChebCg.  The hierarchy must have been prepared for the solve's k, h2.
template <typename Tr, typename Tp>
sem_status pmg_precond(const sem_mesh* m, SolveWork& W, const Tr* r, Tr* z, const ChebCg& cg,
                       hipStream_t s, int* applies);

// The Schwarz smoother of one level as a flexible-CG preconditioner (for the
// Lanczos bound of the Schwarz-preconditioned operator): z = S r.
sem_status schwarz_precond(Pmg& P, int level, const double* r, double* z, const ChebCg& cg,
                           hipStream_t s);

}  // namespace sem
