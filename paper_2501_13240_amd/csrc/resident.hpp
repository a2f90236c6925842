// Jacobi-PCG of a small mesh as one resident kernel (see resident.hip).
#pragma once

#include "solver.hpp"

namespace sem {

// whether the mesh's solve in T can stay resident
template <typename T>
bool resident_fits(const sem_mesh* m);

// A solve's operator and free vectors: x, z = S r and p as k_init_pz leaves
// them, and S.
template <typename T>
struct ResidentArgs {
  Op<T> op;
  T *x, *z, *p;
  const T* dinv;
  bool profile;
};

// clears the exchange words for one solve
sem_status resident_begin(const sem_mesh* m, SolveWork& W, hipStream_t s);
// up to `iters` further iterations of the solve whose scalars are in W.sc
template <typename T>
sem_status resident_run(const sem_mesh* m, SolveWork& W, const ResidentArgs<T>& a, int iters,
                        hipStream_t s);

}  // namespace sem
