// Sparse coding of arbitrary shapes (omp_group.h) in FP64: used for every shape without a
// one-wave-per-signal kernel and for kernel option 1.
#include "omp_group_launch.h"

namespace sdl {

hipError_t omp_generic_f64_init_device() { return group_allow_lds<double>(); }

template <>
hipError_t launch_omp_generic<double>(const OmpArgs<double>& a, hipStream_t st) {
  return group_launch<double>(a, st);
}

int omp_generic_cost_f64(int m1, int m2, int n1, int n2, int s) {
  const GroupVariant* v = pick<double>(m1, m2, n1, n2, s);
  return v ? v->lanes * v->elems : 0;
}

}  // namespace sdl
