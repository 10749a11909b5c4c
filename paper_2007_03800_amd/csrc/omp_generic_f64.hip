// Sparse coding of arbitrary shapes (omp_group.h) in FP64: used for every shape without a
// one-wave-per-signal kernel and for kernel option 1.
#include "omp_group_launch.h"

namespace sdl {

hipError_t omp_generic_f64_init_device() { return group_allow_lds<double>(); }

template <>
hipError_t launch_omp_generic<double>(const OmpArgs<double>& a, hipStream_t st) {
  return group_launch<double>(a, st);
}

}  // namespace sdl
