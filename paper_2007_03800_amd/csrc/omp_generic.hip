// Sparse coding of arbitrary shapes (omp_group.h) in FP32: used for every shape without a kernel of
// its own and for kernel option 1.
#include "omp_group_launch.h"

namespace sdl {

hipError_t omp_generic_f64_init_device();  // omp_generic_f64.hip

// Elements of LDS the first form of this path (one signal per workgroup, everything in LDS) took;
// shapes beyond 160 KiB of it are refused (every shape within it has a variant that fits).
size_t omp_generic_lds_bytes(int m1, int m2, int n1, int n2, int s, size_t elem) {
  const size_t end = (size_t)m1 * n1 + m2 * n2 + n1 * n1 + n2 * n2 + m1 * m2 + n1 * m2 + n1 * n2 + s * s + 3 * s;
  return end * elem + sizeof(int) * (size_t)s + (size_t)n1 * n2 + 16;
}

hipError_t omp_generic_init_device() {
  const hipError_t e = group_allow_lds<float>();
  return e == hipSuccess ? omp_generic_f64_init_device() : e;
}

template <>
hipError_t launch_omp_generic<float>(const OmpArgs<float>& a, hipStream_t st) {
  return group_launch<float>(a, st);
}

}  // namespace sdl
