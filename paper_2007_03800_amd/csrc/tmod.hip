// TMOD dictionary update kernels (Algorithm 1 steps 1-4; Corollary 1, Result 1).
//
// Side 1 (D1 update, Corollary 1):  T_k = X_k D2^T (n1 x m2)
//     A = sum_k T_k T_k^T (n1 x n1),  B = sum_k Y_k T_k^T (m1 x n1),  D1* = B A^{-1}
// Side 2 (D2 update, Result 1): Z_k = D1 X_k (m1 x n2), U_k = Z_k^T
//     A = sum_k Z_k^T Z_k (n2 x n2),  B = sum_k Y_k^T Z_k (m2 x n2),  D2* = B A^{-1}
// Both are written once with "row atoms" ra (i for side 1, j for side 2), the
// signal seen as Yt (Y for side 1, Y^T for side 2) and the fixed dictionary Do
// (D2 for side 1, D1 for side 2): T[ra][c] = sum over code entries x * Do[c, rb].
//
// One GPU plays every node of Algorithm 1: each workgroup owns a contiguous
// slice of signals (a "node"), accumulates its partial sums, and writes them as
// FP64 partials; a fixed-order FP64 reduction (the master's sum) and an FP64
// Cholesky solve on one workgroup follow.  Nothing uses floating-point atomics,
// so results are bitwise reproducible.
#include <math.h>

#include "sdl_internal.h"
#include "tmod_device.h"

namespace sdl {
namespace {

// Fixed-order two-stage reduction of P partial rows of nent doubles: stage 1 sums
// consecutive chunks of kChunk rows per entry (in row order), stage 2 the chunk sums
// (in chunk order).
constexpr int kChunk = 64;

__global__ void reduce_stage1_kernel(const double* __restrict__ part, int P, int nent, double* stage) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const int c = blockIdx.y;
  if (e >= nent) return;
  const int b0 = c * kChunk, b1 = (c + 1) * kChunk < P ? (c + 1) * kChunk : P;
  double v = 0.0;
  if (b1 - b0 == kChunk) {
    // a whole chunk: every load issued before the adds, which stay in row order
    double q[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) q[u] = part[(size_t)(b0 + u) * nent + e];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) v += q[u];
  } else {
    for (int b = b0; b < b1; ++b) v += part[(size_t)b * nent + e];
  }
  stage[(size_t)c * nent + e] = v;
}

// The last reduction stage alone: out[e] = sum over the nrow rows of src (row stride ld)
// in row order, for e < n (the same order as the solve kernel's first stage).
__global__ void reduce_final_kernel(const double* __restrict__ src, int nrow, int ld, int n, double* out) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  double v = 0.0;
  for (int b = 0; b < nrow; ++b) v += src[(size_t)b * ld + e];
  out[e] = v;
}

constexpr int kSolveThreads = 512;
constexpr int kDirectRows = 2 * kChunk;  // up to this many partial rows the solve sums them itself

// The master step of Algorithm 1 (steps 2 and 4) in one workgroup: the last stage of
// the fixed-order reduction, sums[e] = sum over the nrow rows of src (row stride ld)
// in row order, then the solve and normalisation on the reduced [A | B]; optionally
// the reduced sum of squared residuals (sums[r.idx]) becomes the RMSE of the sweep
// that produced the codes.
template <typename T>
__global__ void __launch_bounds__(kSolveThreads)
    tmod_solve_kernel(const double* __restrict__ src, int nrow, int ld, double* sums, int mr, int na, double* D,
                      T* Dc, T* Gc, double* w, int* status, unsigned long long* counters, RmseOut r,
                      int sums_in_lds) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int tid = threadIdx.x;
  // the reduced sums go to global memory (the caller's copy) and, when sums_in_lds, to the
  // front of LDS, where the solve reads them
  double* ssum = reinterpret_cast<double*>(smem_raw);
  for (int e = tid; e < ld; e += blockDim.x) {
    double v = 0.0;
    int b = 0;
    for (; b + 8 <= nrow; b += 8) {  // eight loads in flight, adds in row order
      double q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = src[(size_t)(b + u) * ld + e];
#pragma unroll
      for (int u = 0; u < 8; ++u) v += q[u];
    }
    for (; b < nrow; ++b) v += src[(size_t)b * ld + e];
    sums[e] = v;
    if (sums_in_lds) ssum[e] = v;
  }
  __syncthreads();
  const double* rs = sums_in_lds ? ssum : sums;
  if (r.trace && tid == 0) {
    const int it = *r.counter;
    r.trace[(size_t)it + r.offset] = r.denom > 0 ? sqrt(rs[r.idx] / r.denom) : 0.0;
    *r.counter = it + 1;
  }
  solve_update_block<T>(rs, mr, na, D, Dc, Gc, w, status, counters,
                        smem_raw + (sums_in_lds ? solve_sums_lds_bytes(ld) : 0), tid, blockDim.x);
}

// What a call needs before its first sparse coding, in one launch: every dictionary's compute-type
// copy and Gram matrix, and the call's status words and counters set to zero (five launches of about
// 1.5 us each and their gaps before, a third of a 64-signal call).  A dictionary may be given as the
// Kronecker product of several modes' (n-dimensional problems).  Workgroups of one dictionary each
// stage it in LDS at an odd column stride, so that the Gram entries read LDS without bank conflicts,
// and share the Gram matrix (256 entries each, at most kPrepParts of them; a 72-atom Kronecker factor
// in 8 parts took 13 us).
constexpr int kPrepParts = 24;

template <typename T>
struct PrepBatch {
  PrepJob<T> j[kMaxPrepJobs];
  int first[kMaxPrepJobs + 1];
  int* zero[kMaxPrepZero];
  int nzero[kMaxPrepZero];
};

template <typename T>
__global__ void __launch_bounds__(256) call_prep_kernel(PrepBatch<T> b) {
  __shared__ double sD[(SDL_MAX_M + 1) * SDL_MAX_N];
  const int tid = threadIdx.x, nt = blockDim.x;
  if ((int)blockIdx.x >= b.first[kMaxPrepJobs]) {
#pragma unroll
    for (int z = 0; z < kMaxPrepZero; ++z)
      for (int i = tid; i < b.nzero[z]; i += nt) b.zero[z][i] = 0;
    return;
  }
  int which = 0;
  while (which < kMaxPrepJobs - 1 && (int)blockIdx.x >= b.first[which + 1]) ++which;
  const PrepJob<T>& g = b.j[which];
  const int part = (int)blockIdx.x - b.first[which], nparts = b.first[which + 1] - b.first[which];
  if (part == 0 && tid == 0 && g.zero) *g.zero = 0;
  int mr = 1, na = 1;
  for (int q = 0; q < g.nfac; ++q) {
    mr *= g.m[q];
    na *= g.n[q];
  }
  const int ldd = mr + 1;
  for (int e = tid; e < mr * na; e += nt) {
    const int r = e % mr, c = e / mr;
    double v;
    if (g.nfac == 1) {
      v = g.F[0][e];
    } else {
      v = 1.0;
      int p = r, j = c;
      for (int q = 0; q < g.nfac; ++q) {
        const int pq = p % g.m[q], iq = j % g.n[q];
        p /= g.m[q];
        j /= g.n[q];
        v *= g.F[q][pq + g.m[q] * iq];
      }
    }
    sD[r + ldd * c] = v;
    if (part == 0) g.Dc[e] = (T)v;
  }
  __syncthreads();
  for (int e = tid + nt * part; e < na * na; e += nt * nparts) {
    const int i = e % na, j = e / na;
    double v = 0.0;
    for (int p = 0; p < mr; ++p) v += sD[p + ldd * i] * sD[p + ldd * j];
    g.Gc[e] = (T)v;
  }
}

template <typename T>
__global__ void rescale_kernel(int side, int n1, int s, int64_t N, const int32_t* supp, T* coef,
                               const double* w) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N * s) return;
  const int at = supp[e];
  if (at < 0) return;
  const int idx = side == 1 ? at % n1 : at / n1;
  coef[e] = (T)((double)coef[e] * w[idx]);
}

constexpr int kRmseThreads = 256;

// Sum of N squared residuals in a fixed order: each workgroup writes its slice's sum, the last one to
// finish (a counter that it sets back to zero) adds the slices' sums, writes the RMSE and moves the
// trace position on.  (Sweeps that an update follows leave this to the update's sums.)  The slices' sums pass between workgroups by device-scope
// atomics.  (A second launch whose single lane walked the slices took 4-15 us.)
template <typename T>
__global__ void __launch_bounds__(kRmseThreads)
    res2_sum_kernel(const T* res2, int64_t N, double* part, int* done, double denom, double* trace, int stride, int offset,
                    int* counter) {
  __shared__ double red[kRmseThreads];
  __shared__ int last;
  const int nblk = gridDim.x, tid = threadIdx.x;
  const int64_t k0 = (N * blockIdx.x) / nblk, k1 = (N * (blockIdx.x + 1)) / nblk;
  auto block_sum = [&](double v) {
    red[tid] = v;
    __syncthreads();
    for (int o = kRmseThreads / 2; o > 0; o >>= 1) {
      if (tid < o) red[tid] += red[tid + o];
      __syncthreads();
    }
  };
  double v = 0.0;
#pragma unroll 4
  for (int64_t k = k0 + tid; k < k1; k += kRmseThreads) v += (double)res2[k];
  block_sum(v);
  if (tid == 0) {
    __hip_atomic_store(&part[blockIdx.x], red[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == nblk - 1;
  }
  __syncthreads();
  if (!last) return;
  v = 0.0;
  for (int b = tid; b < nblk; b += kRmseThreads) v += __hip_atomic_load(&part[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  block_sum(v);
  if (tid == 0) {
    *done = 0;
    const int it = *counter;
    trace[(size_t)it * stride + offset] = denom > 0 ? sqrt(red[0] / denom) : 0.0;
    *counter = it + 1;
  }
}

__global__ void fill_double_kernel(double* p, int n, double v) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) p[e] = v;
}

template <typename T>
__global__ void check_finite_kernel(const T* x, int64_t n, int* status) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    if (!isfinite((double)x[e])) {
      atomicOr(status, kStatusNonfinite);
      return;
    }
  }
}

__global__ void check_finite_bf16_kernel(const uint16_t* x, int64_t n, int* status) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    if ((x[e] & 0x7F80u) == 0x7F80u) {  // exponent all ones: infinity or NaN
      atomicOr(status, kStatusNonfinite);
      return;
    }
  }
}

}  // namespace

int launch_reduce_stage1(const double* part, int P, int ld, double* stage, const double** src, hipStream_t st,
                         hipError_t* err) {
  *err = hipSuccess;
  if (P <= kDirectRows) {
    *src = part;
    return P;
  }
  const int nchunk = (P + kChunk - 1) / kChunk;
  hipLaunchKernelGGL(reduce_stage1_kernel, dim3((ld + 255) / 256, nchunk), dim3(256), 0, st, part, P, ld, stage);
  *err = hipGetLastError();
  *src = stage;
  return nchunk;
}

int reduce_stage_rows(int P) { return (P + kChunk - 1) / kChunk; }

hipError_t launch_reduce_final(const double* src, int nrow, int ld, int n, double* out, hipStream_t st) {
  hipLaunchKernelGGL(reduce_final_kernel, dim3((n + 255) / 256), dim3(256), 0, st, src, nrow, ld, n, out);
  return hipGetLastError();
}

hipError_t launch_fill_double(double* p, int n, double v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_double_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tmod_solve(const double* src, int nrow, int ld, double* sums, int mr, int na, double* D, T* Dc,
                             T* Gc, double* w, int* status, unsigned long long* counters,
                             const RmseOut& r, hipStream_t st) {
  // the reduced sums stay in LDS too when they fit beside the solve's workspace
  const size_t base = solve_lds_bytes(na, mr), with = base + solve_sums_lds_bytes(ld);
  const int in_lds = with <= solve_lds_bytes(SDL_MAX_N, SDL_MAX_M) ? 1 : 0;
  hipLaunchKernelGGL(tmod_solve_kernel<T>, dim3(1), dim3(kSolveThreads), in_lds ? with : base, st, src, nrow, ld,
                     sums, mr, na, D, Dc, Gc, w, status, counters, r, in_lds);
  return hipGetLastError();
}

hipError_t tmod_solve_init_device() {
  const int bytes = (int)solve_lds_bytes(SDL_MAX_N, SDL_MAX_M);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tmod_solve_kernel<float>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&tmod_solve_kernel<double>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <typename T>
hipError_t launch_call_prep(const PrepJob<T>* jobs, int n, int* const* zero, const int* nzero, int nz, hipStream_t st) {
  if (nz > kMaxPrepZero) return hipErrorInvalidValue;
  for (int j0 = 0; j0 < n || j0 == 0; j0 += kMaxPrepJobs) {
    PrepBatch<T> b{};
    int blocks = 0;
    for (int q = 0; q < kMaxPrepJobs; ++q) {
      b.first[q] = blocks;
      if (j0 + q >= n) continue;
      const PrepJob<T>& g = b.j[q] = jobs[j0 + q];
      int mr = 1, na = 1;
      for (int d = 0; d < g.nfac; ++d) {
        mr *= g.m[d];
        na *= g.n[d];
      }
      if ((mr + 1) * na > (SDL_MAX_M + 1) * SDL_MAX_N) return hipErrorInvalidValue;
      const int parts = (na * na + 255) / 256;
      blocks += parts < kPrepParts ? parts : kPrepParts;
    }
    b.first[kMaxPrepJobs] = blocks;
    if (j0 == 0 && nz > 0) {
      for (int z = 0; z < nz; ++z) {
        b.zero[z] = zero[z];
        b.nzero[z] = nzero[z];
      }
      ++blocks;
    }
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(call_prep_kernel<T>, dim3(blocks), dim3(256), 0, st, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
hipError_t launch_rescale(int side, int n1, int s, int64_t N, const int32_t* supp, T* coef, const double* w,
                          hipStream_t st) {
  const int64_t n = N * s;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(rescale_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, side, n1, s, N, supp,
                     coef, w);
  return hipGetLastError();
}

int rmse_num_blocks(int64_t N) {
  int64_t b = (N + 4095) / 4096;
  if (b > 1024) b = 1024;
  if (b < 1) b = 1;
  return (int)b;
}

template <typename T>
hipError_t launch_rmse(const T* res2, int64_t N, double denom, double* part, int nblk, int* done, double* trace,
                       int stride, int offset, int* counter, hipStream_t st) {
  hipLaunchKernelGGL(res2_sum_kernel<T>, dim3(nblk), dim3(kRmseThreads), 0, st, res2, N, part, done, denom, trace,
                     stride, offset, counter);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_check_finite(const T* x, int64_t n, int* status, hipStream_t st) {
  if (n == 0) return hipSuccess;
  int64_t g = (n + 255) / 256;
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(check_finite_kernel<T>, dim3((unsigned)g), dim3(256), 0, st, x, n, status);
  return hipGetLastError();
}

hipError_t launch_check_finite_bf16(const uint16_t* x, int64_t n, int* status, hipStream_t st) {
  if (n == 0) return hipSuccess;
  int64_t g = (n + 255) / 256;
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(check_finite_bf16_kernel, dim3((unsigned)g), dim3(256), 0, st, x, n, status);
  return hipGetLastError();
}

#define SDL_INST(T)                                                                                            \
  template hipError_t launch_tmod_solve<T>(const double*, int, int, double*, int, int, double*, T*, T*, \
                                           double*, int*, unsigned long long*, const RmseOut&, hipStream_t);  \
  template hipError_t launch_call_prep<T>(const PrepJob<T>*, int, int* const*, const int*, int, hipStream_t);  \
  template hipError_t launch_rescale<T>(int, int, int, int64_t, const int32_t*, T*, const double*,            \
                                        hipStream_t);                                                         \
  template hipError_t launch_rmse<T>(const T*, int64_t, double, double*, int, int*, double*, int, int, int*,  \
                                     hipStream_t);                                                            \
  template hipError_t launch_check_finite<T>(const T*, int64_t, int*, hipStream_t);
SDL_INST(float)
SDL_INST(double)
#undef SDL_INST

}  // namespace sdl
