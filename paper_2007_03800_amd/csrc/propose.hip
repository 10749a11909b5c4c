// Learned support proposal, inference side: logits -> s atoms -> least squares.
//
// Sixteen lanes (one DPP row) share a signal, four signals per wave: each lane holds every 16th
// logit, s rounds of a row maximum (ties -> smallest atom index) pick the atoms in decreasing logit
// order, then the row solves the least-squares problem on them with the same Gram entries
// G1[i,i'] G2[j,j'] as 2D-OMP: lane t holds row t of the Gram matrix and turns it into row t of its
// Cholesky factor a column at a time, the column's entries reaching the other lanes by row
// broadcasts.  The residual is formed explicitly and the proposal accepted when
// ||r||^2 <= tau * ||Y||^2.  Rejected signals are listed (ascending) for the 2D-OMP fallback by a
// deterministic three-pass compaction.
//
// What bounds it: vector-ALU issue, about half of it the scans of the s rounds.  The earlier form
// factored the Gram matrix redundantly in every lane, with LDS permutes for every reduction and an
// integer division per table index; every entry is still computed by the same operations in the
// same order (written out below, so that a product and a subtraction fuse where they did), bit for
// bit.
#include <limits.h>
#include <math.h>

#include "lanes.h"
#include "mlp_internal.h"

namespace sdl {
namespace {

constexpr int kGroup = 16;

__device__ inline float row16_sum(float v) {
  v += dpp<kDppXor1>(v, v);
  v += dpp<kDppXor2>(v, v);
  v += dpp<kDppHalfMirror>(v, v);
  return v + dpp<kDppMirror>(v, v);
}
__device__ inline float row16_max(float v) {
  v = fmaxf(v, dpp<kDppXor1>(v, v));
  v = fmaxf(v, dpp<kDppXor2>(v, v));
  v = fmaxf(v, dpp<kDppHalfMirror>(v, v));
  return fmaxf(v, dpp<kDppMirror>(v, v));
}
__device__ inline int row16_min(int v) {
  v = min(v, dpp<kDppXor1>(v, v));
  v = min(v, dpp<kDppXor2>(v, v));
  v = min(v, dpp<kDppHalfMirror>(v, v));
  return min(v, dpp<kDppMirror>(v, v));
}

// f(IntC<0>) ... f(IntC<N - 1>)
template <int V>
struct IntC {
  static constexpr int value = V;
  __device__ constexpr operator int() const { return V; }
};
template <int L, int N, class F>
__device__ __forceinline__ void each(F&& f) {
  if constexpr (L < N) {
    f(IntC<L>{});
    each<L + 1, N>(f);
  }
}

template <int VPL, int SMAX>
__global__ void __launch_bounds__(256) propose_kernel(ProposeArgs a) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) float sm[];
  const int m1 = a.m1, m2 = a.m2, n1 = a.n1, n2 = a.n2, s = a.s, M = m1 * m2, A = n1 * n2;
  float* sG1 = sm;
  float* sG2 = sG1 + n1 * n1;
  float* sD1 = sG2 + n2 * n2;
  float* sD2 = sD1 + m1 * n1;
  for (int e = threadIdx.x; e < n1 * n1; e += blockDim.x) sG1[e] = a.G1[e];
  for (int e = threadIdx.x; e < n2 * n2; e += blockDim.x) sG2[e] = a.G2[e];
  for (int e = threadIdx.x; e < m1 * n1; e += blockDim.x) sD1[e] = a.D1[e];
  for (int e = threadIdx.x; e < m2 * n2; e += blockDim.x) sD2[e] = a.D2[e];
  __syncthreads();
  const int sub = threadIdx.x % kGroup;
  const int64_t k = (int64_t)blockIdx.x * (blockDim.x / kGroup) + threadIdx.x / kGroup;
  const bool valid = k < a.N;
  // a / n1 of an atom (a < 256) and e / m1 of a pixel (e < 64) by multiplication
  const int inv_n1 = 65536 / n1 + 1, inv_m1 = 65536 / m1 + 1;

  float v[VPL];
#pragma unroll
  for (int u = 0; u < VPL; ++u) v[u] = valid ? a.logits[k * A + sub + kGroup * u] : -INFINITY;
  int si[SMAX], sj[SMAX];  // the chosen atoms
  int mi = 0, mj = 0;      // lane t: the t-th
  each<0, SMAX>([&](auto t) __attribute__((always_inline)) {
    si[t] = sj[t] = 0;
    if (t < s) {
      float bv = v[0];
#pragma unroll
      for (int u = 1; u < VPL; ++u) bv = fmaxf(bv, v[u]);
      bv = row16_max(bv);
      int bu = INT_MAX;  // the smallest u that holds it
#pragma unroll
      for (int u = VPL - 1; u >= 0; --u) bu = v[u] == bv ? u : bu;
      // (-infinity is a logit already taken, and NaN never the largest: no atom is left then)
      const bool any = bv > -INFINITY;
      const int ba = row16_min(any && bu != INT_MAX ? sub + kGroup * bu : INT_MAX);
      const int own = (ba & (kGroup - 1)) == sub && ba != INT_MAX ? ba / kGroup : -1;
#pragma unroll
      for (int u = 0; u < VPL; ++u) v[u] = u == own ? -INFINITY : v[u];
      const int at = ba < A ? ba : 0;
      sj[t] = (at * inv_n1) >> 16;
      si[t] = at - n1 * sj[t];
      mi = sub == t ? si[t] : mi;
      mj = sub == t ? sj[t] : mj;
    }
  });
  // least squares on the proposed support
  const float* y = a.Y + (valid ? k : 0) * M;
  float yl[4];
  int pix1[4], pix2[4];
  float yy = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int e = sub + kGroup * w;
    yl[w] = (valid && e < M) ? y[e] : 0.f;
    yy = __builtin_fmaf(yl[w], yl[w], yy);
    const int ec = e < M ? e : 0;
    pix2[w] = (ec * inv_m1) >> 16;
    pix1[w] = ec - m1 * pix2[w];
  }
  yy = row16_sum(yy);
  float b = 0.f;  // lane t: the correlation of atom t
  each<0, SMAX>([&](auto t) __attribute__((always_inline)) {
    if (t < s) {
      const float *d1 = sD1 + m1 * si[t], *d2 = sD2 + m2 * sj[t];
      float c = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) c = __builtin_fmaf(yl[w] * d1[pix1[w]], d2[pix2[w]], c);
      c = row16_sum(c);
      b = sub == t ? c : b;
    }
  });
  // Cholesky of the support Gram matrix: lane t turns row t of the Gram matrix into row t of L
  float p1[SMAX], p2[SMAX], L[SMAX], diag[SMAX];
#pragma unroll
  for (int u = 0; u < SMAX; ++u) {
    p1[u] = sG1[mi + n1 * si[u]];
    p2[u] = sG2[mj + n2 * sj[u]];
    L[u] = p1[u] * p2[u];
  }
  bool bad = !valid;
  each<0, SMAX>([&](auto l) __attribute__((always_inline)) {
    diag[l] = 1.f;
    if (l < s) {
      const float d = bcast16<l.value>(L[l]);
      bad = bad || (sub == l && !(L[l] > 1e-6f * (p1[l] * p2[l])));
      diag[l] = d > 0.f ? sqrtf(d) : 1.f;
      L[l] = L[l] / diag[l];
      each<l.value + 1, SMAX>([&](auto u) __attribute__((always_inline)) {
        const float o = bcast16<u.value>(L[l]);
        L[u] = l == 0 ? __builtin_fmaf(p1[u], p2[u], -(L[l] * o)) : __builtin_fmaf(-L[l], o, L[u]);
      });
    }
  });
  // L L^T x = c: forward a column at a time, back a row at a time
  float x[SMAX];
  each<0, SMAX>([&](auto l) __attribute__((always_inline)) {
    x[l] = 0.f;
    if (l < s) {
      x[l] = bcast16<l.value>(b) / diag[l];
      b = __builtin_fmaf(-L[l], x[l], b);
    }
  });
  each<0, SMAX>([&](auto r) __attribute__((always_inline)) {
    constexpr int t = SMAX - 1 - r.value;
    if (t < s) {
      float q = x[t];
      each<t + 1, SMAX>([&](auto l) __attribute__((always_inline)) {
        const float o = bcast16<l.value>(L[t]);
        if (l < s) q = __builtin_fmaf(-o, x[l], q);
      });
      x[t] = q / diag[t];
    }
  });
  float rr = 0.f, mx = 0.f;
  float r[4] = {yl[0], yl[1], yl[2], yl[3]};
  each<0, SMAX>([&](auto t) __attribute__((always_inline)) {
    if (t < s) {
      const float *d1 = sD1 + m1 * si[t], *d2 = sD2 + m2 * sj[t];
#pragma unroll
      for (int w = 0; w < 4; ++w) r[w] = __builtin_fmaf(-(x[t] * d1[pix1[w]]), d2[pix2[w]], r[w]);
      mx = sub == t ? x[t] : mx;
    }
  });
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if (sub + kGroup * w < M) rr = __builtin_fmaf(r[w], r[w], rr);
  rr = row16_sum(rr);
  const unsigned long long bads = __ballot(bad) >> (threadIdx.x % kWave / kGroup * kGroup);
  const bool ok = (bads & ((1u << kGroup) - 1u)) == 0;
  if (valid) {
    if (sub < s) {
      a.supp[k * s + sub] = mi + n1 * mj;
      a.coef[k * s + sub] = ok ? mx : 0.f;
    }
    if (sub == 0) {
      if (a.res2) a.res2[k] = rr;
      a.accept[k] = (ok && (double)rr <= a.tau * (double)yy) ? 1 : 0;
    }
  }
}

constexpr int kCompact = 1024;  // signals per compaction block

__global__ void __launch_bounds__(kCompact) compact_count_kernel(const int32_t* accept, int64_t N, int32_t* blkcount) {
  __shared__ int wc[kCompact / 64];
  const int64_t k = (int64_t)blockIdx.x * kCompact + threadIdx.x;
  const bool rej = k < N && accept[k] == 0;
  const unsigned long long b = __ballot(rej);
  if (threadIdx.x % 64 == 0) wc[threadIdx.x / 64] = __popcll(b);
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < kCompact / 64; ++w) t += wc[w];
    blkcount[blockIdx.x] = t;
  }
}

// Exclusive sums of the block counts (one workgroup, kCompact counts a pass; one lane walking them
// took 92 us at 977 blocks).
__global__ void __launch_bounds__(kCompact) compact_scan_kernel(int32_t* blkcount, int nblk, int32_t* count) {
  __shared__ int ws[kCompact / kWave];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  int run = 0;
  for (int b0 = 0; b0 < nblk; b0 += kCompact) {
    const int b = b0 + (int)threadIdx.x;
    const int c = b < nblk ? blkcount[b] : 0;
    int inc = c;  // inclusive within the wave
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int up = __shfl_up(inc, o, kWave);
      if (lane >= o) inc += up;
    }
    if (lane == kWave - 1) ws[w] = inc;
    __syncthreads();
    int base = run;
    for (int q = 0; q < kCompact / kWave; ++q) {
      if (q < w) base += ws[q];
      run += ws[q];
    }
    if (b < nblk) blkcount[b] = base + inc - c;
    __syncthreads();
  }
  if (threadIdx.x == 0) *count = run;
}

__global__ void __launch_bounds__(kCompact) compact_write_kernel(const int32_t* accept, int64_t N, const int32_t* offs,
                                                                 int32_t* list) {
  __shared__ int wc[kCompact / 64];
  const int64_t k = (int64_t)blockIdx.x * kCompact + threadIdx.x;
  const bool rej = k < N && accept[k] == 0;
  const unsigned long long b = __ballot(rej);
  const int lane = threadIdx.x % 64, w = threadIdx.x / 64;
  if (lane == 0) wc[w] = __popcll(b);
  __syncthreads();
  int base = offs[blockIdx.x];
  for (int q = 0; q < w; ++q) base += wc[q];
  if (rej) list[base + __popcll(b & ((1ull << lane) - 1ull))] = (int32_t)k;
}

template <int VPL, int SMAX>
hipError_t launch_vs(const ProposeArgs& a, hipStream_t st) {
  const size_t lds = sizeof(float) * (a.n1 * a.n1 + a.n2 * a.n2 + a.m1 * a.n1 + a.m2 * a.n2);
  const int64_t blocks = (a.N + 15) / 16;
  hipLaunchKernelGGL((propose_kernel<VPL, SMAX>), dim3((unsigned)blocks), dim3(256), lds, st, a);
  return hipGetLastError();
}

}  // namespace

bool propose_supported(int n1, int n2, int s) {
  const int A = n1 * n2;
  return (A == 256 || A == 144) && s >= 1 && s <= 16 && n1 <= 64 && n2 <= 64;
}

hipError_t launch_propose(const ProposeArgs& a, hipStream_t st) {
  if (a.N == 0) return hipSuccess;
  if (a.m1 * a.m2 > 4 * kGroup) return hipErrorInvalidValue;
  const int A = a.n1 * a.n2;
  if (A == 256) return a.s <= 8 ? launch_vs<16, 8>(a, st) : launch_vs<16, 16>(a, st);
  if (A == 144) return a.s <= 8 ? launch_vs<9, 8>(a, st) : launch_vs<9, 16>(a, st);
  return hipErrorInvalidValue;
}

int compact_blocks(int64_t N) { return (int)((N + kCompact - 1) / kCompact); }

hipError_t launch_compact_rejected(const int32_t* accept, int64_t N, int32_t* blkcount, int32_t* list, int32_t* count,
                                   hipStream_t st) {
  const int nblk = compact_blocks(N);
  if (nblk == 0) return hipSuccess;
  hipLaunchKernelGGL(compact_count_kernel, dim3(nblk), dim3(kCompact), 0, st, accept, N, blkcount);
  hipLaunchKernelGGL(compact_scan_kernel, dim3(1), dim3(kCompact), 0, st, blkcount, nblk, count);
  hipLaunchKernelGGL(compact_write_kernel, dim3(nblk), dim3(kCompact), 0, st, accept, N, blkcount, list);
  return hipGetLastError();
}

}  // namespace sdl
