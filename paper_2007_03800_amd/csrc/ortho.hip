// Orthonormal variant of the method (Remark 1): square dictionaries with orthonormal columns
// (n1 = m1, n2 = m2).  Sparse coding needs no least squares: X_k = T_s(D1^T Y_k D2), the s
// entries of largest magnitude.  The dictionary update is the orthogonal Procrustes solution:
// the polar factor U V^T of the update's B sum (sum_k Y_k D2 X_k^T for D1, sum_k Y_k^T D1 X_k
// for D2), on one wave in FP64 by Newton's iteration, by one-sided Jacobi rotations where the sum is too
// far from well conditioned for that.
//
// Codes: a wave codes four signals, sixteen lanes per signal.  The signals are staged in LDS;
// V = Y D2 and C = D1^T V are formed entry by entry (lane l of the signal owns entries
// e = l + 16 u), C stays in registers, and s rounds of a 16-lane argmax (exact magnitude
// comparison, ties to the smaller atom) take the largest entries in decreasing order.  The
// residual energy comes from the explicit residual, as in the oracle.
#include <limits.h>
#include <math.h>

#include "sdl_internal.h"

namespace sdl {
namespace {

constexpr int kOWaves = 4;
constexpr int kOLanes = 16;  // lanes per signal
constexpr int kOSigs = 4;    // signals per wave
constexpr int kOMaxPer = 16;  // entries of C per lane (m1 m2 <= 256)
constexpr int kOMaxBlocks = 4096;

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
__device__ inline T sig_load(const OmpArgs<T>& a, int64_t e) {
  return a.Y[e];
}

// Cross-lane moves inside a row of 16 lanes by DPP (no LDS round trip): quad swaps (lane xor 1,
// xor 2), half-row mirror (lane i <-> 7 - i within each 8) and row mirror (i <-> 15 - i).  After
// the four steps of a commutative, associative combine every lane of the row holds the row's
// result.
constexpr int kDppX1 = 0xB1, kDppX2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
template <int CTRL>
__device__ inline int dpp_int(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL, typename U>
__device__ inline U dpp_move(U v) {
  if constexpr (sizeof(U) == 4) {
    return __builtin_bit_cast(U, dpp_int<CTRL>(__builtin_bit_cast(int, v)));
  } else {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = dpp_int<CTRL>((int)(b & 0xffffffffll)), hi = dpp_int<CTRL>((int)(b >> 32));
    return __builtin_bit_cast(U, ((long long)hi << 32) | (unsigned int)lo);
  }
}
template <typename U>
__device__ inline U row16_sum(U v) {
  v += dpp_move<kDppX1>(v);
  v += dpp_move<kDppX2>(v);
  v += dpp_move<kDppHalfMirror>(v);
  v += dpp_move<kDppMirror>(v);
  return v;
}
// (value, index) maximum over the row, ties to the smaller index
template <int CTRL, typename U>
__device__ inline void argmax_step(U& v, int& idx) {
  const U ov = dpp_move<CTRL>(v);
  const int oi = dpp_int<CTRL>(idx);
  const bool take = ov > v || (ov == v && oi < idx);
  v = take ? ov : v;
  idx = take ? oi : idx;
}
template <typename U>
__device__ inline void row16_argmax(U& v, int& idx) {
  argmax_step<kDppX1>(v, idx);
  argmax_step<kDppX2>(v, idx);
  argmax_step<kDppHalfMirror>(v, idx);
  argmax_step<kDppMirror>(v, idx);
}
template <typename U>
__device__ inline U lane_value(U v, int k) {  // value of lane k (k uniform)
  if constexpr (sizeof(U) == 4) {
    return __builtin_bit_cast(U, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
  } else {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), k);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __builtin_bit_cast(U, ((long long)hi << 32) | (unsigned int)lo);
  }
}

template <typename T>
__global__ void __launch_bounds__(kWave* kOWaves) ortho_code_kernel(OmpArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int m1 = a.m1, m2 = a.m2, M = m1 * m2, s = a.s;
  T* sD1 = reinterpret_cast<T*>(smem_raw);  // m1 x m1
  T* sD2 = sD1 + m1 * m1;                    // m2 x m2
  T* wsY = sD2 + m2 * m2;                    // [kOWaves][kOSigs][M] signals
  T* wsV = wsY + (size_t)kOWaves * kOSigs * M;  // [kOWaves][kOSigs][M] Y D2
  T* wsC = wsV + (size_t)kOWaves * kOSigs * M;  // [kOWaves][kOSigs][32] chosen values
  int* wsA = reinterpret_cast<int*>(wsC + (size_t)kOWaves * kOSigs * 32);  // [..][32] chosen atoms
  const int tid = threadIdx.x, wv = tid / kWave, lane = tid % kWave;
  const int g = lane / kOLanes, l = lane % kOLanes;
  for (int e = tid; e < m1 * m1; e += blockDim.x) sD1[e] = a.D1[e];
  for (int e = tid; e < m2 * m2; e += blockDim.x) sD2[e] = a.D2[e];
  __syncthreads();
  T* ys = wsY + (size_t)(wv * kOSigs + g) * M;
  T* vs = wsV + (size_t)(wv * kOSigs + g) * M;
  T* cs = wsC + (size_t)(wv * kOSigs + g) * 32;
  int* as = wsA + (size_t)(wv * kOSigs + g) * 32;
  const int64_t ngroups = (a.N + kOSigs - 1) / kOSigs;
  const int nper = (M + kOLanes - 1) / kOLanes;
  for (int64_t grp = (int64_t)blockIdx.x * kOWaves + wv; grp < ngroups; grp += (int64_t)gridDim.x * kOWaves) {
    const int64_t k = grp * kOSigs + g;
    const bool valid = k < a.N;
    for (int e = l; e < M; e += kOLanes) ys[e] = valid ? sig_load(a, k * M + e) : T(0);
    wave_sync();
    // V = Y D2: entry (p, j) at p + m1 j
    for (int e = l; e < M; e += kOLanes) {
      const int p = e % m1, j = e / m1;
      T v = 0;
      for (int q = 0; q < m2; ++q) v += ys[p + m1 * q] * sD2[q + m2 * j];
      vs[e] = v;
    }
    wave_sync();
    // C = D1^T V: entry (i, j), atom a = i + m1 j, owned by lane a % 16
    T cv[kOMaxPer];
#pragma unroll
    for (int u = 0; u < kOMaxPer; ++u) {
      const int e = l + kOLanes * u;
      T v = 0;
      if (u < nper && e < M) {
        const int i = e % m1, j = e / m1;
        for (int p = 0; p < m1; ++p) v += sD1[p + m1 * i] * vs[p + m1 * j];
      }
      cv[u] = v;
    }
    unsigned taken = 0u;  // bit u: entry u of this lane already chosen
    for (int t = 0; t < s; ++t) {
      // this lane's largest remaining |C| (ties: smaller atom, i.e. smaller u)
      T best = T(-1);
      int ba = INT_MAX;
#pragma unroll
      for (int u = 0; u < kOMaxPer; ++u) {
        const int e = l + kOLanes * u;
        const T m = fabs(cv[u]);
        const bool ok = u < nper && e < M && !((taken >> u) & 1u) && m > best;
        best = ok ? m : best;
        ba = ok ? e : ba;
      }
      // across the signal's 16 lanes (one DPP row)
      row16_argmax(best, ba);
      // the owner lane marks it and provides the signed value
      T val = 0;
      if (ba != INT_MAX && ba % kOLanes == l) {
        const int u = ba / kOLanes;
#pragma unroll
        for (int uu = 0; uu < kOMaxPer; ++uu) val = uu == u ? cv[uu] : val;
        taken |= 1u << u;
      }
      val = row16_sum(val);  // only the owner is nonzero
      if (valid && l == 0) {
        a.supp[k * s + t] = ba == INT_MAX ? -1 : ba;
        a.coef[k * s + t] = ba == INT_MAX ? T(0) : val;
      }
      // the chosen values for the residual
      if (l == 0) {
        cs[t] = val;
        as[t] = ba == INT_MAX ? -1 : ba;
      }
    }
    wave_sync();
    // explicit residual energy
    T rr = 0;
    for (int e = l; e < M; e += kOLanes) {
      const int p = e % m1, q = e / m1;
      T r = ys[e];
      for (int t = 0; t < s; ++t) {
        const int at = as[t];
        if (at >= 0) r -= cs[t] * sD1[p + m1 * (at % m1)] * sD2[q + m2 * (at / m1)];
      }
      rr += r * r;
    }
    rr = row16_sum(rr);
    if (valid && l == 0 && a.res2) a.res2[k] = rr;
    wave_sync();
  }
}

__device__ inline double wave_sum(double v) {
  v = row16_sum(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
__device__ inline double reciprocal(double x) {  // the hardware's estimate, corrected twice
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}
// the magnitude's leading bits with the row in the low five, rows already used last
__device__ inline unsigned pivot_key(double v, int row, bool used) {
  const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32);
  return used ? 0u : 0x80000000u | (hi & 0x7FFFFFE0u) | (unsigned)row;
}

// Polar factor of the n x n matrix W (column-major, LDS) by Newton's iteration
// X <- (mu X + X^-T / mu) / 2, mu = sqrt(|X^-1|_F / |X|_F) (Higham), each inverse by Gauss-Jordan in
// place with row pivoting.  False, W unchanged, where |X|_F |X^-1|_F exceeds 1e6 or the iteration does
// not settle: the caller then takes the singular values themselves.  R: n x n scratch, buf: 64 doubles,
// perm: 64 ints.  What bounds it: the chain of one wave, about 200 cycles a pivot at n <= 8, where
// entry (i, j) of X stays in lane i + 8 j and rows and columns are broadcast by lane permutes.  Five to
// seven inverses replace about 45 rounds of Jacobi rotations: 128,000 signals, n = 8: 23 -> 15 us a launch.
constexpr double kPolarCond = 1e6, kPolarDone = 2e-16;  // the last step's change squared: error below 1e-16
__device__ inline bool polar_newton8(double* W, int n) {
  const int x = threadIdx.x, i = x % 8, j = x / 8;
  const bool in = i < n && j < n;
  const double eye = i == j ? 1.0 : 0.0;
  double X = in ? W[i + n * j] : 0.0;
  const double f = wave_sum(X * X);
  if (!(f > 0.0) || !(f < 1e300) || !(f > 1e-300)) return false;
  X = in ? X * (sqrt((double)n) / sqrt(f)) : eye;  // lanes beyond n x n hold the identity throughout
  bool scaled = true;
  for (int it = 0; it < 24; ++it) {
    double R = X;
    unsigned used = 0xFFu & ~((1u << n) - 1u), prow = 0x76543210u, pinv = 0x76543210u;
    for (int k = 0; k < n; ++k) {
      const double c = __shfl(R, i + 8 * k, kWave);
      unsigned key = pivot_key(c, i, (used >> i) & 1u);
      key = max(key, (unsigned)dpp_int<kDppX1>((int)key));
      key = max(key, (unsigned)dpp_int<kDppX2>((int)key));
      key = max(key, (unsigned)dpp_int<kDppHalfMirror>((int)key));
      const int p = __builtin_amdgcn_readfirstlane((int)(key & 7u));
      const double pv = lane_value(R, p + 8 * k);
      if (!(fabs(pv) > 1e-200)) return false;
      const double rp = reciprocal(pv), row = __shfl(R, p + 8 * j, kWave) * rp;
      used |= 1u << p;
      prow = (prow & ~(15u << (4 * k))) | ((unsigned)p << (4 * k));
      pinv = (pinv & ~(15u << (4 * p))) | ((unsigned)k << (4 * p));
      const double v = j == k ? -c * rp : __builtin_fma(-c, row, R);
      const double w = j == k ? rp : row;
      R = i == p ? w : v;
    }
    // row p_k of R is row k of the inverse, its column l belongs to row p_l of X
    const double Y = __shfl(R, (int)((prow >> (4 * j)) & 7u) + 8 * (int)((pinv >> (4 * i)) & 7u), kWave);
    const double fx = wave_sum(in ? X * X : 0.0), fy = wave_sum(in ? Y * Y : 0.0);
    if (!(fx * fy <= kPolarCond * kPolarCond)) return false;
    const double mu = scaled ? sqrt(sqrt(fy / fx)) : 1.0;
    const double Z = in ? 0.5 * (mu * X + Y * reciprocal(mu)) : eye;
    const double d = wave_sum((Z - X) * (Z - X));
    X = Z;
    if (d <= kPolarDone) {
      if (in) W[i + n * j] = X;
      wave_sync();
      return true;
    }
    scaled = d > 1e-2;
  }
  return false;
}
__device__ inline bool polar_newton(double* W, double* R, double* X, double* buf, int* perm, int n) {
  const int x = threadIdx.x, nent = n * n;
  double f = 0.0;
  for (int e = x; e < nent; e += kWave) f += W[e] * W[e];
  f = wave_sum(f);
  if (!(f > 0.0) || !(f < 1e300) || !(f > 1e-300)) return false;
  const double f1 = sqrt((double)n) / sqrt(f);
  for (int e = x; e < nent; e += kWave) X[e] = W[e] * f1;
  wave_sync();
  const int di = kWave % n, dj = kWave / n;
  double *col = buf, *row = buf + 32;
  int *prow = perm, *pinv = perm + 32;
  bool scaled = true;
  for (int it = 0; it < 24; ++it) {
    for (int e = x; e < nent; e += kWave) R[e] = X[e];
    bool used = x >= n;
    wave_sync();
    for (int k = 0; k < n; ++k) {
      const double c = x < n ? R[x + n * k] : 0.0;
      unsigned key = pivot_key(c, x, used);
      key = max(key, (unsigned)dpp_int<kDppX1>((int)key));
      key = max(key, (unsigned)dpp_int<kDppX2>((int)key));
      key = max(key, (unsigned)dpp_int<kDppHalfMirror>((int)key));
      key = max(key, (unsigned)dpp_int<kDppMirror>((int)key));
      const int p = (int)(max((unsigned)__builtin_amdgcn_readlane((int)key, 0),
                              (unsigned)__builtin_amdgcn_readlane((int)key, 16)) & 31u);
      const double pv = lane_value(c, p);
      if (!(fabs(pv) > 1e-200)) return false;
      const double rp = reciprocal(pv);
      if (x < n) {
        col[x] = c;
        row[x] = R[p + n * x] * rp;
      }
      if (x == 0) {
        prow[k] = p;
        pinv[p] = k;
      }
      used = used || x == p;
      wave_sync();
      int i = x % n, j = x / n;
      for (int e = x; e < nent; e += kWave) {
        const double ci = col[i], rj = row[j], r = R[e];
        const double v = j == k ? -ci * rp : __builtin_fma(-ci, rj, r);
        const double w = j == k ? rp : rj;
        R[e] = i == p ? w : v;
        i += di;
        j += dj;
        if (i >= n) {
          i -= n;
          ++j;
        }
      }
      wave_sync();
    }
    double fx = 0.0, fy = 0.0;
    for (int e = x; e < nent; e += kWave) {
      fx += X[e] * X[e];
      fy += R[e] * R[e];
    }
    fx = wave_sum(fx);
    fy = wave_sum(fy);
    if (!(fx * fy <= kPolarCond * kPolarCond)) return false;
    const double mu = scaled ? sqrt(sqrt(fy / fx)) : 1.0, rmu = reciprocal(mu);
    double d = 0.0;
    for (int e = x; e < nent; e += kWave) {
      const double v = X[e], z = 0.5 * (mu * v + R[prow[e / n] + n * pinv[e % n]] * rmu);
      d += (z - v) * (z - v);
      X[e] = z;
    }
    d = wave_sum(d);
    wave_sync();
    if (d <= kPolarDone) {
      for (int e = x; e < nent; e += kWave) W[e] = X[e];
      wave_sync();
      return true;
    }
    scaled = d > 1e-2;
  }
  return false;
}

// One-sided Jacobi rotations of the columns of W (n x n, n <= 8), gathered in V: up to four disjoint
// column pairs rotated at once (round-robin order: n' - 1 rounds of n' / 2 pairs cover every pair once
// per sweep, n' = n rounded up to even, pairs with the dummy column n skipped); lane 8 q + r holds row r
// for the q-th pair of the round.  The polar factor is unique for a full-rank B, so the order of the
// rotations changes only rounding.  (A dictionary update with an ill-conditioned B at n = 8: 75 us a call, 102
// with one pair at a time as above eight columns.)
__device__ inline void jacobi8(double* W, double* V, int n) {
  const int x = threadIdx.x, np = n + (n & 1), q = x / 8, r = x % 8;
  for (int sweep = 0; sweep < 60; ++sweep) {
    bool rotated = false;
    for (int round = 0; round < np - 1; ++round) {
      int i = -1, j = -1;
      if (q < np / 2) {
        if (q == 0) {
          i = np - 1;
          j = round;
        } else {
          i = (round + q) % (np - 1);
          j = (round - q + np - 1) % (np - 1);
        }
        if (i > j) {
          const int tmp = i;
          i = j;
          j = tmp;
        }
      }
      const bool act = j >= 0 && j < n;  // a real pair (the dummy column is n)
      double pa = 0.0, pb = 0.0, pg = 0.0;
      if (act && r < n) {
        const double wi = W[r + n * i], wj = W[r + n * j];
        pa = wi * wi;
        pb = wj * wj;
        pg = wi * wj;
      }
      // sums over the pair's eight lanes (quad swaps and the half-row mirror)
      pa += dpp_move<kDppX1>(pa);
      pb += dpp_move<kDppX1>(pb);
      pg += dpp_move<kDppX1>(pg);
      pa += dpp_move<kDppX2>(pa);
      pb += dpp_move<kDppX2>(pb);
      pg += dpp_move<kDppX2>(pg);
      pa += dpp_move<kDppHalfMirror>(pa);
      pb += dpp_move<kDppHalfMirror>(pb);
      pg += dpp_move<kDppHalfMirror>(pg);
      const bool rot = act && !(fabs(pg) <= 1e-15 * sqrt(pa * pb) || pg == 0.0);
      if (rot) {
        const double zeta = (pb - pa) / (2.0 * pg);
        const double t = (zeta >= 0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
        const double c = 1.0 / sqrt(1.0 + t * t), sn = c * t;
        if (r < n) {
          const double wi = W[r + n * i], wj = W[r + n * j];
          W[r + n * i] = c * wi - sn * wj;
          W[r + n * j] = sn * wi + c * wj;
          const double vi = V[r + n * i], vj = V[r + n * j];
          V[r + n * i] = c * vi - sn * vj;
          V[r + n * j] = sn * vi + c * vj;
        }
      }
      rotated = rotated || rot;
      wave_sync();
    }
    if (__ballot(rotated) == 0ull) break;
  }
}

// One wave: the last stage of the fixed-order reduction of the partial rows (row stride ld), then
// the polar factor of B (the n x n block of the sums after A), which is the new dictionary, with its
// compute-type copy and Gram matrix.  Newton's iteration gives it directly; where B is too far from
// well conditioned for that, one-sided Jacobi rotations (jacobi8; above eight columns lane x holds row x,
// pairs in cyclic row order as the oracle) give the singular vectors and values, D = U V^T, and a
// rank-deficient B leaves the dictionary unchanged and sets the singular status.
template <typename T>
__global__ void __launch_bounds__(kWave) procrustes_kernel(const double* __restrict__ src, int nrow, int ld, int n,
                                                           double* D, T* Dc, T* Gc, int* status,
                                                           unsigned long long* counters, RmseOut ro) {
  __shared__ double W[SDL_ORTHO_MAX_N * SDL_ORTHO_MAX_N];  // column-major n x n
  __shared__ double V[SDL_ORTHO_MAX_N * SDL_ORTHO_MAX_N];
  __shared__ double Dn[SDL_ORTHO_MAX_N * SDL_ORTHO_MAX_N];
  __shared__ double buf[64];
  __shared__ int perm[64];
  __shared__ double sig[SDL_ORTHO_MAX_N];
  const int x = threadIdx.x;
  const int nent = n * n;
  for (int e = x; e < nent; e += kWave) {
    // B follows A in the row; sixteen rows' loads in flight, added in row order
    double v = 0.0;
    int b = 0;
    for (; b + 16 <= nrow; b += 16) {
      double q[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) q[u] = src[(size_t)(b + u) * ld + nent + e];
#pragma unroll
      for (int u = 0; u < 16; ++u) v += q[u];
    }
    for (; b < nrow; ++b) v += src[(size_t)b * ld + nent + e];
    W[e] = v;
  }
  if (ro.trace) {
    // the RMSE of the sweep that wrote the rows, from their residual sums
    double v = 0.0;
    for (int b = x; b < nrow; b += kWave) v += src[(size_t)b * ld + ro.idx];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    if (x == 0) {
      const int it = *ro.counter;
      ro.trace[(size_t)it + ro.offset] = ro.denom > 0 ? sqrt(v / ro.denom) : 0.0;
      *ro.counter = it + 1;
    }
  }
  wave_sync();
  const bool row = x < n;
  const bool direct = n <= 8 ? polar_newton8(W, n) : polar_newton(W, V, Dn, buf, perm, n);
  if (!direct) {
    for (int e = x; e < nent; e += kWave) V[e] = (e % n) == (e / n) ? 1.0 : 0.0;
    wave_sync();
    if (n <= 8) jacobi8(W, V, n);
    for (int sweep = 0; n > 8 && sweep < 60; ++sweep) {
      int rotated = 0;
      for (int i = 0; i < n - 1; ++i)
        for (int j = i + 1; j < n; ++j) {
          double pa = 0.0, pb = 0.0, pg = 0.0;
          if (row) {
            const double wi = W[x + n * i], wj = W[x + n * j];
            pa = wi * wi;
            pb = wj * wj;
            pg = wi * wj;
          }
          // sums over the n <= 32 rows in a fixed order: each 16-lane row by DPP, then rows 0 and
          // 1 added from their first lanes (uniform values: every lane takes the same decision)
          pa = row16_sum(pa);
          pb = row16_sum(pb);
          pg = row16_sum(pg);
          pa = n > 16 ? lane_value(pa, 0) + lane_value(pa, 16) : lane_value(pa, 0);
          pb = n > 16 ? lane_value(pb, 0) + lane_value(pb, 16) : lane_value(pb, 0);
          pg = n > 16 ? lane_value(pg, 0) + lane_value(pg, 16) : lane_value(pg, 0);
          if (fabs(pg) <= 1e-15 * sqrt(pa * pb) || pg == 0.0) continue;
          rotated = 1;
          const double zeta = (pb - pa) / (2.0 * pg);
          const double t = (zeta >= 0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
          const double c = 1.0 / sqrt(1.0 + t * t), sn = c * t;
          if (row) {
            const double wi = W[x + n * i], wj = W[x + n * j];
            W[x + n * i] = c * wi - sn * wj;
            W[x + n * j] = sn * wi + c * wj;
            const double vi = V[x + n * i], vj = V[x + n * j];
            V[x + n * i] = c * vi - sn * vj;
            V[x + n * j] = sn * vi + c * vj;
          }
          wave_sync();
        }
      if (!rotated) break;
    }
    wave_sync();
    if (row) {
      double v = 0.0;
      for (int r = 0; r < n; ++r) v += W[r + n * x] * W[r + n * x];
      sig[x] = sqrt(v);
    }
    wave_sync();
    double smax = 0.0;
    for (int i = 0; i < n; ++i) smax = fmax(smax, sig[i]);
    bool ok = true;
    for (int i = 0; i < n; ++i) ok = ok && sig[i] > 1e-12 * smax;
    if (!ok) {
      if (x == 0) {
        atomicOr(status, kStatusSingular);
        atomicAdd(&counters[kCtrSingular], 1ull);
      }
      return;
    }
  }
  // D (D[r][c] = sum_i (W[r][i] / sigma_i) V[c][i] after the rotations) and its Gram matrix, one entry
  // per lane and pass
  wave_sync();
  if (!direct && row) sig[x] = 1.0 / sig[x];
  wave_sync();
  for (int e = x; e < nent; e += kWave) {
    const int r = e % n, c = e / n;
    double v = direct ? W[e] : 0.0;
    if (!direct)
#pragma unroll 4
      for (int i = 0; i < n; ++i) v += (W[r + n * i] * sig[i]) * V[c + n * i];
    Dn[e] = v;
    D[e] = v;
    Dc[e] = (T)v;
  }
  wave_sync();
  for (int e = x; e < nent; e += kWave) {
    const int i = e % n, c = e / n;
    double v = 0.0;
#pragma unroll 4
    for (int r = 0; r < n; ++r) v += Dn[r + n * i] * Dn[r + n * c];
    Gc[e] = (T)v;
  }
}

size_t ortho_lds(int m1, int m2, size_t elem) {
  const int M = m1 * m2;
  return elem * ((size_t)m1 * m1 + (size_t)m2 * m2 + 2 * (size_t)kOWaves * kOSigs * M + (size_t)kOWaves * kOSigs * 32) +
         4 * (size_t)kOWaves * kOSigs * 32;
}

}  // namespace

bool ortho_supported(int m1, int m2, int n1, int n2, int s) {
  return n1 == m1 && n2 == m2 && m1 <= SDL_ORTHO_MAX_N && m2 <= SDL_ORTHO_MAX_N && m1 * m2 <= kOLanes * kOMaxPer &&
         s <= 32 && s <= m1 * m2;
}

template <typename T>
hipError_t launch_ortho_code(const OmpArgs<T>& a, hipStream_t st) {
  if (a.N == 0) return hipSuccess;
  const int64_t ngroups = (a.N + kOSigs - 1) / kOSigs;
  int64_t blocks = (ngroups + kOWaves - 1) / kOWaves;
  if (blocks > kOMaxBlocks) blocks = kOMaxBlocks;
  hipLaunchKernelGGL(ortho_code_kernel<T>, dim3((unsigned)blocks), dim3(kWave * kOWaves), ortho_lds(a.m1, a.m2, sizeof(T)),
                     st, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_procrustes(const double* src, int nrow, int ld, int n, double* D, T* Dc, T* Gc,
                             int* status, unsigned long long* counters, const RmseOut& r, hipStream_t st) {
  hipLaunchKernelGGL(procrustes_kernel<T>, dim3(1), dim3(kWave), 0, st, src, nrow, ld, n, D, Dc, Gc, status,
                     counters, r);
  return hipGetLastError();
}

hipError_t ortho_init_device() {
  const int bytes = 160 * 1024;  // at most ortho_lds(32, 8, 8), about 75 KiB
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ortho_code_kernel<float>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&ortho_code_kernel<double>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template hipError_t launch_ortho_code<float>(const OmpArgs<float>&, hipStream_t);
template hipError_t launch_ortho_code<double>(const OmpArgs<double>&, hipStream_t);
template hipError_t launch_procrustes<float>(const double*, int, int, int, double*, float*, float*, int*,
                                             unsigned long long*, const RmseOut&, hipStream_t);
template hipError_t launch_procrustes<double>(const double*, int, int, int, double*, double*, double*, int*,
                                              unsigned long long*, const RmseOut&, hipStream_t);

}  // namespace sdl
