// 2D-OMP sparse coding for any shape: the kernel template.
//
// Method (Sec. III step 1; Sec. II: 2D-OMP is OMP on D2 (x) D1 without forming it): for s steps,
// choose the unselected atom a = i + n1*j with the largest |corr_a| (ties: smallest a), then
// re-fit all chosen coefficients by least squares.  The least squares is carried by an
// incrementally grown Cholesky factor L of the support's Gram matrix, whose entries are
// G1[i,i'] * G2[j,j'] with G1 = D1^T D1, G2 = D2^T D2 (the Gram identity stated after
// Algorithm 1).  Correlations are kept in Gram form: corr starts as C = D1^T Y D2 and, when atom a
// joins with new Cholesky row [w^T, delta] (L w = G_{S,a}, delta^2 = G_aa - |w|^2),
//     corr <- corr - (corr_a / delta^2) * (G_{:,a} - G_{:,S} v),   v = L^{-T} w,
//     x_S  <- x_S  - (corr_a / delta^2) * v,   x_a = corr_a / delta^2.
// The residual and its squared norm are formed explicitly at the end.
//
// Mapping: LR x LC = G lanes share a signal (16: four signals per wave; 64: one).  Lane (sr, sc)
// keeps the correlations of the RI x CJ block of atoms i = sr RI + ri, j = sc CJ + cj in registers,
// so a refresh term v_q G1[:, i_q] G2[j_q, :] is RI + CJ contiguous LDS reads and RI CJ multiply-adds
// with no index arithmetic (n1 <= LR RI and n2 <= LC CJ: elements beyond n1, n2 read whatever follows
// in LDS and are NaN from the start, which never compares as the largest).  Lane k of the signal
// holds support element k: its atom, its coefficient and, while a step runs, its entries of w and v;
// they reach the other lanes by DPP row broadcasts (G = 16) or lane reads (G = 64), so the triangular
// solves are a column at a time over the lanes instead of every lane running both serially.
//
// What bounds it: the issue of vector-ALU instructions (the step loop's compares and multiply-adds)
// with the LDS reads of the refresh close behind; four signals per wave share every instruction of
// the serial parts of a step (argmax merge, solves), which is why 16 lanes take a signal wherever its
// block of correlations fits their registers.  Vector ALUs busy 83% of the time in FP64, 99% in FP32
// (100,000 signals 8x8, 16x16 atoms, s = 8).  Against the earlier form
// of this path (one wave per signal, correlations in LDS, an integer division per element and term):
// 100,000 FP64 signals 8x8, 16x16 atoms, s = 8: 1676 -> 154 us; 20,011 FP32 signals 9x7, 13x11 atoms,
// s = 6: 147 -> 28 us; 20,000 FP64 signals 8x32, 12x72 atoms, s = 8 (three modes before): 1630 -> 225 us.
//
// FP32 runs exactly the operations of that earlier form in its order, element by element (each
// multiply-add fused or not as written below), so FP32 codes are the same bit for bit; FP64
// keeps L^{-1} instead of L (w = L^{-1} g and v = L^{-T} w are then products with no chain from one
// entry to the next) and folds the step's coefficient into the refresh terms.
#pragma once

#include "lanes.h"
#include "sdl_internal.h"

namespace sdl {
namespace {

template <typename T_, int LR_, int LC_, int RI_, int CJ_, int SM_>
struct GCfg {
  using T = T_;
  static constexpr int LR = LR_, LC = LC_, RI = RI_, CJ = CJ_, SM = SM_;
  static constexpr int G = LR * LC, NS = kWave / G, E = RI * CJ, P1 = LR * RI, P2 = LC * CJ;
  // waves per SIMD the registers must allow
  static constexpr int WPE = E <= 16 ? 4 : 2;
  static constexpr int MAXW = 4 * WPE;  // waves per workgroup, at most what a CU's registers hold
  // table rows start on the boundary that a lane's run of RI (CJ) elements is read at
  __host__ __device__ static constexpr int run_align(int n) {
    const int b = n * (int)sizeof(T);
    return (b % 16 == 0 ? 16 : b % 8 == 0 ? 8 : 4) / (int)sizeof(T);
  }
  __host__ __device__ static constexpr int ld1(int n1) { return (n1 + run_align(RI) - 1) / run_align(RI) * run_align(RI); }
  __host__ __device__ static constexpr int ld2(int n2) { return (n2 + run_align(CJ) - 1) / run_align(CJ) * run_align(CJ); }
  static_assert(G == 16 || G == 64, "a signal takes a DPP row or a wave");
  static_assert(SM <= G && SM <= SDL_MAX_S, "support element k lives in lane k of the signal");
};

// LDS of one workgroup of wpb waves, in elements of T: the tables, then per signal its pixels and
// the space shared by W (first correlation) and L (step loop)
struct GLay {
  int d1, d2, g1, g2, tab, lds, stride;  // lds: offset of W / L inside a signal's space
  int ld1, ld2, ldd;                     // strides of G1 and W, of G2 and D2, of D1 (odd)
  int slack;                             // elements a run of the last row may read past the end
};
template <class C>
__host__ __device__ inline GLay group_layout(int m1, int m2, int n1, int n2, int s) {
  GLay l;
  auto up4 = [](int v) { return (v + 3) & ~3; };
  l.ld1 = C::ld1(n1);
  l.ld2 = C::ld2(n2);
  l.ldd = m1 | 1;
  l.slack = C::P1 > C::P2 ? C::P1 : C::P2;
  int o = 0;
  l.d2 = o; o += up4(m2 * l.ld2);
  l.g1 = o; o += up4(n1 * l.ld1);
  l.g2 = o; o += up4(n2 * l.ld2);
  l.d1 = o; o += up4(n1 * l.ldd);
  l.tab = o;
  l.lds = up4(m1 * m2);
  const int w = m2 * l.ld1, f = s * (s | 1);
  // signals of a wave sit 4 elements (mod 16) apart, so their broadcast reads hit different banks
  const int e = l.lds + up4(w > f ? w : f);
  l.stride = C::NS == 1 ? e : (e + 11) / 16 * 16 + 4;
  return l;
}

__device__ inline float gfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double gfma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ inline float gabs(float a) { return __builtin_fabsf(a); }
__device__ inline double gabs(double a) { return __builtin_fabs(a); }

__device__ inline void group_sync() {  // LDS written by this wave is visible to all its lanes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// calls f(integral_constant l) or f(int l) for l = l0 .. n-1 in order: compile-time indices where a
// lane broadcast needs them (G = 16), a runtime loop otherwise.  n is uniform over the wave.
template <int V>
struct IntC {
  static constexpr int value = V;
  __device__ constexpr operator int() const { return V; }
};
template <int L, int SM, class F>
__device__ __forceinline__ void upward_static(int n, F&& f) {
  if constexpr (L < SM) {
    if (L < n) {
      f(IntC<L>{});
      upward_static<L + 1, SM>(n, f);
    }
  }
}
template <int L, class F>
__device__ __forceinline__ void downward_static(int n, F&& f) {
  if constexpr (L >= 0) {
    if (L < n) f(IntC<L>{});
    downward_static<L - 1>(n, f);
  }
}
template <class C, class F>
__device__ __forceinline__ void upward(int n, F&& f) {
  if constexpr (C::G == 16) {
    upward_static<0, C::SM>(n, f);
  } else {
#pragma unroll 1
    for (int l = 0; l < n; ++l) f(l);
  }
}
template <class C, class F>
__device__ __forceinline__ void downward(int n, F&& f) {
  if constexpr (C::G == 16) {
    downward_static<C::SM - 1>(n, f);
  } else {
#pragma unroll 1
    for (int l = n - 1; l >= 0; --l) f(l);
  }
}
// lane l's value of v, within each signal's lanes
template <class C, class L, typename U>
__device__ inline U from_lane(U v, L l) {
  if constexpr (C::G == 16) {
    return bcast16<L::value>(v);
  } else {
    return lane_read(v, l);
  }
}

// the sum over a signal's lanes, in the order of a 64-lane butterfly over elements e mod 64
// (G = 16: c[u] holds the partial sum of the elements with (e / 16) mod 4 = u)
template <class C, typename T>
__device__ inline T signal_sum(const T* c) {
#pragma clang fp contract(off)
  if constexpr (C::G == 16) {
    T v = (c[0] + c[2]) + (c[1] + c[3]);
    v = v + dpp<0x128>(v, v);  // row_ror:8
    v = v + dpp<0x124>(v, v);  // row_ror:4
    v = v + dpp<0x4E>(v, v);   // quad_perm [2,3,0,1]
    return v + dpp<0xB1>(v, v);
  } else {
    T v = c[0];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = v + __shfl_xor(v, o, kWave);
    return v;
  }
}

// (signed value, code) of the largest magnitude over a signal's lanes, ties to the smaller code
template <int CTRL, int ROWS, typename T>
__device__ inline void argmax_merge(T& v, int& code) {
  const T ov = dpp<CTRL, ROWS>(v, v);
  const int oc = dpp32<CTRL, ROWS>(code, code);
  const bool take = gabs(ov) > gabs(v) || (gabs(ov) == gabs(v) && oc < code);
  v = take ? ov : v;
  code = take ? oc : code;
}
template <class C, typename T>
__device__ inline void signal_argmax(T& v, int& code) {
  argmax_merge<0xB1, 0xF>(v, code);   // quad_perm [1,0,3,2]
  argmax_merge<0x4E, 0xF>(v, code);   // quad_perm [2,3,0,1]
  argmax_merge<0x141, 0xF>(v, code);  // row_half_mirror
  argmax_merge<0x140, 0xF>(v, code);  // row_mirror
  if constexpr (C::G == 64) {
    argmax_merge<0x142, 0xA>(v, code);  // row_bcast:15 into rows 1 and 3
    argmax_merge<0x143, 0xC>(v, code);  // row_bcast:31 into rows 2 and 3
    v = lane_read(v, 63);
    code = __builtin_amdgcn_readlane(code, 63);
  }
}

// N contiguous elements of a table row; the run starts on the widest boundary its size allows
template <int N, typename T>
__device__ inline void load_run(const T* p, T* out) {
  constexpr int bytes = N * (int)sizeof(T), W = (bytes % 16 == 0 ? 16 : bytes % 8 == 0 ? 8 : 4) / (int)sizeof(T);
  if constexpr (W <= 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = p[i];
  } else {
    typedef T V __attribute__((ext_vector_type(W)));
#pragma unroll
    for (int i = 0; i < N; i += W) {
      const V v = *reinterpret_cast<const V*>(p + i);
#pragma unroll
      for (int u = 0; u < W; ++u) out[i + u] = v[u];
    }
  }
}

// 1 / sqrt(x) of a positive normal x: the hardware's estimate (relative error below 2^-22) and one
// third-order correction y (1 + e/2 + 3 e^2/8), e = 1 - x y^2
__device__ inline double rsqrt64(double x) {
  const double y = __builtin_amdgcn_rsq(x), e = gfma(-(x * y), y, 1.0);
  return gfma(y * e, gfma(0.375, e, 0.5), y);
}
__device__ inline float rsqrt64(float x) { return x; }  // never called

template <class C>
__global__ void __launch_bounds__(kWave* C::MAXW) __attribute__((amdgpu_waves_per_eu(C::WPE)))
    omp_group_kernel(OmpArgs<typename C::T> a) {
#pragma clang fp contract(off)
  using T = typename C::T;
  constexpr int RI = C::RI, CJ = C::CJ, E = C::E, P1 = C::P1, P2 = C::P2, G = C::G, NS = C::NS;
  constexpr bool F64 = sizeof(T) == 8;
  // Where a signal stops that has no correlation above the threshold: inside the search, or after it where
  // that compiles to less (20,000 FP64 signals 16x8, 64x33 atoms, s = 20: 1,434 against 1,553 us; the 4 x 16 grid
  // 231 against 224 us a sweep of 20,000 signals, 12x72 atoms)
  constexpr bool STOP_FIRST = !(F64 && C::LR == 8);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int m1 = a.m1, m2 = a.m2, n1 = a.n1, n2 = a.n2, s = a.s, M = m1 * m2;
  const GLay lay = group_layout<C>(m1, m2, n1, n2, s);
  const int ld1 = lay.ld1, ld2 = lay.ld2, ldd = lay.ldd;
  T* sD1 = sm + lay.d1;  // D1[p, i] at i ldd + p
  T* sD2 = sm + lay.d2;  // D2[q, j] at q ld2 + j
  T* sG1 = sm + lay.g1;  // G1[i, i'] at i' ld1 + i
  T* sG2 = sm + lay.g2;  // G2[j, j'] at j' ld2 + j
  const int tid = threadIdx.x, wv = tid / kWave, lane = tid % kWave, wpb = blockDim.x / kWave;
  for (int e = tid; e < m1 * n1; e += blockDim.x) sD1[(e / m1) * ldd + e % m1] = a.D1[e];
  for (int e = tid; e < m2 * n2; e += blockDim.x) sD2[(e % m2) * ld2 + e / m2] = a.D2[e];
  for (int e = tid; e < n1 * n1; e += blockDim.x) sG1[(e / n1) * ld1 + e % n1] = a.G1[e];
  for (int e = tid; e < n2 * n2; e += blockDim.x) sG2[(e / n2) * ld2 + e % n2] = a.G2[e];
  __syncthreads();

  const int g = lane / G, l = lane % G, sr = l % C::LR, sc = l / C::LR;
  const unsigned long long gmask = G == 64 ? ~0ull : ((1ull << (G % 64)) - 1ull) << (g * G);
  T* ys = sm + lay.tab + (size_t)(wv * NS + g) * lay.stride;
  T* Ws = ys + lay.lds;  // W[i, q] at q ld1 + i
  T* Lr = Ws;            // L[k, q] (FP64: L^{-1}[k, q]), q <= k, at k ldl + q (after W is read)
  const int ldl = s | 1;
  const int ls = l < s ? l : 0;  // a row / column of L that exists
  const T* rG1 = sG1 + sr * RI;  // this lane's rows and columns of the tables
  const T* rG2 = sG2 + sc * CJ;
  const int base_code = (sc * CJ) << 8 | (sr * RI);  // codes j << 8 | i order like the atoms i + n1 j
  const unsigned inv_m1 = ((1u << 20) + (unsigned)m1 - 1u) / (unsigned)m1;  // e / m1 for e < 4096

  unsigned n_early = 0;  // early-stopped signals (first lane of each signal), added up at the end
  // few signals: every workgroup gets one wave's before any gets a second (the others only load tables)
  const bool few = a.N <= (int64_t)gridDim.x * (wpb - 1) * NS;
  const int wu = __builtin_amdgcn_readfirstlane(wv);
  const int64_t w0 = few ? (int64_t)wu * gridDim.x + blockIdx.x : (int64_t)blockIdx.x * wpb + wu;
  for (int64_t k0 = w0 * NS; k0 < a.N; k0 += (int64_t)gridDim.x * wpb * NS) {
    const int64_t k = k0 + g;
    const bool valid = k < a.N;
    T part[4] = {0, 0, 0, 0};
    for (int e0 = 0; e0 < M; e0 += kWave) {
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int e = e0 + G * u + l;
        if (e < M) {
          T v = 0;
          if (valid) {
            if constexpr (F64) v = a.Y[k * M + e];
            else v = a.Yh ? (T)bf16_to_float(a.Yh[k * M + e]) : a.Y[k * M + e];
          }
          ys[e] = v;
          part[u] = gfma(v, v, part[u]);
        }
      }
    }
    const T yy = signal_sum<C>(part);
    const T ynorm = sqrt(yy);
    T renergy = yy;  // ||r||^2 by the recurrence ||r||^2 -= corr_a^2 / pivot per appended atom
    group_sync();
    // C = D1^T Y D2, as W = D1^T Y (n1 x m2; lanes over rows, four columns at a time) then W D2
    {
      constexpr int QI = P1 < G ? G / P1 : 1;  // columns handled side by side
      const int i0 = l % (P1 < G ? P1 : G), qo = P1 < G ? l / P1 : 0;
      if (qo < QI) {
        for (int i = i0; i < n1; i += G) {
          const T* d1 = sD1 + i * ldd;
          for (int q0 = qo; q0 < m2; q0 += 4 * QI) {
            T v[4] = {0, 0, 0, 0};
            const T* y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int q = q0 + u * QI;
              y[u] = ys + m1 * (q < m2 ? q : m2 - 1);
            }
#pragma unroll 4
            for (int p = 0; p < m1; ++p) {
              const T d = d1[p];
#pragma unroll
              for (int u = 0; u < 4; ++u) v[u] = gfma(d, y[u][p], v[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (q0 + u * QI < m2) Ws[(q0 + u * QI) * ld1 + i] = v[u];
          }
        }
      }
    }
    group_sync();
    T al[E];
#pragma unroll
    for (int e = 0; e < E; ++e) al[e] = 0;
#pragma unroll 2
    for (int q = 0; q < m2; ++q) {
      T wi[RI], dj[CJ];
      load_run<RI>(Ws + q * ld1 + sr * RI, wi);
      load_run<CJ>(sD2 + q * ld2 + sc * CJ, dj);
#pragma unroll
      for (int cj = 0; cj < CJ; ++cj)
#pragma unroll
        for (int ri = 0; ri < RI; ++ri) al[cj * RI + ri] = gfma(wi[ri], dj[cj], al[cj * RI + ri]);
    }
    // opaque copies: the compares stay here instead of living in scalar registers throughout
    int rows = n1 - sr * RI, cols = n2 - sc * CJ;
    asm volatile("" : "+v"(rows), "+v"(cols));
#pragma unroll
    for (int e = 0; e < E; ++e) al[e] = e % RI < rows && e / RI < cols ? al[e] : T(__builtin_nanf(""));
    group_sync();  // W is read: L takes its place
    if constexpr (F64) {
      for (int e = l; e < s * ldl; e += G) Lr[e] = 0;
      group_sync();
    }

    const T thr = T(a.stop_rel) * ynorm;
    bool active = valid, early = false;
    int nt = 0;                     // atoms of this signal
    int my_code = -1, my_off = 0;   // support element l: its code, its rows of G1 and G2
    T my_x = 0, my_d = 1;           // its coefficient; L[l, l] (FP32)
    int t = 0;
#pragma unroll 1
    for (; t < s; ++t) {
      // error-driven stop (denoising runs, Sec. IV): no further atom once ||r||^2 <= err2
      if (a.err2 > 0.0) {
        const bool stop = active && !(renergy > T(a.err2));
        early |= stop;
        active = active && !stop;
      }
      T bs;
      int code;
      // At most two passes: a signal that goes on has a value above the threshold (at least 0), so an
      // element was found, and once its support is masked no element found is in it.  The threshold
      // has to come before the repeat: where every correlation left is exactly zero (a signal that fewer
      // than s atoms represent exactly) the merge gives value 0 and code 0, masked or not.
      for (;;) {
        bs = 0;
        int be = 0;
        // a lane's elements in (cj, ri) order have increasing codes: a strict comparison keeps the
        // first of equal values; NaN (a masked element) never compares larger
#pragma unroll
        for (int cj = 0; cj < CJ; ++cj)
#pragma unroll
          for (int ri = 0; ri < RI; ++ri) {
            const T v = al[cj * RI + ri];
            const bool take = gabs(v) > gabs(bs);
            bs = take ? v : bs;
            be = take ? cj * RI + ri : be;
          }
        code = base_code + ((be / RI) << 8 | (be % RI));
        signal_argmax<C>(bs, code);
        const bool above = gabs(bs) > thr;
        if constexpr (STOP_FIRST) {
          early |= active && !above;
          active = active && above;
        }
        // a chosen atom's correlation is zero up to rounding after the re-fit, so it comes up
        // again only when every correlation is at rounding level: only then is the support masked
        const bool again = active && above && ((__ballot(l < t && my_code == code) & gmask) != 0ull);
        if (__ballot(again) == 0ull) break;
#pragma unroll 1
        for (int q = 0; q < t; ++q) {
          const int cq = __shfl(my_code, g * G + q, kWave) - base_code;
#pragma unroll
          for (int e = 0; e < E; ++e) al[e] = again && ((e / RI) << 8 | (e % RI)) == cq ? T(__builtin_nanf("")) : al[e];
        }
      }
      if constexpr (!STOP_FIRST) {
        const bool above = gabs(bs) > thr;
        early |= active && !above;
        active = active && above;
      }
      if (__ballot(active) == 0ull) break;
      const int ia = code & 255, ja = code >> 8;
      const int off_a = (ia * ld1) | (ja * ld2) << 16;
      const T* g1a = sG1 + ia * ld1;
      const T* g2a = sG2 + ja * ld2;
      const T a1 = g1a[ia], a2 = g2a[ja];
      const T gaa = a1 * a2;
      // new Cholesky row: L w = G_{S,a}, lane k < t holding entry k (a signal that stopped before the
      // others of its wave has fewer than t atoms: its other lanes read atom 0's entry, which is not used)
      const int mc = l < t && (G == kWave || my_code >= 0) ? my_code : 0;
      T b = g1a[mc & 255] * g2a[mc >> 8], w = 0, ww = 0, v = 0;
      if constexpr (F64) {
        upward<C>(t, [&](auto q) __attribute__((always_inline)) { w = gfma(Lr[ls * ldl + q], from_lane<C>(b, q), w); });
        w = l < t ? w : T(0);
        // and v = L^{-T} w (rows and columns of L^{-1} not yet written are zero)
        upward<C>(t, [&](auto q) __attribute__((always_inline)) {
          const T wq = from_lane<C>(w, q);
          ww = gfma(wq, wq, ww);
          v = gfma(Lr[q * ldl + ls], wq, v);
        });
      } else {
        upward<C>(t, [&](auto q) __attribute__((always_inline)) {
          const T wq = from_lane<C>(b / my_d, q);
          ww = gfma(wq, wq, ww);
          w = l == q ? wq : w;
          const T nb = gfma(-Lr[ls * ldl + q], wq, b);
          b = l > q && l < t ? nb : b;
        });
      }
      T d2 = gfma(a1, a2, -ww);
      if constexpr (!F64) {
        const bool small = active && d2 < T(a.pivot_fp64) * gaa;
        if (__ballot(small) != 0ull) {
          // small pivot: this row again in FP64 (cancellation in G_aa - |w|^2)
          double b64 = (double)g1a[mc & 255] * (double)g2a[mc >> 8], w64 = 0.0, acc = 0.0;
          upward<C>(t, [&](auto q) __attribute__((always_inline)) {
            const double wq = from_lane<C>(b64 / (double)my_d, q);
            acc = gfma(wq, wq, acc);
            w64 = l == q ? wq : w64;
            const double nb = gfma(-(double)Lr[ls * ldl + q], wq, b64);
            b64 = l > q && l < t ? nb : b64;
          });
          w = small ? (T)w64 : w;
          d2 = small ? (T)((double)gaa - acc) : d2;
          if (small && l == 0) atomicAdd(&a.counters[kCtrFp64Pivot], 1ull);
        }
      }
      const bool dep = !(d2 > T(a.dep_eps) * gaa);
      early |= active && dep;
      active = active && !dep;
      if (__ballot(active) == 0ull) break;
      T cst;
      if constexpr (F64) {
        const T r = rsqrt64(d2);
        cst = bs * (r * r);
        if (active) {
          if (l < t) Lr[t * ldl + l] = -(v * r);
          if (l == t) Lr[t * ldl + l] = r;
        }
      } else {
        // v = L^{-T} w, lane k < t holding entry k.  Entry q subtracts its products in increasing
        // order of the row, so it starts once entry q + 1 is known: a serial chain (every lane
        // computes it)
        downward<C>(t, [&](auto q) __attribute__((always_inline)) {
          T acc = from_lane<C>(w, q);
          upward<C>(t, [&](auto r) __attribute__((always_inline)) {
            if (r > q) acc = gfma(-Lr[r * ldl + q], from_lane<C>(v, r), acc);
          });
          acc = acc / from_lane<C>(my_d, q);
          v = l == q ? acc : v;
        });
        cst = bs / d2;
        const T dl = sqrt(d2);
        if (active) {
          if (l < t) Lr[t * ldl + l] = w;
          if (l == t) my_d = dl;
        }
      }
      renergy = gfma(-cst, bs, renergy);
      if (active) {
        if (l < t) my_x = gfma(-cst, v, my_x);
        if (l == t) {
          my_x = cst;
          my_code = code;
          my_off = off_a;
        }
        nt = t + 1;
      }
      if (t + 1 < s) {
        T u[RI], h[CJ];
        load_run<RI>(rG1 + ia * ld1, u);
        load_run<CJ>(rG2 + ja * ld2, h);
        if constexpr (F64) {
          // corr += sum_q gamma_q G1[:, i_q] G2[j_q, :], gamma = c v_q, and -c for the new atom
#pragma unroll
          for (int ri = 0; ri < RI; ++ri) u[ri] *= -cst;
#pragma unroll
          for (int e = 0; e < E; ++e) al[e] = gfma(u[e % RI], h[e / RI], al[e]);
          const T gam = cst * v;
          upward<C>(t, [&](auto q) __attribute__((always_inline)) {
            const T gq = from_lane<C>(gam, q);
            const int o = from_lane<C>(my_off, q);
            load_run<RI>(rG1 + (o & 0xFFFF), u);
            load_run<CJ>(rG2 + (o >> 16), h);
#pragma unroll
            for (int ri = 0; ri < RI; ++ri) u[ri] *= gq;
#pragma unroll
            for (int e = 0; e < E; ++e) al[e] = gfma(u[e % RI], h[e / RI], al[e]);
          });
        } else {
          // corr -= c (G_{:,a} - sum_q v_q G1[:, i_q] G2[j_q, :])
          T gr[E];
#pragma unroll
          for (int e = 0; e < E; ++e) gr[e] = u[e % RI] * h[e / RI];
          upward<C>(t, [&](auto q) __attribute__((always_inline)) {
            const T vq = from_lane<C>(v, q);
            const int o = from_lane<C>(my_off, q);
            load_run<RI>(rG1 + (o & 0xFFFF), u);
            load_run<CJ>(rG2 + (o >> 16), h);
#pragma unroll
            for (int ri = 0; ri < RI; ++ri) u[ri] = vq * u[ri];
#pragma unroll
            for (int e = 0; e < E; ++e) gr[e] = gfma(-u[e % RI], h[e / RI], gr[e]);
          });
#pragma unroll
          for (int e = 0; e < E; ++e) al[e] = gfma(-cst, gr[e], al[e]);
        }
      }
      group_sync();  // the new row of L is visible
    }
    // explicit residual Y - sum_q x_q d1_{i_q} d2_{j_q}^T.  Beyond a signal's atoms x_q = 0 with the signal's
    // first atom, which was chosen and so is finite (atom 0 may hold NaN); a signal without atoms keeps Y.
    const int first = from_lane<C>(my_code, IntC<0>{}), mc0 = my_code < 0 ? first : my_code;
    const int mi = mc0 < 0 ? 0 : mc0 & 255, mj = mc0 < 0 ? 0 : mc0 >> 8;
    const int my_pix = mi * ldd | (mj << 16);
    const bool bare = __ballot(valid && nt == 0) != 0ull;
    T rp[4] = {0, 0, 0, 0};
    for (int e0 = 0; e0 < M; e0 += kWave) {
      T r[NS];
      int p1[NS], p2[NS];
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int e = e0 + G * u + l < M ? e0 + G * u + l : M - 1;
        const int q = (int)(((unsigned)e * inv_m1) >> 20);
        p1[u] = e - q * m1;
        p2[u] = q * ld2;
        r[u] = ys[e];
      }
      upward<C>(t < s ? t + 1 : s, [&](auto q) __attribute__((always_inline)) {
        const T x = from_lane<C>(my_x, q);
        const int o = from_lane<C>(my_pix, q);
#pragma unroll
        for (int u = 0; u < NS; ++u)
          r[u] = gfma(-(x * sD1[p1[u] + (o & 0xFFFF)]), sD2[p2[u] + (o >> 16)], r[u]);
      });
      if (bare) {
#pragma unroll
        for (int u = 0; u < NS; ++u)
          if (nt == 0) r[u] = ys[e0 + G * u + l < M ? e0 + G * u + l : M - 1];
      }
#pragma unroll
      for (int u = 0; u < NS; ++u)
        if (e0 + G * u + l < M) rp[u] = gfma(r[u], r[u], rp[u]);
    }
    const T rr = signal_sum<C>(rp);
    if (valid) {
      if (l < s) {
        a.supp[k * s + l] = l < nt ? (my_code & 255) + n1 * (my_code >> 8) : -1;
        a.coef[k * s + l] = l < nt ? my_x : T(0);
      }
      if (l == 0) {
        if (a.res2) a.res2[k] = rr;
        n_early += early ? 1u : 0u;
      }
    }
    group_sync();
  }
  // one atomic per workgroup: atomics on one address from every wave serialise
  __syncthreads();
  unsigned* cnt = reinterpret_cast<unsigned*>(smem_raw);
  if (tid == 0) *cnt = 0;
  __syncthreads();
  if (n_early) atomicAdd(cnt, n_early);
  __syncthreads();
  if (tid == 0 && *cnt) atomicAdd(&a.counters[kCtrEarlyStop], (unsigned long long)*cnt);
}

}  // namespace
}  // namespace sdl
