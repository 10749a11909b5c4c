// The instantiations of omp_group.h and the rule that picks one, included by the two translation
// units that compile them (omp_generic.hip: FP32, omp_generic_f64.hip: FP64).
#pragma once

#include "omp_group.h"

namespace sdl {
namespace {

constexpr size_t kLdsPerCu = 160 * 1024;
constexpr int kGroupMaxBlocks = 4096;

struct GroupVariant {
  int lanes;     // lanes per signal
  int nmax1, nmax2, smax, elems, maxw;
  size_t (*lds)(int m1, int m2, int n1, int n2, int s, int wpb);
  const void* kernel;
};

template <class C>
size_t lds_bytes(int m1, int m2, int n1, int n2, int s, int wpb) {
  const GLay l = group_layout<C>(m1, m2, n1, n2, s);
  return sizeof(typename C::T) * ((size_t)l.tab + (size_t)wpb * C::NS * l.stride + l.slack);
}

template <class C>
GroupVariant variant() {
  return GroupVariant{C::G, C::P1, C::P2, C::SM, C::E, C::MAXW, &lds_bytes<C>, reinterpret_cast<const void*>(&omp_group_kernel<C>)};
}

// Blocks of correlations per lane (RI x CJ).  Sixteen lanes per signal: up to 24 x 24 atoms and 16
// chosen atoms (larger blocks would leave one wave per SIMD); 64 lanes: everything else.
#define SDL_GROUP16(X) X(2, 2) X(2, 4) X(4, 2) X(3, 3) X(3, 4) X(4, 3) X(4, 4) X(4, 6) X(6, 4) X(6, 6)
#define SDL_GROUP64(X) \
  X(2, 2) X(2, 4) X(4, 2) X(2, 8) X(8, 2) X(4, 4) X(4, 6) X(6, 4) X(4, 8) X(8, 4) X(6, 6) X(8, 8)

// A 4 x 16 lane grid for a narrow dictionary against a wide one: FP64 n-dimensional problems whose
// later modes are collapsed into one Kronecker factor.
#define SDL_GROUP64W(X) X(3, 2) X(3, 3) X(3, 4) X(3, 5) X(4, 4) X(4, 6)

template <typename T>
const GroupVariant* variants(int* n) {
  if constexpr (sizeof(T) == 8) {
    static const GroupVariant v[] = {
#define X(R_, C_) variant<GCfg<T, 4, 4, R_, C_, 8>>(), variant<GCfg<T, 4, 4, R_, C_, 16>>(),
        SDL_GROUP16(X)
#undef X
#define X(R_, C_) variant<GCfg<T, 8, 8, R_, C_, 32>>(),
        SDL_GROUP64(X)
#undef X
#define X(R_, C_) variant<GCfg<T, 4, 16, R_, C_, 32>>(),
        SDL_GROUP64W(X)
#undef X
    };
    *n = (int)(sizeof(v) / sizeof(v[0]));
    return v;
  }
  static const GroupVariant v[] = {
#define X(R_, C_) variant<GCfg<T, 4, 4, R_, C_, 8>>(), variant<GCfg<T, 4, 4, R_, C_, 16>>(),
      SDL_GROUP16(X)
#undef X
#define X(R_, C_) variant<GCfg<T, 8, 8, R_, C_, 32>>(),
      SDL_GROUP64(X)
#undef X
  };
  *n = (int)(sizeof(v) / sizeof(v[0]));
  return v;
}

// The variant of a shape: sixteen lanes per signal before 64, then the smallest block that covers
// the atoms, then the shortest unrolled support.
template <typename T>
const GroupVariant* pick(int m1, int m2, int n1, int n2, int s) {
  int n = 0;
  const GroupVariant* v = variants<T>(&n);
  const GroupVariant* best = nullptr;
  for (int i = 0; i < n; ++i) {
    if (n1 > v[i].nmax1 || n2 > v[i].nmax2 || s > v[i].smax) continue;
    if (v[i].lds(m1, m2, n1, n2, s, 1) > kLdsPerCu) continue;
    if (!best || v[i].lanes < best->lanes ||
        (v[i].lanes == best->lanes && (v[i].elems < best->elems || (v[i].elems == best->elems && v[i].smax < best->smax))))
      best = &v[i];
  }
  return best;
}

template <typename T>
hipError_t group_launch(const OmpArgs<T>& a, hipStream_t st) {
  if (a.N == 0) return hipSuccess;
  const GroupVariant* v = pick<T>(a.m1, a.m2, a.n1, a.n2, a.s);
  if (!v) return hipErrorInvalidValue;
  const int ns = kWave / v->lanes;
  const int64_t waves = (a.N + ns - 1) / ns;
  // waves per workgroup: the most waves per CU that LDS and registers allow, the waves of a workgroup
  // sharing one copy of the tables (8x32 signals with 12x72 atoms in FP64, 62 KB of tables: 310 us
  // with eight, 229 us with sixteen for 20,000 signals), four where that is no worse.  Few signals spread
  // over the CUs, a workgroup each, whose waves still load the tables together (a call of one signal
  // 6x6x2 with 12x16x6 atoms in FP64, 85 KB of tables: 57 us with one wave a workgroup, 24 us so)
  int wpb = 1, best = 0;
  for (int w = 1; w <= v->maxw; w *= 2) {
    const size_t lds = v->lds(a.m1, a.m2, a.n1, a.n2, a.s, w);
    if (lds > kLdsPerCu) break;
    int on = (int)(kLdsPerCu / lds) * w;
    if (on > v->maxw) on = v->maxw;
    if (on > best || (on == best && w <= 4)) {
      best = on;
      wpb = w;
    }
  }
  int64_t grid = (waves + wpb - 1) / wpb;
  if (grid < 256) grid = waves < 256 ? waves : 256;
  if (grid > kGroupMaxBlocks) grid = kGroupMaxBlocks;
  OmpArgs<T> args = a;
  void* p[] = {&args};
  return hipLaunchKernel(v->kernel, dim3((unsigned)grid), dim3(kWave * wpb), p,
                         v->lds(a.m1, a.m2, a.n1, a.n2, a.s, wpb), st);
}

template <typename T>
hipError_t group_allow_lds() {
  // allow the dynamic LDS of large shapes (up to the 160 KiB of a gfx950 CU)
  int n = 0;
  const GroupVariant* v = variants<T>(&n);
  for (int i = 0; i < n; ++i) {
    const hipError_t e = hipFuncSetAttribute(v[i].kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace
}  // namespace sdl
