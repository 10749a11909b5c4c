// Learned support proposal: the kernels of a small MLP (vec(Y)/||Y|| -> hidden ->
// hidden -> one logit per atom) and of the proposal step that turns its logits into
// a code.  Not a step of the paper's method: a learned front end whose output is
// only accepted when its least-squares residual passes a calibrated test, 2D-OMP
// (Sec. III step 1) being the fallback.
//
// GEMMs run on the matrix cores: 16x16x32 BF16 MFMA with FP32 accumulation
// (lane l supplies A[l%16][8(l/16)..8(l/16)+7] and B[8(l/16)..+7][l%16]; result v of
// lane l is D[4(l/16)+v][l%16]), or 16x16x4 FP32 MFMA in the FP32 check mode.
// FP32: workgroup tile 64x64x32 staged through LDS in K-contiguous layout, four waves of 32x32 (all
// operand layouts).  BF16: inference in one kernel (mlp_forward_kernel), training-sized GEMMs in
// batches of 64x64 tiles (gemm_tile_kernel), layers over many signals in 128x128 tiles
// (gemm_nt_bf16_kernel: training batches of 8,192 and more, networks wider than 512 units).
// Epilogues are fused: bias + exact-erf GELU (keeping the pre-activation for the backward pass),
// multiplication by GELU'(z) when back-propagating, FP32 store.
#include <hip/hip_bf16.h>
#include <math.h>

#include "mlp_internal.h"

namespace sdl {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int BM = 64, BN = 64, BK = 32, KP = BK + 8;  // LDS row length (16-byte aligned, bank spread)

template <typename T>
__device__ inline T from_float(float x);
template <>
__device__ inline float from_float<float>(float x) { return x; }
template <>
__device__ inline __bf16 from_float<__bf16>(float x) { return (__bf16)x; }

__device__ inline float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ inline float gelu_grad(float z) {
  // d/dz [z Phi(z)] = Phi(z) + z phi(z)
  const float cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752f));
  const float pdf = 0.39894228040143268f * expf(-0.5f * z * z);
  return cdf + z * pdf;
}

// A(M x K), B(K x N): opA 0 = row-major A[m*lda+k], 1 = stored transposed A[k*lda+m];
// opB 0 = row-major B[k*ldb+n], 1 = stored transposed B[n*ldb+k].
template <int OPA, int OPB>
__global__ void __launch_bounds__(256) gemm_kernel(GemmArgs g) {
  using T = float;
  __shared__ __align__(16) T As[BM][KP];
  __shared__ __align__(16) T Bs[BN][KP];
  const T* A = static_cast<const T*>(g.A);
  const T* B = static_cast<const T*>(g.B);
  const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int wm = (w / 2) * 32, wn = (w % 2) * 32;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int k0 = 0; k0 < g.K; k0 += BK) {
    // stage A tile -> As[m][k], B tile -> Bs[n][k]  (BM*BK = 2048 elements, 8 per thread)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = tid + 256 * u;
      if (OPA == 0) {
        const int m = e / BK, k = e % BK;
        As[m][k] = A[(size_t)(m0 + m) * g.lda + k0 + k];
      } else {
        const int k = e / BM, m = e % BM;
        As[m][k] = A[(size_t)(k0 + k) * g.lda + m0 + m];
      }
      if (OPB == 0) {
        const int k = e / BN, n = e % BN;
        Bs[n][k] = B[(size_t)(k0 + k) * g.ldb + n0 + n];
      } else {
        const int n = e / BK, k = e % BK;
        Bs[n][k] = B[(size_t)(n0 + n) * g.ldb + k0 + k];
      }
    }
    __syncthreads();
    const int r16 = lane % 16, kq = lane / 16;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      float af[2], bfr[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) af[i] = (float)As[wm + 16 * i + r16][kk + kq];
#pragma unroll
      for (int j = 0; j < 2; ++j) bfr[j] = (float)Bs[wn + 16 * j + r16][kk + kq];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  // epilogue
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + wm + 16 * i + 4 * (lane / 16) + v;
        const int n = n0 + wn + 16 * j + lane % 16;
        float x = acc[i][j][v];
        const size_t o = (size_t)m * g.ldc + n;
        switch (g.epi) {
          case kEpiStoreF32:
            if (g.bias) x += g.bias[n];
            static_cast<float*>(g.C)[o] = x;
            break;
          case kEpiBiasGelu: {
            const float z = x + g.bias[n];
            if (g.Z) g.Z[o] = z;
            static_cast<T*>(g.C)[o] = from_float<T>(gelu(z));
            break;
          }
          case kEpiGeluGrad:
            static_cast<T*>(g.C)[o] = from_float<T>(x * gelu_grad(g.Z[o]));
            break;
          default:
            break;
        }
      }
}

// BF16 C = A B^T (A: M x K activations, row-major; B: N x K weights, row-major) for the
// forward layers.  Each MFMA operand fragment (one row, 8 consecutive k) is 16 contiguous
// bytes of A or B, so lanes load their fragments straight from global memory into
// registers (no LDS, no barriers), four K slices in flight.  Workgroup tile 128 x 128,
// four waves of 64 x 64 (4 x 4 MFMA 16x16x32 tiles), rows >= M masked.  Same epilogues as
// gemm_kernel.
constexpr int TM = 128, TN = 128, TK = 32;
constexpr int kXcds = 8;  // accelerator complex dies of an MI355X

__global__ void __launch_bounds__(256) gemm_nt_bf16_kernel(GemmArgs g) {
  const __bf16* A = static_cast<const __bf16*>(g.A);
  const __bf16* B = static_cast<const __bf16*>(g.B);
  const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
  // workgroups are dealt round-robin to the 8 XCDs (each with its own L2): give each XCD a
  // contiguous run of tiles, so the N tiles of one row panel of A share an L2
  const int ntn = gridDim.x, ntiles = gridDim.x * gridDim.y;
  const int lin = blockIdx.x + gridDim.x * blockIdx.y;
  int tile = lin;
  if (ntiles % kXcds == 0) tile = (lin % kXcds) * (ntiles / kXcds) + lin / kXcds;
  const int m0 = (tile / ntn) * TM, n0 = (tile % ntn) * TN;
  const int wm = (w / 2) * 64, wn = (w % 2) * 64;
  const int r16 = lane % 16, kq = lane / 16;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const __bf16* pa[4];
  const __bf16* pb[4];
  bool va[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + wm + 16 * i + r16;
    va[i] = m < g.M;
    pa[i] = A + (size_t)(va[i] ? m : 0) * g.lda + 8 * kq;
    pb[i] = B + (size_t)(n0 + wn + 16 * i + r16) * g.ldb + 8 * kq;
  }
  auto load = [&](bf16x8 (&a)[4], bf16x8 (&b)[4], int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = *reinterpret_cast<const bf16x8*>(pa[i] + k0);
      if (!va[i]) a[i] = bf16x8{};
      b[i] = *reinterpret_cast<const bf16x8*>(pb[i] + k0);
    }
  };
  auto mma = [&](const bf16x8 (&a)[4], const bf16x8 (&b)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };
  // four K slices in flight per wave (the global-load latency is several times one
  // slice's MFMA work); stage indices are static after unrolling by four
  constexpr int NS = 4;
  bf16x8 a[NS][4], b[NS][4];
  const int nk = g.K / TK;
#pragma unroll
  for (int u = 0; u < NS - 1; ++u)
    if (u < nk) load(a[u], b[u], u * TK);
  for (int ks = 0; ks < nk; ks += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int k = ks + u;
      if (k < nk) {
        if (k + NS - 1 < nk) load(a[(u + NS - 1) % NS], b[(u + NS - 1) % NS], (k + NS - 1) * TK);
        mma(a[u], b[u]);
      }
    }
  }
  // epilogue through LDS, 32 rows of the wave's 64 x 64 tile at a time: the raw sums go in
  // in the MFMA layout and come out as runs of 4 consecutive columns, where bias, GELU /
  // GELU' and the conversion are applied and every store is a contiguous 8- or 16-byte chunk
  __shared__ __align__(16) float stile[4][32][64 + 4];
  float(*st)[68] = stile[w];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) st[16 * i + 4 * kq + v][16 * j + r16] = acc[2 * h + i][j][v];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = lane + 64 * u, r = e / 16, c4 = 4 * (e % 16);
      const int m = m0 + wm + 32 * h + r, n = n0 + wn + c4;
      if (m >= g.M) continue;
      const float4 x = *reinterpret_cast<const float4*>(&st[r][c4]);
      const size_t o = (size_t)m * g.ldc + n;
      float y[4] = {x.x, x.y, x.z, x.w};
      if (g.epi == kEpiStoreF32) {
        if (g.bias) {
          const float4 b = *reinterpret_cast<const float4*>(g.bias + n);
          y[0] += b.x; y[1] += b.y; y[2] += b.z; y[3] += b.w;
        }
        *reinterpret_cast<float4*>(static_cast<float*>(g.C) + o) = make_float4(y[0], y[1], y[2], y[3]);
      } else {
        if (g.epi == kEpiBiasGelu) {
          const float4 b = *reinterpret_cast<const float4*>(g.bias + n);
          y[0] += b.x; y[1] += b.y; y[2] += b.z; y[3] += b.w;
          if (g.Z) *reinterpret_cast<float4*>(g.Z + o) = make_float4(y[0], y[1], y[2], y[3]);
#pragma unroll
          for (int q = 0; q < 4; ++q) y[q] = gelu(y[q]);
        } else {  // kEpiGeluGrad
          const float4 z = *reinterpret_cast<const float4*>(g.Z + o);
          y[0] *= gelu_grad(z.x); y[1] *= gelu_grad(z.y); y[2] *= gelu_grad(z.z); y[3] *= gelu_grad(z.w);
        }
        __bf16* co = static_cast<__bf16*>(g.C) + o;
        bf16x4 ov;
#pragma unroll
        for (int q = 0; q < 4; ++q) ov[q] = (__bf16)y[q];
        *reinterpret_cast<bf16x4*>(co) = ov;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Training-sized BF16 GEMMs, several independent ones in one launch (a layer's weight gradient beside
// the gradient it passes down).  Workgroup tile 64 x 64, four waves of 32 x 32 (16x16x32 MFMA), K in
// slices of 64: the next slice is loaded 16 bytes a lane into registers while the current one
// multiplies from LDS (two buffers, one barrier a slice).  Either operand may be stored with k as the
// row (a weight gradient contracts over the batch): two k rows are then interleaved into 32-bit LDS
// writes.  LDS rows hold 8-element chunks at chunk ^ (row / 8), which keeps both kinds of writes and
// the fragment reads free of bank conflicts.  A weight gradient may split its K (the batch) over
// workgroups, each writing its own partial; the row sums of its A (the bias gradient) are one more
// MFMA against ones.  What bounds it at a batch of 1,024 is latency, a few slices of one tile per CU:
// small tiles and the split put 100-300 workgroups on the 256 CUs where the 128 x 128 tiles had 32
// (forward layer of 512 units 21 us, weight gradient 26 us, bias gradients 427 us a step with one
// lane per column, before).  The products of a result are added in the order of the other kernels, so
// activations and the gradients passed down are the same bit for bit.
constexpr int TB = 64, kTileLd = TB + 8, kMaxJobs = 3;
// rows up to which a single GEMM takes these tiles: 8,192 rows of 512 units are 512 of the 128 x 128
// tiles, two a CU
constexpr int kTileMaxRows = 8192;

struct TileJob {
  const __bf16 *A, *B;
  void* C;
  const float* bias;
  float* Z;
  float* rowsum;  // sums of A's rows over k (null: none), in the partial's buffer
  int M, N, K, lda, ldb, ldc, opA, opB, epi;
  int ksplit;           // workgroups that share a tile's K
  int64_t part_stride;  // floats between their results
};
struct TileJobs {
  TileJob j[kMaxJobs];
  int first[kMaxJobs + 1];  // first workgroup of each job
};

__device__ inline int tile_at(int row, int k) {
  return row * kTileLd + ((((k >> 3) ^ (row >> 3)) & 7) << 3) + (k & 7);
}
// slice k0 .. k0+63 of rows r0 .. r0+63; kmajor: element (row, k) at k ld + row, else at row ld + k
__device__ inline void tile_load(const __bf16* p, int kmajor, int ld, int r0, int k0, uint4* r) {
  const int t = threadIdx.x;
  if (kmajor) {
    const __bf16* q = p + (size_t)(k0 + 2 * (t / 8)) * ld + r0 + 8 * (t % 8);
    r[0] = *reinterpret_cast<const uint4*>(q);
    r[1] = *reinterpret_cast<const uint4*>(q + ld);
  } else {
    const __bf16* q = p + (size_t)(r0 + t / 4) * ld + k0 + 16 * (t % 4);
    r[0] = *reinterpret_cast<const uint4*>(q);
    r[1] = *reinterpret_cast<const uint4*>(q + 8);
  }
}
__device__ inline void tile_store(__bf16* s, int kmajor, const uint4* r) {
  const int t = threadIdx.x;
  if (kmajor) {
    const unsigned a[4] = {r[0].x, r[0].y, r[0].z, r[0].w}, b[4] = {r[1].x, r[1].y, r[1].z, r[1].w};
    const int k = 2 * (t / 8), row = 8 * (t % 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<unsigned*>(s + tile_at(row + 2 * i, k)) = (a[i] & 0xFFFFu) | (b[i] << 16);
      *reinterpret_cast<unsigned*>(s + tile_at(row + 2 * i + 1, k)) = (a[i] >> 16) | (b[i] & 0xFFFF0000u);
    }
  } else {
    const int row = t / 4, k = 16 * (t % 4);
    *reinterpret_cast<uint4*>(s + tile_at(row, k)) = r[0];
    *reinterpret_cast<uint4*>(s + tile_at(row, k + 8)) = r[1];
  }
}

__global__ void __launch_bounds__(256) gemm_tile_kernel(TileJobs js) {
  __shared__ __align__(16) __bf16 sA[2][TB * kTileLd], sB[2][TB * kTileLd];
  int which = 0;
  while (which < kMaxJobs - 1 && (int)blockIdx.x >= js.first[which + 1]) ++which;
  const TileJob& g = js.j[which];
  const int local = (int)blockIdx.x - js.first[which];
  const int ntn = g.N / TB, split = local % g.ksplit, tile = local / g.ksplit;
  const int m0 = (tile / ntn) * TB, n0 = (tile % ntn) * TB;
  const int nk = g.K / TB, s0 = nk * split / g.ksplit, s1 = nk * (split + 1) / g.ksplit;
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64, r16 = lane % 16, kq = lane / 16;
  const int wm = (w / 2) * 32, wn = (w % 2) * 32;
  const bool sums = g.rowsum && n0 == 0 && wn == 0;
  f32x4 acc[2][2], asum[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    asum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  bf16x8 ones;
#pragma unroll
  for (int q = 0; q < 8; ++q) ones[q] = (__bf16)1.f;
  uint4 ra[2], rb[2];
  const int ka = g.opA == 1, kb = g.opB == 0;
  if (s0 < s1) {
    tile_load(g.A, ka, g.lda, m0, s0 * TB, ra);
    tile_load(g.B, kb, g.ldb, n0, s0 * TB, rb);
    tile_store(sA[0], ka, ra);
    tile_store(sB[0], kb, rb);
  }
  __syncthreads();
  for (int ks = s0; ks < s1; ++ks) {
    const int cur = (ks - s0) & 1;
    if (ks + 1 < s1) {
      tile_load(g.A, ka, g.lda, m0, (ks + 1) * TB, ra);
      tile_load(g.B, kb, g.ldb, n0, (ks + 1) * TB, rb);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8*>(&sA[cur][tile_at(wm + 16 * i + r16, 32 * h + 8 * kq)]);
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = *reinterpret_cast<const bf16x8*>(&sB[cur][tile_at(wn + 16 * j + r16, 32 * h + 8 * kq)]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
      if (sums) {
#pragma unroll
        for (int i = 0; i < 2; ++i) asum[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], ones, asum[i], 0, 0, 0);
      }
    }
    if (ks + 1 < s1) {
      tile_store(sA[1 - cur], ka, ra);
      tile_store(sB[1 - cur], kb, rb);
    }
    __syncthreads();
  }
  if (sums && r16 == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) g.rowsum[(size_t)split * g.part_stride + m0 + wm + 16 * i + 4 * kq + v] = asum[i][v];
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + wm + 16 * i + 4 * kq + v, n = n0 + wn + 16 * j + r16;
        const size_t o = (size_t)m * g.ldc + n;
        float x = acc[i][j][v];
        if (g.epi == kEpiStoreF32) {
          if (g.bias) x += g.bias[n];
          static_cast<float*>(g.C)[(size_t)split * g.part_stride + o] = x;
        } else if (g.epi == kEpiBiasGelu) {
          const float z = x + g.bias[n];
          if (g.Z) g.Z[o] = z;
          static_cast<__bf16*>(g.C)[o] = (__bf16)gelu(z);
        } else {  // kEpiGeluGrad
          static_cast<__bf16*>(g.C)[o] = (__bf16)(x * gelu_grad(g.Z[o]));
        }
      }
}

// g[i] = sum of the S partials of parameter i, in order; the last workgroup adds up the loss
__global__ void __launch_bounds__(256) gather_grad_kernel(const float* part, int S, int64_t n, float* g, const double* lp,
                                                          int64_t B, double scale, double* loss) {
  if (blockIdx.x + 1 == gridDim.x) {
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < B; i += 256) s += lp[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0] * scale;
    return;
  }
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float v = part[i];
  for (int q = 1; q < S; ++q) v += part[(size_t)q * n + i];
  g[i] = v;
}

// The whole network for inference in one kernel (BF16): normalisation, three layers, GELU, logits.
// A workgroup of eight waves carries 64 signals through all layers with the activations in LDS (one
// buffer: a layer's results wait in registers, already activated and rounded, until every wave has
// read its inputs), so only the signals are read and only the logits written; the weights (0.9 MB at
// 512 units) are read from L2 as MFMA fragments, 16 contiguous bytes a lane.  A wave owns the
// 16-column tiles w, w + 8, ... of a layer.
// What bounds it: the vector-ALU instructions of erff (25-45 a value, 2 x 512 values a signal) and the
// waits between a layer's phases; two workgroups share a CU so that one's products run beside the
// other's GELUs.  Four waves a SIMD (128 registers) hide the weights' latency better than loading a
// slice ahead, whose 16 registers spilled (171 against 152 us); one rolled copy of the two hidden
// layers spilled more.  Same operations as the layer-by-layer kernels in the same order, bit for bit:
// 65,536 signals, 512 units: 60 + 142 + 70 us for the three layers and 17 us for the normalisation
// before.
constexpr int kFwdRows = 64, kFwdWaves = 8;

template <int NT>
__global__ void __launch_bounds__(64 * kFwdWaves) __attribute__((amdgpu_waves_per_eu(4)))
    mlp_forward_kernel(MlpForwardArgs g) {
  extern __shared__ __align__(16) unsigned char fwd_smem[];
  __bf16* act = reinterpret_cast<__bf16*>(fwd_smem);
  const int H = g.H, ld = H + 8;  // 16-byte aligned rows, spread over the banks
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = threadIdx.x % 64;
  const int r16 = lane % 16, kq = lane / 16;
  const int64_t row0 = (int64_t)blockIdx.x * kFwdRows;
  // x = vec(Y) / ||Y||_F: a wave normalises eight signals, lane p holding pixel p
  constexpr int RW = kFwdRows / kFwdWaves;
  float y[RW];
#pragma unroll
  for (int u = 0; u < RW; ++u) {
    const int64_t r = row0 + w * RW + u;
    y[u] = r < g.N ? g.Y[r * 64 + lane] : 0.f;
  }
#pragma unroll
  for (int u = 0; u < RW; ++u) {
#pragma clang fp contract(off)
    float q = y[u] * y[u];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
    const float inv = q > 0.f ? rsqrtf(q) : 0.f;
    act[(w * RW + u) * ld + lane] = (__bf16)(y[u] * inv);
  }
  __syncthreads();
  auto products = [&](const __bf16* W, int K, int ntiles, f32x4(&acc)[4][NT]) __attribute__((always_inline)) {
    const __bf16* pb[NT];  // uniform: the tiles' first rows (a tile past the last reads the first)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int nt = w + kFwdWaves * j;
      pb[j] = W + (size_t)(16 * (nt < ntiles ? nt : 0)) * K;
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    unsigned ob = (unsigned)(r16 * K + 8 * kq);  // this lane's place in a tile
    const __bf16* pa = act + r16 * ld + 8 * kq;
    for (int k = 0; k < K; k += 32) {
      bf16x8 b[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) b[j] = *reinterpret_cast<const bf16x8*>(pb[j] + (ob + k));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(pa + 16 * i * ld + k);
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[j], acc[i][j], 0, 0, 0);
      }
    }
  };
  auto hidden = [&](const __bf16* W, const float* bias, int K) __attribute__((always_inline)) {
    f32x4 acc[4][NT];
    products(W, K, H / 16, acc);
    unsigned h[4][NT][2];  // the rounded results, in pairs
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int nt = w + kFwdWaves * j;
      const float bj = bias[16 * (nt < H / 16 ? nt : 0) + r16];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          const __bf16 lo = (__bf16)gelu(acc[i][j][2 * v] + bj), hi = (__bf16)gelu(acc[i][j][2 * v + 1] + bj);
          h[i][j][v] = __builtin_bit_cast(unsigned short, lo) | (unsigned)__builtin_bit_cast(unsigned short, hi) << 16;
          asm volatile("" : "+v"(h[i][j][v]));  // finished here, not after the barrier
        }
    }
    __syncthreads();  // every wave has read the layer's inputs
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int nt = w + kFwdWaves * j;
      if (nt >= H / 16) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          act[(16 * i + 4 * kq + v) * ld + 16 * nt + r16] =
              __builtin_bit_cast(__bf16, (unsigned short)(h[i][j][v / 2] >> (16 * (v % 2))));
    }
    __syncthreads();
  };
  hidden(g.W1, g.b1, 64);
  hidden(g.W2, g.b2, H);
  f32x4 acc[4][NT];
  for (int t0 = 0; t0 < g.A / 16; t0 += kFwdWaves * NT) {
    products(g.W3 + (size_t)16 * t0 * H, H, g.A / 16 - t0, acc);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int nt = w + kFwdWaves * j + t0;
      if (nt >= g.A / 16) continue;
      const float bj = g.b3[16 * nt + r16];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t r = row0 + 16 * i + 4 * kq + v;
          if (r < g.N) g.logits[r * g.A + 16 * nt + r16] = acc[i][j][v] + bj;
        }
    }
  }
}

// X[b][p] = Y_{idx(b)}[p] / ||Y_{idx(b)}||_F in the compute type (vec order = column-major)
template <typename T>
__global__ void prep_input_kernel(const float* Y, const int32_t* idx, int64_t B, int M, T* X, float* ynorm2) {
  const int64_t b = blockIdx.x;
  if (b >= B) return;
  const int64_t src = idx ? idx[b] : b;
  const float* y = Y + src * M;
  __shared__ float red[64];
  float s = 0.f;
  for (int p = threadIdx.x; p < M; p += blockDim.x) s += y[p] * y[p];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 32; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const float nrm2 = red[0];
  const float inv = nrm2 > 0.f ? rsqrtf(nrm2) : 0.f;
  for (int p = threadIdx.x; p < M; p += blockDim.x) X[b * M + p] = from_float<T>(y[p] * inv);
  if (ynorm2 && threadIdx.x == 0) ynorm2[b] = nrm2;
}

// dZ = (sigmoid(z) - label) / (B * A), label = 1 on the atoms of the code; per-block FP64 loss partials
template <typename T>
__global__ void __launch_bounds__(256) bce_grad_kernel(const float* Z, const int32_t* supp, const int32_t* idx, int64_t B,
                                                       int A, int s, T* dZ, double* loss_part) {
  __shared__ double red[256];
  const int64_t b = blockIdx.x;
  const int64_t src = idx ? idx[b] : b;
  double l = 0.0;
  const float scale = 1.0f / ((float)B * (float)A);
  for (int a = threadIdx.x; a < A; a += blockDim.x) {
    float y = 0.f;
    for (int t = 0; t < s; ++t) y = supp[src * s + t] == a ? 1.f : y;
    const float z = Z[b * A + a];
    const float sig = 1.f / (1.f + expf(-z));
    dZ[b * A + a] = from_float<T>((sig - y) * scale);
    // stable BCE with logits: max(z,0) - z*y + log(1 + exp(-|z|))
    l += (double)(fmaxf(z, 0.f) - z * y + log1pf(expf(-fabsf(z))));
  }
  red[threadIdx.x] = l;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss_part[b] = red[0];
}

// db[n] = sum_b dZ[b][n], fixed order (one thread per column; FP32 check mode)
__global__ void bias_grad_kernel(const float* dZ, int64_t B, int N, float* db) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  float s = 0.f;
  for (int64_t b = 0; b < B; ++b) s += dZ[b * N + n];
  db[n] = s;
}

__global__ void sum_kernel(const double* x, int64_t n, double scale, double* out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0.0;
  for (int64_t i = 0; i < n; ++i) s += x[i];
  *out = s * scale;
}

TileJob tile_job(const GemmArgs& g, int opA, int opB) {
  return TileJob{static_cast<const __bf16*>(g.A), static_cast<const __bf16*>(g.B), g.C, g.bias, g.Z, nullptr,
                 g.M, g.N, g.K, g.lda, g.ldb, g.ldc, opA, opB, g.epi, 1, 0};
}

// Adam on the FP32 master parameters, then the compute-type copy
template <typename T>
__global__ void adam_kernel(float* p, float* m, float* v, const float* g, T* pc, int64_t n, float lr, float b1, float b2,
                            float eps, float bc1, float bc2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / bc1, vh = vi / bc2;
  const float pi = p[i] - lr * mh / (sqrtf(vh) + eps);
  p[i] = pi;
  if (pc) pc[i] = from_float<T>(pi);
}

template <typename T>
__global__ void copy_params_kernel(const float* p, T* pc, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) pc[i] = from_float<T>(p[i]);
}

}  // namespace

hipError_t launch_gemm_batch(const GemmJob* jobs, int n, hipStream_t st) {
  TileJobs js{};
  int blocks = 0;
  for (int q = 0; q < kMaxJobs; ++q) {
    js.first[q] = blocks;
    if (q >= n) continue;
    const GemmArgs& g = jobs[q].g;
    if (n > kMaxJobs || g.M % TB || g.N % TB || g.K % TB || jobs[q].ksplit < 1) return hipErrorInvalidValue;
    js.j[q] = tile_job(g, jobs[q].opA, jobs[q].opB);
    js.j[q].rowsum = jobs[q].rowsum;
    js.j[q].ksplit = jobs[q].ksplit;
    js.j[q].part_stride = jobs[q].part_stride;
    blocks += (g.M / TB) * (g.N / TB) * jobs[q].ksplit;
  }
  js.first[kMaxJobs] = blocks;
  hipLaunchKernelGGL(gemm_tile_kernel, dim3(blocks), dim3(256), 0, st, js);
  return hipGetLastError();
}

hipError_t launch_gather_grad(const float* part, int S, int64_t n, float* g, const double* loss_part, int64_t B, int A,
                              double* loss, hipStream_t st) {
  hipLaunchKernelGGL(gather_grad_kernel, dim3((unsigned)((n + 255) / 256 + 1)), dim3(256), 0, st, part, S, n, g, loss_part,
                     B, 1.0 / ((double)B * A), loss);
  return hipGetLastError();
}

template <>
hipError_t launch_gemm<__bf16>(const GemmArgs& g, int opA, int opB, hipStream_t st) {
  // many rows: 128 x 128 tiles; few leave those with too few workgroups
  if (g.M >= kTileMaxRows && opA == 0 && opB == 1 && g.N % TN == 0 && g.K % TK == 0) {
    hipLaunchKernelGGL(gemm_nt_bf16_kernel, dim3(g.N / TN, (g.M + TM - 1) / TM), dim3(256), 0, st, g);
    return hipGetLastError();
  }
  const GemmJob j{g, opA, opB, nullptr, 1, 0};
  return launch_gemm_batch(&j, 1, st);
}

template <>
hipError_t launch_gemm<float>(const GemmArgs& g, int opA, int opB, hipStream_t st) {
  const dim3 grid(g.N / BN, g.M / BM);
  if (opA == 0 && opB == 1) hipLaunchKernelGGL((gemm_kernel<0, 1>), grid, dim3(256), 0, st, g);
  else if (opA == 0 && opB == 0) hipLaunchKernelGGL((gemm_kernel<0, 0>), grid, dim3(256), 0, st, g);
  else if (opA == 1 && opB == 0) hipLaunchKernelGGL((gemm_kernel<1, 0>), grid, dim3(256), 0, st, g);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

bool mlp_forward_supported(int M, int H, int A) { return M == 64 && H % 64 == 0 && H <= 512 && A % 16 == 0; }

hipError_t launch_mlp_forward(const MlpForwardArgs& g, hipStream_t st) {
  if (g.N <= 0) return hipSuccess;
  const dim3 grid((unsigned)((g.N + kFwdRows - 1) / kFwdRows)), block(64 * kFwdWaves);
  const size_t lds = sizeof(__bf16) * (size_t)kFwdRows * (g.H + 8);
  const int nt = (g.H / 16 + kFwdWaves - 1) / kFwdWaves;
  switch (nt) {
    case 1: hipLaunchKernelGGL(mlp_forward_kernel<1>, grid, block, lds, st, g); break;
    case 2: hipLaunchKernelGGL(mlp_forward_kernel<2>, grid, block, lds, st, g); break;
    case 3: hipLaunchKernelGGL(mlp_forward_kernel<3>, grid, block, lds, st, g); break;
    case 4: hipLaunchKernelGGL(mlp_forward_kernel<4>, grid, block, lds, st, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t mlp_init_device() {
  // 64 rows of 520 units: just above the default LDS limit
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_forward_kernel<4>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
}

template <typename T>
hipError_t launch_prep_input(const float* Y, const int32_t* idx, int64_t B, int M, T* X, float* ynorm2, hipStream_t st) {
  if (B == 0) return hipSuccess;
  hipLaunchKernelGGL(prep_input_kernel<T>, dim3((unsigned)B), dim3(64), 0, st, Y, idx, B, M, X, ynorm2);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_bce_grad(const float* Z, const int32_t* supp, const int32_t* idx, int64_t B, int A, int s, T* dZ,
                           double* loss_part, double* loss, hipStream_t st) {
  hipLaunchKernelGGL(bce_grad_kernel<T>, dim3((unsigned)B), dim3(256), 0, st, Z, supp, idx, B, A, s, dZ, loss_part);
  if (!loss) return hipGetLastError();  // the caller adds the parts up
  hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(64), 0, st, loss_part, B, 1.0 / ((double)B * A), loss);
  return hipGetLastError();
}

hipError_t launch_bias_grad(const float* dZ, int64_t B, int N, float* db, hipStream_t st) {
  hipLaunchKernelGGL(bias_grad_kernel, dim3((N + 255) / 256), dim3(256), 0, st, dZ, B, N, db);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_adam(float* p, float* m, float* v, const float* g, T* pc, int64_t n, float lr, int step,
                       hipStream_t st) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float bc1 = 1.f - powf(b1, (float)step), bc2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, m, v, g, pc, n, lr, b1, b2,
                     eps, bc1, bc2);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_copy_params(const float* p, T* pc, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(copy_params_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, pc, n);
  return hipGetLastError();
}

#define SDL_MLP_INST(T)                                                                                           \
  template hipError_t launch_prep_input<T>(const float*, const int32_t*, int64_t, int, T*, float*, hipStream_t); \
  template hipError_t launch_bce_grad<T>(const float*, const int32_t*, const int32_t*, int64_t, int, int, T*,    \
                                         double*, double*, hipStream_t);                                         \
  template hipError_t launch_adam<T>(float*, float*, float*, const float*, T*, int64_t, float, int, hipStream_t); \
  template hipError_t launch_copy_params<T>(const float*, T*, int64_t, hipStream_t);
SDL_MLP_INST(float)
SDL_MLP_INST(__bf16)
#undef SDL_MLP_INST

}  // namespace sdl
