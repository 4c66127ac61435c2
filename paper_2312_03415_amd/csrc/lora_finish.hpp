// Second kernel of the few-token forward, Y = X W + (s X A) B + bias for up to a few hundred rows of X (Section 2's forward 1
// of arxiv 2312.03415 where a generating program calls it, one or a few dozen tokens at a time).
//
// Such a call reads W and little else, and four launches in a row (X A, its reduce, [X|T] [W;B] split over K, its reduce)
// spent more time on being launched and on waiting for each other than on W.  Here the first launch (gemm_mt.hpp, XA
// build) forms the fp32 partials of X W and of X A side by side, K split over enough workgroups to fill the chip, and this
// one sums them in slice order, rounds T = s X A to the storage type as the stored T is everywhere else, and adds T B and
// the bias: 1 x 4096 -> 4096, r 16: 21.9 us on the GPU in four launches, 13.2 in two (of which this one 4.7); 48 x 4096 ->
// 11008, r 32: 41.5 and 23.7 (6.0).
//
// Bound by latency: a thread owns 16 bytes of a row of Y; a workgroup is cx column chunks by ry rows (ry covers the rows up
// to 32, so that one row still spreads over 64 threads), with its rows of T in LDS.
#pragma once
#include "gemm_engine.hpp"

namespace rl {

struct FinishArgs {
  const float *partial, *partial_t;  // [splits][M][N], [splits][M][R]
  const void *B, *bias;              // [R, N]; [N] or nullptr
  void *C, *T;                       // [M, N]; [M, R] or nullptr (T is kept for the backward)
  int64_t ldb, ldc, ldt;
  int M, N, R, splits;
  float t_alpha;
};

template <typename T>
__global__ __launch_bounds__(256) void lora_finish_kernel(FinishArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  float* const sT = reinterpret_cast<float*>(smem_raw);  // [blockDim.y][R]
  const int m0 = (int)(blockIdx.y * blockDim.y), m = m0 + (int)threadIdx.y;
  const int n = ((int)(blockIdx.x * blockDim.x) + (int)threadIdx.x) * 8;
  const bool ok = m < g.M && n < g.N;  // N is a multiple of 8
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  const T* const b = static_cast<const T*>(g.B) + n;
  i32x4 first[8];  // the first eight rows of B (R is a multiple of 8), on their way while T is formed
  if (ok) {
#pragma unroll
    for (int k = 0; k < 8; ++k) first[k] = *reinterpret_cast<const i32x4*>(b + (int64_t)k * g.ldb);
    const float* src = g.partial + (int64_t)m * g.N + n;
#pragma unroll 4
    for (int z = 0; z < g.splits; ++z) {
      const f32x4 p0 = *reinterpret_cast<const f32x4*>(src + (int64_t)z * g.M * g.N);
      const f32x4 p1 = *reinterpret_cast<const f32x4*>(src + (int64_t)z * g.M * g.N + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { acc[e] += p0[e]; acc[4 + e] += p1[e]; }
    }
  }
  // this workgroup's rows of T (a row per threadIdx.y, its columns over threadIdx.x)
  for (int k = (int)threadIdx.x; k < g.R; k += (int)blockDim.x) {
    float t = 0.f;
    if (m < g.M) {
      const float* src = g.partial_t + (int64_t)m * g.R + k;
#pragma unroll 4
      for (int z = 0; z < g.splits; ++z) t += src[(int64_t)z * g.M * g.R];
    }
    const T tr = from_f32<T>(g.t_alpha * t);
    sT[(int)threadIdx.y * g.R + k] = (float)tr;
    if (g.T != nullptr && blockIdx.x == 0 && m < g.M) static_cast<T*>(g.T)[(int64_t)m * g.ldt + k] = tr;
  }
  __syncthreads();
  if (!ok) return;
  const float* const tr = sT + (int)threadIdx.y * g.R;
  auto add = [&](const i32x4& v, float t) {
    const T* v8 = reinterpret_cast<const T*>(&v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += t * (float)v8[e];
  };
#pragma unroll
  for (int k = 0; k < 8; ++k) add(first[k], tr[k]);
#pragma unroll 8
  for (int k = 8; k < g.R; ++k) add(*reinterpret_cast<const i32x4*>(b + (int64_t)k * g.ldb), tr[k]);
  if (g.bias != nullptr) {
    const i32x4 v = *reinterpret_cast<const i32x4*>(static_cast<const T*>(g.bias) + n);
    const T* v8 = reinterpret_cast<const T*>(&v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += (float)v8[e];
  }
  T o8[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o8[e] = from_f32<T>(acc[e]);
  *reinterpret_cast<i32x4*>(static_cast<T*>(g.C) + (int64_t)m * g.ldc + n) = *reinterpret_cast<const i32x4*>(o8);
}

}  // namespace rl
