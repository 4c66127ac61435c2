// Second kernel of the few-token forward, Y = X W + (s X A) B + bias for up to a few hundred rows of X (Section 2's forward 1
// of arxiv 2312.03415 where a generating program calls it, one or a few dozen tokens at a time).
//
// Such a call reads W and little else, and four launches in a row (X A, its reduce, [X|T] [W;B] split over K, its reduce)
// spent more time on being launched and on waiting for each other than on W.  Here the first launch (gemm_mt.hpp, XA
// build) forms the fp32 partials of X W and of X A side by side, K split over enough workgroups to fill the chip, and this
// one sums them in slice order, rounds T = s X A to the storage type as the stored T is everywhere else, and adds T B and
// the bias: 1 x 4096 -> 4096, r 16: 21.9 us on the GPU in four launches, 12.2 in two (of which this one 4.1); 48 x 4096 ->
// 11008, r 32: 41.5 and 21.5 (5.2).
//
// Bound by latency, that is by the number of trips to memory one behind the other: the slices are summed four at a time, and what
// is left of them together (as a rolled remainder the last three of seven took a trip each), T's columns of a thread four at a
// time, sixteen rows of B ahead of T and the others a block of eight ahead.  Together 9.0 -> 5.9 us at 3 x 8192 -> 8192 r 48, 13.6
// -> 12.2 at 16 x 4096 -> 4096 r 128, 5.7 -> 5.2 at 48 x 4096 -> 11008 r 32.  (Eight slices at a time, padded or each count
// unrolled, cost registers and instruction fetches: 94 x 9568 -> 1024 in twelve slices 5.0 -> 6.3.)  A thread owns 16 bytes of a
// row of Y; a workgroup is cx column chunks by ry rows (ry covers the rows up to 32, so that one row still spreads over 64
// threads), with its rows of T in LDS.
#pragma once
#include "gemm_engine.hpp"

#include <type_traits>

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
  i32x4 first[16];  // the first sixteen rows of B (R is a multiple of 8), on their way while T is formed
  const bool second = g.R > 8;  // uniform
  if (ok) {
#pragma unroll
    for (int k = 0; k < 8; ++k) first[k] = *reinterpret_cast<const i32x4*>(b + (int64_t)k * g.ldb);
    if (second) {
#pragma unroll
      for (int k = 8; k < 16; ++k) first[k] = *reinterpret_cast<const i32x4*>(b + (int64_t)k * g.ldb);
    }
  }
  // f(first slice, how many: a constant up to four) over all slices in order
  auto slices = [&](auto f) {
    int z = 0;
    for (; z + 4 <= g.splits; z += 4) f(z, std::integral_constant<int, 4>{});
    switch (g.splits - z) {
      case 1: f(z, std::integral_constant<int, 1>{}); break;
      case 2: f(z, std::integral_constant<int, 2>{}); break;
      case 3: f(z, std::integral_constant<int, 3>{}); break;
      default: break;
    }
  };
  if (ok) {
    const float* const src = g.partial + (int64_t)m * g.N + n;
    slices([&](int z, auto u_c) {
      constexpr int U = decltype(u_c)::value;
      f32x4 p[U][2];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        p[u][0] = *reinterpret_cast<const f32x4*>(src + (int64_t)(z + u) * g.M * g.N);
        p[u][1] = *reinterpret_cast<const f32x4*>(src + (int64_t)(z + u) * g.M * g.N + 4);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) { acc[e] += p[u][0][e]; acc[4 + e] += p[u][1][e]; }
    });
  }
  // this workgroup's rows of T (a row per threadIdx.y, its columns over threadIdx.x: Q of them a thread at a time)
  auto sum_t = [&](auto q_c, int k0) {
    constexpr int Q = decltype(q_c)::value;
    float t[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) t[q] = 0.f;
    if (m < g.M) {
      const float* const src = g.partial_t + (int64_t)m * g.R;
      slices([&](int z, auto u_c) {
        constexpr int U = decltype(u_c)::value;
        float p[U][Q];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int k = k0 + q * (int)blockDim.x;
            p[u][q] = src[(int64_t)(z + u) * g.M * g.R + (k < g.R ? k : k0)];
          }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int q = 0; q < Q; ++q) t[q] += p[u][q];
      });
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = k0 + q * (int)blockDim.x;
      if (k < g.R) {
        const T tr = from_f32<T>(g.t_alpha * t[q]);
        sT[(int)threadIdx.y * g.R + k] = (float)tr;
        if (g.T != nullptr && blockIdx.x == 0 && m < g.M) static_cast<T*>(g.T)[(int64_t)m * g.ldt + k] = tr;
      }
    }
  };
  if (g.R <= (int)blockDim.x) {
    if ((int)threadIdx.x < g.R) sum_t(std::integral_constant<int, 1>{}, (int)threadIdx.x);
  } else {
    for (int k0 = (int)threadIdx.x; k0 < g.R; k0 += 4 * (int)blockDim.x) sum_t(std::integral_constant<int, 4>{}, k0);
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
  if (second) {
#pragma unroll
    for (int k = 8; k < 16; ++k) add(first[k], tr[k]);
  }
  // the others in blocks of eight, the next one on its way while a block is multiplied
  if (g.R > 16) {
    i32x4 rows[2][8];
    auto fetch = [&](i32x4 (&to)[8], int k0) {
#pragma unroll
      for (int u = 0; u < 8; ++u) to[u] = *reinterpret_cast<const i32x4*>(b + (int64_t)((k0 < g.R ? k0 : 16) + u) * g.ldb);
    };
    fetch(rows[0], 16);
    for (int k0 = 16; k0 < g.R; k0 += 16) {
      fetch(rows[1], k0 + 8);
#pragma unroll
      for (int u = 0; u < 8; ++u) add(rows[0][u], tr[k0 + u]);
      fetch(rows[0], k0 + 16);
      if (k0 + 8 < g.R) {  // uniform
#pragma unroll
        for (int u = 0; u < 8; ++u) add(rows[1][u], tr[k0 + 8 + u]);
      }
    }
  }
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
