// Second kernel of the few-token forward, Y = X W + (s X A) B + bias for up to a few hundred rows of X (Section 2's forward 1
// of arxiv 2312.03415 where a generating program calls it, one or a few dozen tokens at a time).
//
// Such a call reads W and little else, and four launches in a row (X A, its reduce, [X|T] [W;B] split over K, its reduce)
// spent more time on being launched and on waiting for each other than on W.  Here the first launch (gemm_mt.hpp, XA
// build) forms the fp32 partials of X W and of X A side by side, K split over enough workgroups to fill the chip, and this
// one sums them in slice order, rounds T = s X A to the storage type as the stored T is everywhere else, and adds T B and
// the bias: 1 x 4096 -> 4096, r 16: 21.9 us on the GPU in four launches, 12.2 in two; 48 x 4096 -> 11008, r 32:
// 41.5 and 21.5.
//
// Bound by latency, that is by the number of trips to memory one behind the other: a wave's tile of B and the first U slices of X W and
// of X A (all of them, up to U: finish_shape) are on their way at once, further slices U at a time.  A workgroup is one wave with 16 rows
// of Y and 32 P columns; T B runs on the matrix cores, B turned by the transposing LDS read, T summed and rounded by every wave that
// needs it, in the registers in which the products take it.  The columns of a pair of 16-wide blocks interleave in fours, so that a lane
// holds eight in a row: 16-byte stores.
// With T B on the vector units, 256 threads sharing T through LDS behind a barrier and each walking B's rows from memory, 16 x 2048 ->
// 8192 r 128 took 13.1 us (now 3.9), 58 x 2304 -> 768 r 64 6.8 (3.4), 48 x 4096 -> 11008 r 32 5.7 (4.0), 1 x 4096 -> 4096 r 16 3.9 (3.9).
#pragma once
#include "gemm_mt.hpp"

namespace rl {

struct FinishArgs {
  const float *partial, *partial_t;  // [splits][M][N], [splits][M][R]
  const void *B, *bias;              // [R, N]; [N] or nullptr
  void *C, *T;                       // [M, N]; [M, R] or nullptr (T is kept for the backward)
  int64_t ldb, ldc, ldt;
  int M, N, R, splits;
  float t_alpha;
};

// How a launch is built: 64 columns a wave where those are enough waves to go round, and U slices on their way at a time: four, two where
// 64 columns and a rank beyond 64 leave no registers for more, eight where 32 columns and up to 32 of the rank do and there are more than four.
struct FinishShape {
  int cols, u;
};
inline FinishShape finish_shape(int64_t M, int64_t N, int64_t R, int splits) {
  const bool wide = ((N + 63) / 64) * ((M + 15) / 16) >= 512;
  return {wide ? 64 : 32, wide ? (R > 64 ? 2 : 4) : (R <= 32 && splits > 4 ? 8 : 4)};
}

// KS: K steps of 32 that cover the rank
template <typename T, int KS, int P, int U>
__global__ __launch_bounds__(64) void lora_finish_kernel(FinishArgs g) {
  constexpr int COLS = 32 * P, LD = COLS + 8, NB = 2 * KS * P;
  __shared__ __attribute__((aligned(16))) T sB[KS * 32 * LD];
  const int lane = threadIdx.x, s16 = lane & 15, grp = lane >> 4;
  const int m = (int)blockIdx.y * 16 + s16, n0 = (int)blockIdx.x * COLS;
  const bool row_ok = m < g.M;
  i32x4 breg[NB];  // this lane's chunks of B[0:R, n0:n0+COLS], zeros beyond it
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int c = lane + 64 * j, k = c / (4 * P), col = (c % (4 * P)) * 8;
    i32x4 v = {0, 0, 0, 0};
    if (k < g.R && n0 + col < g.N) v = *reinterpret_cast<const i32x4*>(static_cast<const T*>(g.B) + (int64_t)k * g.ldb + n0 + col);
    breg[j] = v;
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[P][2], t[KS][2];  // X W: columns n0 + 32 p + 8 grp + 4 b ..; X A: columns 32 ks + 8 grp + 4 h .. of row m
#pragma unroll
  for (int p = 0; p < P; ++p) acc[p][0] = acc[p][1] = zero;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) t[ks][0] = t[ks][1] = zero;
  bool col_ok[P], t_ok[KS];  // N and R are multiples of 8: a lane's eight columns are valid together
#pragma unroll
  for (int p = 0; p < P; ++p) col_ok[p] = row_ok && n0 + 32 * p + 8 * grp < g.N;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) t_ok[ks] = row_ok && 32 * ks + 8 * grp < g.R;
  const float* const src = g.partial + (int64_t)m * g.N + n0 + 8 * grp;
  const float* const src_t = g.partial_t + (int64_t)m * g.R + 8 * grp;
  // U slices at a time in their order, the loads of all of them first (those beyond the last are zeros)
  for (int z = 0; z < g.splits; z += U) {
    f32x4 y[U][P][2], x[U][KS][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live = z + u < g.splits;  // uniform
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          y[u][p][b] = zero;
          if (live && col_ok[p]) y[u][p][b] = *reinterpret_cast<const f32x4*>(src + (int64_t)(z + u) * g.M * g.N + 32 * p + 4 * b);
        }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          x[u][ks][h] = zero;
          if (live && t_ok[ks]) x[u][ks][h] = *reinterpret_cast<const f32x4*>(src_t + (int64_t)(z + u) * g.M * g.R + 32 * ks + 4 * h);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[p][b] += y[u][p][b];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int h = 0; h < 2; ++h) t[ks][h] += x[u][ks][h];
    }
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int c = lane + 64 * j;
    *reinterpret_cast<i32x4*>(sB + (c / (4 * P)) * LD + (c % (4 * P)) * 8) = breg[j];
  }
  i32x4 tf[KS];  // T = s X A, rounded as the stored T is everywhere else
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    T t8[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      t8[e] = from_f32<T>(g.t_alpha * t[ks][0][e]);
      t8[4 + e] = from_f32<T>(g.t_alpha * t[ks][1][e]);
    }
    tf[ks] = *reinterpret_cast<const i32x4*>(t8);
    if (g.T != nullptr && blockIdx.x == 0 && t_ok[ks]) *reinterpret_cast<i32x4*>(static_cast<T*>(g.T) + (int64_t)m * g.ldt + 32 * ks + 8 * grp) = tf[ks];
  }
  __syncthreads();  // (one wave)
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // lane s of 16 points at four columns of row k0 + s / 4 and receives one column of rows k0 .. k0 + 3
        const T* const q = sB + (32 * ks + 8 * grp + (s16 >> 2)) * LD + 32 * p + 8 * (s16 & 3) + 4 * b;
        const i32x2 lo = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q)));
        const i32x2 hi = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q + 4 * LD)));
        acc[p][b] = Mma16<T>::mma(i32x4{lo[0], lo[1], hi[0], hi[1]}, tf[ks], acc[p][b]);
      }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (!col_ok[p]) continue;
    const int n = n0 + 32 * p + 8 * grp;
    T o8[8];
    i32x4 bv = {0, 0, 0, 0};
    if (g.bias != nullptr) bv = *reinterpret_cast<const i32x4*>(static_cast<const T*>(g.bias) + n);
    const T* const b8 = reinterpret_cast<const T*>(&bv);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o8[e] = from_f32<T>(acc[p][0][e] + (float)b8[e]);
      o8[4 + e] = from_f32<T>(acc[p][1][e] + (float)b8[4 + e]);
    }
    *reinterpret_cast<i32x4*>(static_cast<T*>(g.C) + (int64_t)m * g.ldc + n) = *reinterpret_cast<const i32x4*>(o8);
  }
}

}  // namespace rl
