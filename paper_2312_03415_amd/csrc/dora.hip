// Small kernels of the DoRA layer (see dora.hpp).  Only the dm pass moves real data (it reads dY and Y once,
// 2 n o e bytes, HBM-bound); the others touch o or r x o elements.
#include "dora.hpp"

#include "gemm.hpp"

namespace rl {
namespace {

constexpr int kThreads = 256;

// A workgroup owns 64 columns, four row groups of 64 threads.  With partials: c[j] = sqrt(the column's partial sums, rows q,
// q + 4, ... per group, the groups in order); without: c is read.  Then g[j] = m[j] / c[j], and out = in diag(g).  One launch:
// both halves are latency (a few loads deep), 11.4 + 3.6 us as two kernels with a thread per column walking all rows,
// 6.2 in one (8192 columns, 32 partial rows, r 16); without the sums 2.6 + 3.6 and 3.6.
template <typename T>
__global__ __launch_bounds__(kThreads) void dora_scale_kernel(const float* __restrict__ partial, int rows, const T* __restrict__ m,
                                                              float* __restrict__ c, float* __restrict__ g, const T* in, int64_t ldi,
                                                              T* out, int64_t ldo, int R, int O) {
  __shared__ float part[4][64];
  const int jj = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + jj;
  float cj = 1.f;
  if (partial != nullptr) {
    float sum = 0.f;
    for (int y0 = q; y0 < rows; y0 += 64) {  // sixteen rows on their way at a time, zeros beyond the last
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = j < O && y0 + 4 * u < rows ? partial[(int64_t)(y0 + 4 * u) * O + j] : 0.f;
#pragma unroll
      for (int u = 0; u < 16; ++u) sum += v[u];
    }
    part[q][jj] = sum;
    __syncthreads();
    cj = sqrtf(((part[0][jj] + part[1][jj]) + part[2][jj]) + part[3][jj]);
    if (q == 0 && j < O) c[j] = cj;
  } else if (j < O) {
    cj = c[j];
  }
  if (j >= O) return;
  const float gj = (float)m[j] / cj;
  if (q == 0) g[j] = gj;
  if (in == nullptr) return;
#pragma unroll 4
  for (int k = q; k < R; k += 4) out[(int64_t)k * ldo + j] = (T)((float)in[(int64_t)k * ldi + j] * gj);
}

// out[k,j] = in[k,j] g[j], eight columns per thread (O is a multiple of 8, rows are 16-byte aligned)
template <typename T>
__global__ __launch_bounds__(kThreads) void dora_colscale_kernel(const T* in, int64_t ldi, const float* __restrict__ g, T* out,
                                                                 int64_t ldo, int R, int O) {
  using V4 = __attribute__((__vector_size__(4 * sizeof(int)))) int;
  const int j = (blockIdx.x * kThreads + threadIdx.x) * 8;
  const int k = blockIdx.y;
  if (j >= O || k >= R) return;
  const V4 v = *reinterpret_cast<const V4*>(in + (int64_t)k * ldi + j);
  const T* v8 = reinterpret_cast<const T*>(&v);
  T o8[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o8[e] = (T)((float)v8[e] * g[j + e]);
  *reinterpret_cast<V4*>(out + (int64_t)k * ldo + j) = *reinterpret_cast<const V4*>(o8);
}

// A workgroup owns 128 columns and a slice of rows.  Thread (rr, cg) = (tid / 16, tid % 16) reads 16 bytes
// (8 columns) of dY and of Y from the rows rr, rr + 16, ... of the slice (a wave instruction covers four whole
// 256-byte row segments) and keeps 8 running sums; the 16 threads of a column group are then added in the
// order of rr through LDS.  Requires o % 8 == 0 and 16-byte aligned rows.
template <typename T>
__global__ __launch_bounds__(kThreads) void dora_dm_partial_kernel(const T* __restrict__ dY, int64_t lddy,
                                                                   const T* __restrict__ Y, int64_t ldy,
                                                                   const T* __restrict__ bias, float* __restrict__ partial,
                                                                   int n, int O, int rows_per_slice) {
  __shared__ float part[16][128];
  using V4 = __attribute__((__vector_size__(4 * sizeof(int)))) int;
  const int rr = threadIdx.x >> 4, cg = threadIdx.x & 15;
  const int j0 = blockIdx.x * 128 + cg * 8;
  const bool col_ok = j0 < O;
  float acc[8], bj[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    acc[e] = 0.f;
    bj[e] = (bias != nullptr && col_ok) ? (float)bias[j0 + e] : 0.f;
  }
  const int t0 = blockIdx.y * rows_per_slice;
  int t1 = t0 + rows_per_slice;
  if (t1 > n) t1 = n;
  if (col_ok) {
#pragma unroll 4
    for (int t = t0 + rr; t < t1; t += 16) {
      const V4 a = *reinterpret_cast<const V4*>(dY + (int64_t)t * lddy + j0);
      const V4 y = *reinterpret_cast<const V4*>(Y + (int64_t)t * ldy + j0);
      const T* a8 = reinterpret_cast<const T*>(&a);
      const T* y8 = reinterpret_cast<const T*>(&y);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += (float)a8[e] * ((float)y8[e] - bj[e]);
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[rr][cg * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < 128) {
    const int j = blockIdx.x * 128 + threadIdx.x;
    float sum = part[0][threadIdx.x];
#pragma unroll
    for (int q = 1; q < 16; ++q) sum += part[q][threadIdx.x];
    if (j < O) partial[(int64_t)blockIdx.y * O + j] = sum;
  }
}

// dm[j] = the column's slices / m[j]: 64 columns per workgroup, slices q, q + 4, ... per group of 64 threads, groups in order.
// With R > 0 also out = in diag(g): the workgroups beyond the first of a column group (blockIdx.y) scale 16 rows of dB~ each (as a launch
// of its own 4.8 us next to this one's 4.2, both of them latency; by the first workgroup, behind its sums, 7 us more at r 128).
template <typename T>
__global__ __launch_bounds__(kThreads) void dora_dm_finish_kernel(const float* __restrict__ partial, int rows,
                                                                  const T* __restrict__ m, T* __restrict__ dm, int O, const T* in,
                                                                  int64_t ldi, const float* __restrict__ g, T* out, int64_t ldo, int R) {
  __shared__ float part[4][64];
  const int jj = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + jj;
  if (blockIdx.y > 0) {
    if (j >= O) return;
    const int k0 = ((int)blockIdx.y - 1) * 16 + q;
    const float gj = g[j];
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = k0 + 4 * u < R ? (float)in[(int64_t)(k0 + 4 * u) * ldi + j] * gj : 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      asm("" : "+v"(v[u]));  // rounded to fp32 and then to T, as by dora_colscale_kernel (f16: not by one instruction from the operands)
      if (k0 + 4 * u < R) out[(int64_t)(k0 + 4 * u) * ldo + j] = (T)v[u];
    }
    return;
  }
  float sum = 0.f;
  if (j < O) {
#pragma unroll 8
    for (int y = q; y < rows; y += 4) sum += partial[(int64_t)y * O + j];
  }
  part[q][jj] = sum;
  __syncthreads();
  if (q == 0 && j < O) dm[j] = (T)((((part[0][jj] + part[1][jj]) + part[2][jj]) + part[3][jj]) / (float)m[j]);
}

int rows_per_slice(int64_t n, int64_t o) {
  const int64_t gx = (o + 127) / 128;
  int64_t slices = 1024 / gx;  // about four workgroups per compute unit
  if (slices < 1) slices = 1;
  int64_t rows = (n + slices - 1) / slices;
  rows = (rows + 15) / 16 * 16;
  if (rows < 64) rows = 64;
  return (int)rows;
}

template <typename T>
hipError_t dm_t(const void* dY, int64_t lddy, const void* Y, int64_t ldy, const void* bias, const void* m, float* partial,
                void* dm, int64_t n, int64_t o, const ColScale& b, hipStream_t s) {
  const int rows = rows_per_slice(n, o), slices = dora_dm_slices(n, o);
  hipLaunchKernelGGL(dora_dm_partial_kernel<T>, dim3((unsigned)((o + 127) / 128), (unsigned)slices), dim3(kThreads), 0, s,
                     static_cast<const T*>(dY), lddy, static_cast<const T*>(Y), ldy, static_cast<const T*>(bias), partial,
                     (int)n, (int)o, rows);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned scalers = b.out != nullptr ? (unsigned)((b.R + 15) / 16) : 0u;
  hipLaunchKernelGGL(dora_dm_finish_kernel<T>, dim3((unsigned)((o + 63) / 64), 1 + scalers), dim3(kThreads), 0, s, partial,
                     slices, static_cast<const T*>(m), static_cast<T*>(dm), (int)o, static_cast<const T*>(b.in), b.ldi, b.g,
                     static_cast<T*>(b.out), b.ldo, b.out != nullptr ? (int)b.R : 0);
  return hipGetLastError();
}

template <typename T>
hipError_t colscale_t(const void* in, int64_t ldi, const float* g, void* out, int64_t ldo, int64_t R, int64_t O, hipStream_t s) {
  if (R > 65535) return hipErrorInvalidValue;  // r <= 128 here
  hipLaunchKernelGGL(dora_colscale_kernel<T>, dim3((unsigned)((O / 8 + kThreads - 1) / kThreads), (unsigned)R), dim3(kThreads), 0, s,
                     static_cast<const T*>(in), ldi, g, static_cast<T*>(out), ldo, (int)R, (int)O);
  return hipGetLastError();
}

}  // namespace

int dora_dm_slices(int64_t n, int64_t o) {
  const int rows = rows_per_slice(n, o);
  return (int)((n + rows - 1) / rows);
}

hipError_t dora_scale_run(int dtype, const float* partial, int rows, const void* m, float* c, float* g, const void* in, int64_t ldi,
                          void* out, int64_t ldo, int64_t R, int64_t O, hipStream_t stream) {
  const dim3 grid((unsigned)((O + 63) / 64));
  if (dtype == DT_F16)
    hipLaunchKernelGGL(dora_scale_kernel<_Float16>, grid, dim3(kThreads), 0, stream, partial, rows, static_cast<const _Float16*>(m), c, g,
                       static_cast<const _Float16*>(in), ldi, static_cast<_Float16*>(out), ldo, (int)R, (int)O);
  else if (dtype == DT_BF16)
    hipLaunchKernelGGL(dora_scale_kernel<__bf16>, grid, dim3(kThreads), 0, stream, partial, rows, static_cast<const __bf16*>(m), c, g,
                       static_cast<const __bf16*>(in), ldi, static_cast<__bf16*>(out), ldo, (int)R, (int)O);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t dora_colscale_run(int dtype, const void* in, int64_t ldi, const float* g, void* out, int64_t ldo, int64_t R,
                             int64_t O, hipStream_t stream) {
  if (dtype == DT_F16) return colscale_t<_Float16>(in, ldi, g, out, ldo, R, O, stream);
  if (dtype == DT_BF16) return colscale_t<__bf16>(in, ldi, g, out, ldo, R, O, stream);
  return hipErrorInvalidValue;
}

hipError_t dora_dm_run(int dtype, const void* dY, int64_t lddy, const void* Y, int64_t ldy, const void* bias, const void* m,
                       float* partial, void* dm, int64_t n, int64_t o, const ColScale& b, hipStream_t stream) {
  if (dtype == DT_F16) return dm_t<_Float16>(dY, lddy, Y, ldy, bias, m, partial, dm, n, o, b, stream);
  if (dtype == DT_BF16) return dm_t<__bf16>(dY, lddy, Y, ldy, bias, m, partial, dm, n, o, b, stream);
  return hipErrorInvalidValue;
}

}  // namespace rl
