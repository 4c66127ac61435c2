// Element-wise kernels of the VeRA layer (see vera.hpp): the scaled factor B~ = diag(d) B diag(b) and the
// reduction of dB~ into the gradients of d and b.  Bound by nothing that matters: r x o elements.
#include "vera.hpp"

#include "gemm.hpp"

namespace rl {
namespace {

constexpr int kThreads = 256;

// 16 bytes of a row as VE elements (row lengths are multiples of VE, rows 16-byte aligned)
template <typename T>
struct Chunk {
  static constexpr int VE = 16 / (int)sizeof(T);
  using V4 = __attribute__((__vector_size__(4 * sizeof(int)))) int;
  T e[VE];
  __device__ __forceinline__ void load(const T* p) { *reinterpret_cast<V4*>(e) = *reinterpret_cast<const V4*>(p); }
  __device__ __forceinline__ void store(T* p) const { *reinterpret_cast<V4*>(p) = *reinterpret_cast<const V4*>(e); }
};

// A thread scales 16 bytes of a row (256 x 8192: 6.6 us with an element per thread, 5.2 so).
template <typename T>
__global__ __launch_bounds__(kThreads) void vera_scale_kernel(const T* __restrict__ B, int64_t ldb, const T* __restrict__ d,
                                                              const T* __restrict__ b, T* __restrict__ Bt, int64_t ldt,
                                                              int R, int O) {
  constexpr int VE = Chunk<T>::VE;
  const int j = (blockIdx.x * kThreads + threadIdx.x) * VE;
  const int k = blockIdx.y;
  if (j >= O || k >= R) return;
  Chunk<T> v, w;
  v.load(B + (int64_t)k * ldb + j);
  w.load(b + j);
  const float dk = (float)d[k];
#pragma unroll
  for (int e = 0; e < VE; ++e) v.e[e] = (T)(dk * (float)v.e[e] * (float)w.e[e]);
  v.store(Bt + (int64_t)k * ldt + j);
}

// Both gradients in one launch (two of 5.3 and 4.0 us at 256 x 8192, each of them latency): workgroups [0, db_wgs) sum columns, the
// others rows.  Either part may be absent.
// db: a workgroup owns 32 columns; thread (c, g) sums the rows k = g, g + 8, g + 16, ... of column c in that order, then the eight
// partial sums of a column are added in the order of g.
// dd: one workgroup per row k: every thread sums its 16-byte chunks tid, tid + 256, ... in order, then a fixed binary tree over the
// 256 partial sums (256 x 8192: 12 us with two bytes per load, 4.8 so).
template <typename T>
__global__ __launch_bounds__(kThreads) void vera_grad_kernel(const T* __restrict__ G, int64_t ldg, const T* __restrict__ B, int64_t ldb,
                                                             const T* __restrict__ d, const T* __restrict__ b, T* __restrict__ dd,
                                                             T* __restrict__ db, int R, int O, int db_wgs) {
  __shared__ float part[kThreads];
  if ((int)blockIdx.x < db_wgs) {
    const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int j = blockIdx.x * 32 + c;
    float acc = 0.f;
    if (j < O) {
#pragma unroll 4
      for (int k = g; k < R; k += 8) acc += (float)G[(int64_t)k * ldg + j] * ((float)d[k] * (float)B[(int64_t)k * ldb + j]);
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    if (g == 0 && j < O) {
      float sum = part[c];
#pragma unroll
      for (int q = 1; q < 8; ++q) sum += part[32 * q + c];
      db[j] = (T)sum;
    }
    return;
  }
  constexpr int VE = Chunk<T>::VE;
  const int k = (int)blockIdx.x - db_wgs;
  float acc = 0.f;
#pragma unroll 4
  for (int j = (int)threadIdx.x * VE; j < O; j += kThreads * VE) {
    Chunk<T> x, y, w;
    x.load(G + (int64_t)k * ldg + j);
    y.load(B + (int64_t)k * ldb + j);
    w.load(b + j);
#pragma unroll
    for (int e = 0; e < VE; ++e) acc += (float)x.e[e] * ((float)y.e[e] * (float)w.e[e]);
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) dd[k] = (T)part[0];
}

template <typename T>
hipError_t scale_t(const void* B, int64_t ldb, const void* d, const void* b, void* Bt, int64_t ldt, int64_t R, int64_t O,
                   hipStream_t s) {
  // gridDim.y is limited to 65535: walk the rows in slabs
  for (int64_t k0 = 0; k0 < R; k0 += 65535) {
    const int rows = (int)((R - k0) < 65535 ? (R - k0) : 65535);
    dim3 grid((unsigned)((O / Chunk<T>::VE + kThreads - 1) / kThreads), (unsigned)rows);
    hipLaunchKernelGGL(vera_scale_kernel<T>, grid, dim3(kThreads), 0, s, static_cast<const T*>(B) + k0 * ldb, ldb,
                       static_cast<const T*>(d) + k0, static_cast<const T*>(b), static_cast<T*>(Bt) + k0 * ldt, ldt, rows, (int)O);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
hipError_t grad_t(const void* G, int64_t ldg, const void* B, int64_t ldb, const void* d, const void* b, void* dd, void* db,
                  int64_t R, int64_t O, hipStream_t s) {
  const int64_t db_wgs = db ? (O + 31) / 32 : 0, dd_wgs = dd ? R : 0;
  if (db_wgs + dd_wgs == 0) return hipSuccess;
  hipLaunchKernelGGL(vera_grad_kernel<T>, dim3((unsigned)(db_wgs + dd_wgs)), dim3(kThreads), 0, s, static_cast<const T*>(G), ldg,
                     static_cast<const T*>(B), ldb, static_cast<const T*>(d), static_cast<const T*>(b), static_cast<T*>(dd),
                     static_cast<T*>(db), (int)R, (int)O, (int)db_wgs);
  return hipGetLastError();
}

}  // namespace

hipError_t vera_scale_run(int dtype, const void* B, int64_t ldb, const void* d, const void* b, void* Bt, int64_t ldt,
                          int64_t R, int64_t O, hipStream_t stream) {
  switch (dtype) {
    case DT_F32: return scale_t<float>(B, ldb, d, b, Bt, ldt, R, O, stream);
    case DT_F16: return scale_t<_Float16>(B, ldb, d, b, Bt, ldt, R, O, stream);
    default: return scale_t<__bf16>(B, ldb, d, b, Bt, ldt, R, O, stream);
  }
}

hipError_t vera_grad_run(int dtype, const void* G, int64_t ldg, const void* B, int64_t ldb, const void* d,
                         const void* b, void* dd, void* db, int64_t R, int64_t O, hipStream_t stream) {
  switch (dtype) {
    case DT_F32: return grad_t<float>(G, ldg, B, ldb, d, b, dd, db, R, O, stream);
    case DT_F16: return grad_t<_Float16>(G, ldg, B, ldb, d, b, dd, db, R, O, stream);
    default: return grad_t<__bf16>(G, ldg, B, ldb, d, b, dd, db, R, O, stream);
  }
}

}  // namespace rl
