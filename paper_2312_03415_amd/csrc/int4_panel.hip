// A panel of a 4-bit frozen weight written out densely in scratch (see int4_panel_plan, gemm.hpp): rows [r0, r0 + rows) and
// columns [c0, c0 + cols) of W, dequantised exactly as the GEMMs that read the packed form do it (q * scale in fp32, one
// rounding to the activation type).
//
// Why: the kernels that dequantise on their way to LDS spend their issue slots and load slack on it (0.93-1.05 PFLOP/s against
// 1.3-1.4 on dense operands).  Layer 4096 x 5120 -> 13824, r 64: Y = X W 683 us direct, 560 in panels of 4096 columns; dX
// 650 and 564 (panels of 2048 rows).
// Bound by HBM: a quarter of the panel's bytes read, all of them written (42 MB in 14 us; 16 with 32 rows per wave).  A thread owns eight
// columns (one packed dword, 16 bytes out) of kRun rows of one 64-row group, so that its eight scales are fetched once; a
// wave covers 256 packed bytes and 1 KB of the panel per row.
#include "gemm.hpp"
#include "gemm_engine.hpp"

namespace rl {
namespace {

constexpr int kRun = 16;  // rows per wave

template <typename T>
__global__ __launch_bounds__(256) void int4_panel_kernel(const unsigned char* __restrict__ W, int64_t ldw, const _Float16* __restrict__ scales,
                                                         int64_t lds, T* __restrict__ out, int64_t ldo, int r0, int rows, int c0, int cols) {
  const int col = ((int)blockIdx.x * 64 + (int)(threadIdx.x & 63)) * 8;
  // four waves: four runs of kRun rows, aligned to the scale groups (r0 need not be)
  const int first = r0 / kRun * kRun + ((int)blockIdx.y * 4 + (int)(threadIdx.x >> 6)) * kRun;
  if (col >= cols || first >= r0 + rows) return;
  const int lo = first > r0 ? first : r0, hi = first + kRun < r0 + rows ? first + kRun : r0 + rows;
  const i32x4 sc = *reinterpret_cast<const i32x4*>(scales + (int64_t)(first / 64) * lds + c0 + col);
#pragma unroll 8
  for (int k = lo; k < hi; ++k) {
    const uint32_t w = *reinterpret_cast<const uint32_t*>(W + (((int64_t)k * ldw + c0 + col) >> 1));
    *reinterpret_cast<i32x4*>(out + (int64_t)(k - r0) * ldo + col) = dequant_chunk<T>(w, sc);
  }
}

}  // namespace

hipError_t int4_panel_run(int dtype, const void* W, int64_t ldw, const void* scales, int64_t lds, void* out, int64_t ldo, int64_t r0,
                          int64_t rows, int64_t c0, int64_t cols, hipStream_t stream) {
  if (rows < 1 || cols < 1 || cols % 8 != 0 || c0 % 8 != 0) return hipErrorInvalidValue;
  const int64_t runs = (r0 + rows + kRun - 1) / kRun - r0 / kRun;
  const dim3 grid((unsigned)((cols / 8 + 63) / 64), (unsigned)((runs + 3) / 4));
  const unsigned char* w = static_cast<const unsigned char*>(W);
  const _Float16* s = static_cast<const _Float16*>(scales);
  if (dtype == DT_BF16)
    launch_timed(int4_panel_kernel<__bf16>, grid, dim3(256), 0, stream, w, ldw, s, lds, static_cast<__bf16*>(out), ldo, (int)r0, (int)rows, (int)c0, (int)cols);
  else if (dtype == DT_F16)
    launch_timed(int4_panel_kernel<_Float16>, grid, dim3(256), 0, stream, w, ldw, s, lds, static_cast<_Float16*>(out), ldo, (int)r0, (int)rows, (int)c0, (int)cols);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace rl
