// Host-side interface of the tile GEMM engine (gemm_engine.hpp): problem description, launch plan
// (tile shape + split of the contraction) and launch.  Internal to the library.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>

namespace rl {

enum { DT_F32 = 0, DT_F16 = 1, DT_BF16 = 2 };

// C[M,N] (dtype) = sum_s op(A_s) op(B_s) (+ D).
struct GemmDesc {
  int dtype = DT_BF16;
  int a_strided = 0;  // 0: A_s stored [M,K_s] row-major; 1: A_s stored [K_s,M]
  int b_kcontig = 0;  // 0: B_s stored [K_s,N] row-major; 1: B_s stored [N,K_s]
  int64_t M = 0, N = 0;
  int nseg = 1;
  const void* A[2] = {nullptr, nullptr};
  const void* B[2] = {nullptr, nullptr};
  int64_t lda[2] = {0, 0}, ldb[2] = {0, 0}, K[2] = {0, 0};
  void* C = nullptr;
  int64_t ldc = 0;
  const void* D = nullptr;  // optional addend, same dtype as C (may alias C)
  int64_t ldd = 0;
  bool has_addend = false;  // an addend is part of the product (also set when only shapes are modelled and D is null)
  // B[0] is symmetric int4 (packed nibbles, ldb[0] in elements) with fp16 group scales
  // [rows/64, ldbs]; nullptr = dense.  16-bit types, A stored [M,K].
  const void* Bscale = nullptr;
  int64_t ldbs = 0;
  bool b_int4 = false;  // B[0] is int4 (set together with Bscale; also when only shapes are modelled)
  // C = alpha * (sum of the products) + D + bias;  bias: row vector [N] of the dtype, or nullptr
  float alpha = 1.f;
  const void* bias = nullptr;
  // LoRA dropout (drop_thr != 0): zero output element (m, n) of alpha * (the products) where the mask
  // drops element (m, n) of X; key and threshold as in gemm_engine.hpp, drop_cpr = columns of X / 4
  uint32_t drop_thr = 0, drop_key = 0, drop_cpr = 0;
  // the mask applies to segment 0's product alone, C = mask o (A[0] B[0]) + A[1] B[1] (GemmArgs::mask_seg0), with drop_n4 =
  // (first column of C in X) / 4; where masked_segment_ok holds
  bool mask_seg0 = false;
  uint32_t drop_n4 = 0;
  // A[0] is X with its dropped elements zeroed (GemmArgs::mask_a): rank-r products on the middle-sized kernel (rank_plan)
  bool mask_a = false;
  // optional [N] (16-byte aligned): C = (the products) diag(cscale) + bias; where column_scale_ok holds
  const float* cscale = nullptr;
  // One-pass LoRA forward, C = A[0] B[0] + round(t_alpha A[0] LA) B[1] in one kernel: nseg = 2, A[1] unused,
  // K[1] = R <= kFuseMaxR, LA stored [K[0], R] row-major; A [M,K], B [K,N], dense B, no addend, no K split
  // (plan with gemm_plan_fused).  fuse_t is also set when only shapes are modelled and LA is null.
  const void* LA = nullptr;
  int64_t ldla = 0;
  float t_alpha = 1.f;
  bool fuse_t = false;
  int rotate = 0;  // see GemmArgs::rotate (middle-sized kernel only)
};
constexpr int64_t kFuseMaxR = 32;

enum TileCfg {
  CFG_BIG = 0, CFG_MID, CFG_TALL32, CFG_TALL64, CFG_WIDE32, CFG_WIDE64,
  CFG_MC3,  // matrix-core kernel (gemm_mc.hpp, 16-bit types): 256x256x32, 4 waves, 3-stage LDS ring, 32x32x16 products
            // (the int4 route of the frozen weight runs here)
  CFG_MC4,  // matrix-core kernel (gemm_mc64.hpp, 16-bit types): 256x256x64, 4 waves, 2 LDS stages, 16x16x32 products
            // (the id the heuristics pick for dense B)
  CFG_STREAM,  // id of the streaming kernel in rl_gemm_t (8); 8..11 name the streaming and merge kernels in profile records
  // middle-sized matrix-core kernel (gemm_mt.hpp, 16-bit types): K tile 64, 4 waves, 16x16x32 products
  CFG_MT128 = 12,  // 128x128, 2 LDS stages, two workgroups per compute unit
  CFG_MT128D,      // 128x128, 4 LDS stages, one workgroup per compute unit
  CFG_MT256,       // 256x128, 3 LDS stages, one workgroup per compute unit
  CFG_MTN64,       // 128x64, 3 LDS stages, two workgroups per compute unit
  CFG_MTM64,       // 64x128, 3 LDS stages, two workgroups per compute unit
  CFG_COUNT
};
inline bool cfg_is_mt(int cfg) { return cfg >= CFG_MT128 && cfg < CFG_COUNT; }
inline bool cfg_is_tile(int cfg) { return cfg >= 0 && cfg < CFG_COUNT && (cfg < CFG_STREAM || cfg_is_mt(cfg)); }

struct GemmPlan {
  int cfg = CFG_MID;
  int bm = 128, bn = 128, bk = 64;
  int nbm = 1, nbn = 1;
  int splits = 1;            // > 1: fp32 partials + fixed-order reduce
  int tiles_per_split = 1;
  // scratch to provide for partials (of the launch or of the tail launch); may be more than the plan uses (gemm_plan)
  size_t partial_bytes = 0;
  // > 0: the output columns [tail_n0, N) are a launch of their own, planned by gemm_plan on that
  // sub-problem (a few tiles with the contraction split), so that the main launch is whole rounds of
  // one tile per compute unit instead of ending on a mostly idle round
  int64_t tail_n0 = 0;
  int tail_cfg = -1, tail_splits = 0;  // that launch's tile shape and K split
};

// Tile shape and K split for a problem; depends on shapes and dtype only (never on pointers), so
// the same plan sizes the workspace and drives the launch.  force_cfg / force_splits (>= 0 / > 0)
// override the heuristics (used by the tuning sweeps and tests).
// long_operand: see long_operand below.
GemmPlan gemm_plan(int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1, int force_cfg = -1,
                   int force_splits = 0, bool b_int4 = false, bool long_operand = false);
// For fp32 gemm_plan goes by tile counts (forward 3 takes its shape from there); a product of its own runs on the tile shape and
// K split that this picks by modelled time, in the scratch of that plan.
void gemm_plan_f32(GemmPlan* plan, int64_t M, int64_t N, int64_t K0, int64_t K1);
// An operand beyond what the middle-sized kernel addresses (31-bit byte offsets; the 256x256 kernel takes twice that): the
// product keeps the plan by tile counts (same scratch).
bool long_operand(const GemmDesc& d);
// A plan whose kernels are built with a masked first segment: dense 16-bit operands, A [M,K], B [N,K], no addend, scale or bias.
bool masked_segment_ok(const GemmDesc& d, const GemmPlan& p);
// A plan whose kernels are built with a column scale: dense 16-bit operands, A [M,K], B [K,N], no addend, scale or mask, no split.
bool column_scale_ok(const GemmDesc& d, const GemmPlan& p);

// Modelled time in us of one launch of a 16-bit tile GEMM (CFG_MT*, CFG_MC4, and the generic engine's 128x128, 128x64 and
// 64x128 tiles): nbm x nbn output tiles x K slices of `ktiles` K tiles each; odd = odd_lines of the product.
double launch_time_us(int cfg, int64_t nbm, int64_t nbn, int splits, int64_t ktiles, double odd);
// Share of a 16-bit product's operands whose rows are not whole 128-byte lines, as far as its sizes tell (rows of K and of N
// elements).
inline double odd_lines(int64_t N, int64_t K) { return 0.5 * (K % 64 != 0) + 0.5 * (N % 64 != 0); }
// Modelled time of a plan for a 16-bit product with dense operands (its tail launch and reduce passes included).
double plan_time_us(const GemmPlan& p, int64_t M, int64_t N, int64_t K0, int64_t K1);
// Modelled time of the partials' round trip and the reduce pass behind a contraction split `splits` ways.
double split_time_us(int64_t M, int64_t N, int splits);

// Plan for the one-pass LoRA forward (GemmDesc::fuse_t): a tile shape of the generic engine, the contraction whole.
GemmPlan gemm_plan_fused(int dtype, int64_t M, int64_t N, int64_t K0, int64_t R);

// Plan of the launch that computes the columns [main.tail_n0, N) cut off from `main`.
GemmPlan gemm_tail_plan(const GemmPlan& main, int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1);

// Plan for a product whose B[0] is int4 (GemmDesc::Bscale): matrix-core kernel or the generic
// engine's 128x128 tile.
GemmPlan gemm_plan_int4(int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1);

// A product whose B[0] is int4, with W's columns (rows, for dY W^T) dequantised panel by panel into scratch and multiplied
// by the dense kernels: at most kInt4PanelBytes of it at a time.  Applies where the model says
// it beats the kernels that dequantise on their way to LDS (int4_panel.hip).
constexpr size_t kInt4PanelBytes = 64u << 20;
struct Int4PanelPlan {
  int64_t width = 0;        // output columns per panel; 0 = the route does not apply
  GemmPlan full, last;      // products of a full panel and of the last one
  size_t panel_bytes = 0;   // scratch of a panel; the products' partials come behind it
  size_t scratch_bytes = 0;
  double us = 0;
};
Int4PanelPlan int4_panel_plan(int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1);
hipError_t int4_panel_gemm(const GemmDesc& d, const Int4PanelPlan& plan, void* scratch, hipStream_t stream);
hipError_t int4_panel_run(int dtype, const void* W, int64_t ldw, const void* scales, int64_t lds, void* out, int64_t ldo, int64_t r0,
                          int64_t rows, int64_t c0, int64_t cols, hipStream_t stream);

// Enqueue the product.  `scratch` must hold plan.partial_bytes when plan.splits > 1.
hipError_t gemm_run(const GemmDesc& d, const GemmPlan& plan, float* scratch, hipStream_t stream);

// ---- few-token forward: Y = X W + (t_alpha X A) B + bias in two launches (lora_finish.hpp), 16-bit, dense W -------
struct FewDesc {
  const void *X = nullptr, *W = nullptr, *A = nullptr, *B = nullptr, *bias = nullptr;
  void *Y = nullptr, *T = nullptr;  // T: [n, r] buffer to leave t_alpha X A in, or nullptr
  int64_t ldx = 0, ldw = 0, lda = 0, ldb = 0, ldy = 0, ldt = 0;
  int64_t n = 0, i = 0, o = 0, r = 0;
  float t_alpha = 1.f;
};
struct FewPlan {
  int splits = 0;  // K slices; 0 = the route does not apply
  int tiles_per_split = 0;
  double us = 0;   // modelled time
};
constexpr int64_t kFewMaxRows = 256, kFewMaxR = 128;
// What launch_time_us lacks for few rows, us per MB of X and W from HBM, and few_time_us does not: added to the launches that the route is
// compared with, and taken off its own price where it stands beside launches priced without it (the selector's).
constexpr double kColdUsPerMB = 0.03;
// scratch_bytes: what the call has for partials whatever route it takes
FewPlan few_plan(int64_t n, int64_t i, int64_t o, int64_t r, size_t scratch_bytes);
hipError_t few_run(int dtype, const FewDesc& d, const FewPlan& plan, float* scratch, hipStream_t stream);

// ---- streaming kernel for the rank-r products (skinny.hpp) --------------------------------------
// C[M,N<=128] = op(A)[M,K] op(B)[K,N], optionally stored transposed; up to two problems per launch.
struct SkinnyDesc {
  const void* A = nullptr;
  const void* B = nullptr;
  void* C = nullptr;
  int64_t lda = 0, ldb = 0, ldc = 0;
  int64_t M = 0, N = 0, K = 0;
  int a_strided = 0, b_kcontig = 0, trans_out = 0;
  float alpha = 1.f;  // C = alpha * op(A) op(B)
  uint32_t drop_thr = 0, drop_key = 0, drop_cpr = 0;  // != 0: A is X, masked by LoRA dropout on load
};
struct SkinnyPlan {
  int rt = 1;      // 32-column blocks per row block: N <= 32*rt
  int splits = 1;  // K split over workgroups (fp32 partials + ordered reduce)
  int mr = 1;      // 32-row blocks per workgroup: 2 for paired launches in the [K,M] orientation with N <= 64
  int nwv = 4;     // wavefronts per workgroup
  size_t partial_bytes = 0;
};
inline bool skinny_ok(int64_t N) { return N <= 128; }
SkinnyPlan skinny_plan(int dtype, int nprob, const SkinnyDesc* d, size_t cap = ~(size_t)0);  // cap: partials may take so much
// modelled time of that launch (and its reduce pass) in us
double skinny_time_us(int dtype, int nprob, const SkinnyDesc* d, const SkinnyPlan& plan);

// ---- rank-r products with r > 32 on the middle-sized matrix-core kernel, 16-bit types ------------------
// One product (gemm_run with the plan) or two in one launch (mt_pair_run); `cap` = scratch bytes the plan may use, slice_us = what
// slices cost besides.  False where the streaming kernel is modelled faster.
bool rank_plan(int dtype, const SkinnyDesc& d, size_t cap, GemmPlan* plan, double* plan_us = nullptr, double slice_us = 0.0);
GemmDesc rank_desc(int dtype, const SkinnyDesc& d);  // the product as gemm_run takes it
struct MtPairPlan {
  int cfg[2] = {0, 0};  // CFG_MTN64 / CFG_MTM64
  bool wide = false;    // 128x128 tiles for both instead
  int splits[2] = {1, 1}, tiles_per_split[2] = {0, 0};
  size_t partial_bytes = 0;
  double us = 0;
};
// alone_us: what the two take otherwise (0: a launch of the streaming kernel)
bool mt_pair_plan(int dtype, const SkinnyDesc* d, size_t cap, MtPairPlan* plan, double alone_us = 0.0, double slice_us = 0.0);
hipError_t mt_pair_run(int dtype, const SkinnyDesc* d, const MtPairPlan& plan, float* scratch, hipStream_t stream);
hipError_t skinny_run(int dtype, int nprob, const SkinnyDesc* d, const SkinnyPlan& plan, float* scratch,
                      hipStream_t stream);
struct SkinnyArgs;
hipError_t skinny_launch_bf16(int rt, const SkinnyArgs& a, dim3 grid, int splits, hipStream_t s);
hipError_t skinny_launch_f16(int rt, const SkinnyArgs& a, dim3 grid, int splits, hipStream_t s);
hipError_t skinny_launch_f32(int rt, const SkinnyArgs& a, dim3 grid, int splits, hipStream_t s);

// ---- timing of a step's kernels ----------------------------------------------------------------------
// While event pairs are set here (per host thread), every kernel of the step launched from this thread (the tile
// GEMM, a cut-off tail launch, the streaming kernel, the merge kernel and the reduce kernels behind them) is
// launched with the next unused pair bound to its own dispatch, so that the pair's difference is that kernel's
// duration alone, as a kernel trace reports it.  Pair 0 is the step's first (main) kernel.
struct KernelEvents {
  static constexpr int kMax = 16;
  hipEvent_t start[kMax] = {}, stop[kMax] = {};
  int avail = 0, used = 0;
};
extern thread_local KernelEvents g_kernel_events;
template <typename Kern, typename... Args>
inline void launch_timed(Kern kern, dim3 grid, dim3 block, unsigned lds, hipStream_t s, Args... args) {
  KernelEvents& ke = g_kernel_events;
  if (ke.used < ke.avail) {
    hipExtLaunchKernelGGL(kern, grid, block, lds, s, ke.start[ke.used], ke.stop[ke.used], 0, args...);
    ++ke.used;
  } else {
    hipLaunchKernelGGL(kern, grid, block, lds, s, args...);
  }
}

// ---- M = W + A B (merge.hpp): 16-bit types, r <= 128 --------------------------------------------
struct MergeDesc {
  const void *W = nullptr, *A = nullptr, *B = nullptr;
  void* M = nullptr;
  int64_t ldw = 0, lda = 0, ldb = 0, ldm = 0;
  int64_t I = 0, O = 0, R = 0;
  float alpha = 1.f;  // M = W + alpha A B
  int b_trans = 0;    // B stored [O, R]
  const float* wcol = nullptr;  // optional [O]: M = W diag(wcol) + alpha A B
  // optional: store nothing to M; write the squared column sums of W + alpha A B, one row of O floats per
  // row slice (merge_slices; the caller adds them up)
  float* sq_partial = nullptr;
  // drop_thr != 0: M = W + mask o (alpha A B) with the LoRA dropout keep-mask over M's elements (gemm_engine.hpp)
  uint32_t drop_thr = 0, drop_key = 0, drop_cpr = 0;
};
inline bool merge_ok(int dtype, int64_t r) { return dtype != DT_F32 && r <= 128; }
// the merge kernel's launch shape: gx workgroups of 256 columns, gy row slices of bpw 32-row blocks each: as many workgroups as stay on the
// chip together (four to a compute unit up to r = 32, two beyond), so that what each spends on its columns of B is spent once; sums take
// whole slices instead (merge_slices).  1024 and 512 of them, us (bf16, stored V and sums / M, without that): 2048 x 8192 r 16 16.3 and 16.9 / 15.5 and 17.1, 2048 x 2048 r 32 8.1 and 9.3 / 6.7 and 7.1; 1280 x
// 7328 r 64 17.2 and 15.4 / 17.2 and 14.0, 4096 x 4096 r 128 26.8 and 23.9 / 26.7 and 23.3.
inline void merge_grid(int64_t I, int64_t O, int64_t R, int* gx, int* gy, int* bpw) {
  *gx = (int)((O + 255) / 256);
  const int nb = (int)((I + 31) / 32);
  int y = (R <= 32 ? 1024 : 512) / *gx;
  if (y < 1) y = 1;
  if (y > nb) y = nb;
  *bpw = (nb + y - 1) / y;
  *gy = (nb + *bpw - 1) / *bpw;
}
// The row slices that squared column sums are taken over: `rows` of them, of `blocks` 32-row blocks each.  They fix the order in which a column's
// squares are added, and with it the last bits of DoRA's norms, so they do not follow the launch's shape: a workgroup walks one slice each where
// all of them stay on the chip together, and otherwise as many as make up merge_grid's share of rows (DoRA's forward of 64 tokens, us, in
// merge_grid's own shares / so: 1280 x 7328 r 64 29.5 / 29.4, 4096 x 11008 r 64 85.0 / 86.5, 11008 x 4096 r 40, twelve blocks for eleven, 81.6 / 85.2).
inline void merge_slices(int64_t I, int64_t O, int64_t R, int* rows, int* blocks) {
  const int cols = R <= 64 ? 512 : 256;
  const int nb = (int)((I + 31) / 32);
  int y = 512 / (int)((O + cols - 1) / cols);
  if (y < 1) y = 1;
  if (y > nb) y = nb;
  *blocks = (nb + y - 1) / y;
  *rows = (nb + *blocks - 1) / *blocks;
}
hipError_t merge_run(int dtype, const MergeDesc& d, hipStream_t stream);
struct MergeArgs;
hipError_t merge_launch_bf16(const MergeArgs& a, hipStream_t s);
hipError_t merge_launch_f16(const MergeArgs& a, hipStream_t s);

// per-dtype launchers (one translation unit each)
struct GemmArgs;
struct FinishArgs;
struct SkinnyArgs;
hipError_t mt_pair_launch_bf16(int al, int bl0, int bl1, bool wide, const GemmArgs& g0, const GemmArgs& g1, unsigned grid, hipStream_t s);
hipError_t mt_pair_launch_f16(int al, int bl0, int bl1, bool wide, const GemmArgs& g0, const GemmArgs& g1, unsigned grid, hipStream_t s);
hipError_t skinny_reduce_launch_bf16(const SkinnyArgs& a, int splits0, int splits1, hipStream_t s);
hipError_t skinny_reduce_launch_f16(const SkinnyArgs& a, int splits0, int splits1, hipStream_t s);
hipError_t finish_launch_bf16(const FinishArgs& a, hipStream_t s);
hipError_t finish_launch_f16(const FinishArgs& a, hipStream_t s);
hipError_t gemm_launch_bf16(int cfg, int al, int bl, const GemmArgs& a, dim3 grid, hipStream_t s);
hipError_t gemm_launch_f16(int cfg, int al, int bl, const GemmArgs& a, dim3 grid, hipStream_t s);
hipError_t gemm_launch_f32(int cfg, int al, int bl, const GemmArgs& a, dim3 grid, hipStream_t s);
struct DropMask { uint32_t thr = 0, key = 0, cpr = 0; };
hipError_t splitk_reduce_launch(int dtype, const float* partial, int splits, int M, int N, void* C,
                                int64_t ldc, const void* D, int64_t ldd, float alpha, const void* bias,
                                DropMask drop, hipStream_t s);

}  // namespace rl
