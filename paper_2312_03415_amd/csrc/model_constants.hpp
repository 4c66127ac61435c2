// Constants of the selector's time model, measured on one MI355X with this library's own kernels.
// The values below are GENERATED by `python -m paper_2312_03415_amd.calibrate` (run on the GPU); regenerate after
// changing a kernel.  Times in microseconds, rates in TB/s.  Not among them: the launch models that choose tile shapes, K splits
// and routes (launch_model, few_time_us, skinny_time_us, rank_time_us, split_time_us, int4_direct_us in gemm_host.hip), fitted by
// hand to the sweeps that their comments describe.  The 256x256 kernel has a price in both: here at the power-limited rate of
// long runs, for comparing graphs, there for one product, for comparing tile shapes.
#pragma once
#include "gemm.hpp"

namespace rl {

struct TileModel {
  double tk_us[3];   // time of one K tile of a full round of workgroups, per layout NN / NT / TN
  double tfix_us;    // prologue + epilogue of a round
  double tfix_d_us;  // same with an addend D
  int wg_per_cu;     // workgroups resident per compute unit
};

struct ModelConstants {
  TileModel tile[2][CFG_STREAM];  // [0] = bf16/fp16, [1] = fp32 (the middle-sized kernel's: launch_time_us, gemm.hpp)
  double stream_tbps[2];         // streaming kernel, big operand row-major / stored [K,M]
  double stream_fix_us;          // its fixed cost per launch
  double reduce_tbps;            // second stage of a split contraction: rate over the partials' round trip
  double reduce_fix_us;          // its fixed cost beyond the launch
  double launch_us;              // fixed cost per kernel launch seen by the caller
  double merge_tbps;             // M = W + A B kernel: rate over 2 i o e bytes, W from HBM behind dirty caches, as in a model
  double merge_fix_us;           // its fixed cost
  double merge_r64_us, merge_r128_us;  // what it takes longer at r 64 and 128 than at 32 (4096 x 4096)
};

inline const ModelConstants& model_constants() {
  static const ModelConstants c = {
      {
       {
           {{2.433, 2.385, 2.337}, 11.29, 21.40, 1},  // 256x256
           {{1.394, 1.297, 1.361}, 6.56, 13.95, 2},  // 128x128
           {{0.929, 0.888, 0.966}, 3.77, 4.69, 3},  // 128x32
           {{0.836, 0.814, 0.913}, 5.01, 7.56, 2},  // 128x64
           {{0.892, 0.864, 0.964}, 4.61, 5.81, 3},  // 32x128
           {{1.322, 1.249, 1.390}, 6.41, 9.01, 3},  // 64x128
           {{0.761, 0.815, 0.749}, 10.42, 24.75, 1},  // 256x256x32 matrix-core (id 6)
           {{1.564, 1.509, 1.540}, 8.46, 22.88, 1},  // 256x256x64 matrix-core (id 7)
       },
       {
           {{8.280, 7.804, 7.854}, 20.72, 56.18, 1},  // 256x256
           {{4.433, 4.203, 4.354}, 6.92, 12.65, 2},  // 128x128
           {{2.037, 2.012, 2.132}, 4.29, 5.27, 3},  // 128x32
           {{2.349, 2.361, 2.459}, 4.83, 9.43, 2},  // 128x64
           {{2.078, 1.984, 2.110}, 4.59, 4.87, 3},  // 32x128
           {{3.455, 3.375, 3.495}, 6.61, 7.79, 3},  // 64x128
           {{8.280, 7.804, 7.854}, 20.72, 56.18, 1},  // 256x256x32 matrix-core (id 6)
           {{8.280, 7.804, 7.854}, 20.72, 56.18, 1},  // 256x256x64 matrix-core (id 7)
       }},
      {5.42, 3.30},
      3.03,
      5.58,
      2.75,
      6.44,
      3.96,
      5.48,
      11.04,
      8.04,
  };
  return c;
}

}  // namespace rl
