// Constants of the selector's time model, measured on one MI355X with this library's own kernels.
// GENERATED by `python -m paper_2312_03415_amd.calibrate` (run on the GPU); regenerate after
// changing a kernel.  Times in microseconds, rates in TB/s.
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
  double merge_tbps;             // M = W + A B kernel: rate over 2 i o e bytes
  double merge_fix_us;           // its fixed cost
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
      3.60,  // (W from HBM, as in a model; 4.95 while the Infinity Cache holds part of it)
      2.52,
  };
  return c;
}

}  // namespace rl
