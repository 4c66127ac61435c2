#define RL_T __bf16
#define RL_BK 64
#define RL_FN gemm_launch_bf16
#define RL_SKINNY_FN skinny_launch_bf16
#define RL_MERGE_FN merge_launch_bf16
#define RL_PAIR_FN mt_pair_launch_bf16
#define RL_PAIR_REDUCE_FN skinny_reduce_launch_bf16
#define RL_FINISH_FN finish_launch_bf16
#define RL_PIPE 1
#include "gemm_launch.inc"
