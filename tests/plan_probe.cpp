// Prints what the library's host code plans for the products and layers named on stdin (tests/test_plans.py); links librunlora.so,
// runs nothing on a GPU.
#include <cstdio>
#include <cstring>

#include "../paper_2312_03415_amd/csrc/gemm.hpp"

using namespace rl;

int main() {
  char kind[16];
  long M, N, K0, K1;
  while (std::scanf("%15s %ld %ld %ld %ld", kind, &M, &N, &K0, &K1) == 5) {
    if (std::strcmp(kind, "product") == 0) {  // the plan, its modelled time, and that of the generic engine's tiles for the shape
      const GemmPlan p = gemm_plan(DT_BF16, M, N, K0, K1);
      const GemmPlan f = gemm_plan(DT_F32, M, N, K0, K1);  // (the rule by tile counts names its shape for fp32 too)
      const GemmPlan g = gemm_plan(DT_BF16, M, N, K0, K1, f.cfg == CFG_BIG ? CFG_MC4 : f.cfg);
      std::printf("%d %d %ld %zu %.3f %d %.3f\n", p.cfg, p.splits, (long)p.tail_n0, p.partial_bytes, plan_time_us(p, M, N, K0, K1), g.cfg, plan_time_us(g, M, N, K0, K1));
    }
  }
  return 0;
}
