// Prints what the library's host code plans for the products and layers named on stdin (tests/test_plans.py); links librunlora.so,
// runs nothing on a GPU.
#include <cstdio>
#include <cstring>

#include "../paper_2312_03415_amd/csrc/schedule.hpp"

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
    } else if (std::strcmp(kind, "padded") == 0) {  // K1 = leading dimension of A [M, K0]: the plan gemm_run gets, and the scratch reported for the shape
      GemmDesc d;
      d.dtype = DT_BF16;
      d.M = M; d.N = N; d.K[0] = K0; d.lda[0] = K1;
      const GemmPlan p = gemm_plan(DT_BF16, M, N, K0, 0, -1, 0, false, long_operand(d));
      std::printf("%d %d %zu %zu\n", p.cfg, p.tail_n0 > 0 ? p.tail_cfg : p.cfg, p.partial_bytes, gemm_plan(DT_BF16, M, N, K0, 0).partial_bytes);
    } else if (std::strcmp(kind, "int4") == 0) {  // panels or not, and the direct kernel's id
      std::printf("%d %d\n", int4_panel_plan(DT_BF16, M, N, K0, K1).width > 0 ? 1 : 0, gemm_plan_int4(DT_BF16, M, N, K0, K1).cfg);
    } else if (std::strncmp(kind, "drop", 4) == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: scratch of forward 1 and backward 1 with dropout
      LayerDims L{M, N, K0, K1, kind[4] == '3' ? DT_F32 : DT_BF16};
      L.drop_thr = 26;
      Schedule f, b;
      if (!build_forward(1, L, FwdOperands{}, nullptr, &f) || !build_backward(1, L, BwdOperands{}, nullptr, &b)) return 1;
      std::printf("%zu %zu\n", f.workspace_bytes, b.workspace_bytes);
    } else if (std::strcmp(kind, "few") == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: the few-token route's price and taken or not
      SkinnyDesc d;
      d.M = M; d.N = K1; d.K = N;
      const GemmPlan g = gemm_plan(DT_BF16, M, K0, N, K1);
      const SkinnyPlan t = skinny_plan(DT_BF16, 1, &d);
      const size_t bytes = t.partial_bytes > g.partial_bytes ? t.partial_bytes : g.partial_bytes;
      const FewPlan f = few_plan(M, N, K0, K1, bytes);
      GemmPlan rank;
      double t_us = 0;
      if (!rank_plan(DT_BF16, d, bytes, &rank, &t_us)) t_us = skinny_time_us(DT_BF16, 1, &d, t);
      Schedule sch;
      const bool ok = build_forward(1, LayerDims{M, N, K0, K1, DT_BF16}, FwdOperands{}, nullptr, &sch);
      std::printf("%d %d %.3f %.3f %zu\n", ok && sch.steps[0].is_few ? 1 : 0, f.splits, f.us,
                  t_us + plan_time_us(g, M, K0, N, K1) + kColdUsPerMB * 2e-6 * (double)(M * N + N * K0), sch.workspace_bytes);
    }
  }
  return 0;
}
