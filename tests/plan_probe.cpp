// Prints what the library's host code plans for the products and layers named on stdin (tests/test_plans.py); links librunlora.so,
// runs nothing on a GPU.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../include/runlora.h"
#include "../paper_2312_03415_amd/csrc/schedule.hpp"

using namespace rl;

// every forward (T or M kept or not) and backward (T and M kept or not, each choice of gradients) of a layer, with and without dropout: f(is
// a backward, variant, dA wanted, the schedule it runs, the call's choices)
template <typename F>
static void each_call(LayerDims L, F f) {
  Schedule s;
  FwdOperands a;
  a.X.ld = L.i; a.W.ld = L.o; a.A.ld = L.r; a.B.ld = L.o; a.Y.ld = L.o; a.T.ld = L.r; a.M.ld = L.o;
  BwdOperands b;
  b.dY.ld = L.o; b.X.ld = L.i; b.W.ld = L.o; b.A.ld = L.r; b.B.ld = L.o; b.T.ld = L.r; b.dX.ld = L.i; b.dA.ld = L.r; b.dB.ld = L.o; b.M.ld = L.o;
  for (unsigned thr : {0u, 26u}) {
    L.drop_thr = thr;
    for (int v = 0; v <= 3; ++v)
      for (int keep = 0; keep <= (v == 1 || v == 2 ? 1 : 0); ++keep) {
        if (v == 3 && thr != 0) continue;  // (runs as variant 1, and needs what that needs)
        a.keep_T = v == 1 && keep != 0;
        a.keep_M = v == 2 && keep != 0;
        if (build_forward(v, L, a, nullptr, &s)) f(false, v, true, s, (a.keep_T ? RL_CALL_T : 0) | (a.keep_M ? RL_CALL_M : 0) | (thr ? RL_CALL_DROPOUT : 0));
      }
    for (int v = 0; v <= 8; ++v)
      for (int keep = 0; keep < 4; ++keep)
        for (int want = 1; want < 8; ++want) {
          b.have_T = (keep & 1) != 0 && (v == 1 || v == 5 || v == 6 || v == 7);
          b.have_M = (keep & 2) != 0 && (v == 4 || v == 5 || v == 7 || v == 8);
          b.want_dX = (want & 4) != 0; b.want_dA = (want & 2) != 0; b.want_dB = (want & 1) != 0;
          const int choices = (b.have_T ? RL_CALL_T : 0) | (b.have_M ? RL_CALL_M : 0) | (thr ? RL_CALL_DROPOUT : 0) | (b.want_dX ? 0 : RL_CALL_NO_DX) |
                              (b.want_dA ? 0 : RL_CALL_NO_DA) | (b.want_dB ? 0 : RL_CALL_NO_DB);
          if (build_backward(v, L, b, nullptr, &s)) f(true, v, b.want_dA, s, choices);
        }
  }
}

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
    } else if (std::strncmp(kind, "calls", 5) == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: calls that need more than the query names
      const int dt = kind[5] == '3' ? DT_F32 : DT_BF16, code = kind[5] == '3' ? RL_F32 : RL_BF16;
      const bool int4 = kind[5] == '4';
      const size_t factors = 2 * (((size_t)K1 * (size_t)K0 * dtype_size(dt) + 255) / 256 * 256);
      int beyond = 0, beyond_vera = 0, first = -1, inexact = 0;
      each_call(LayerDims{M, N, K0, K1, dt, int4}, [&](bool bwd, int v, bool dA, const Schedule& s, int choices) {
        const size_t have = runlora_workspace_bytes_w(bwd ? -1 : v, bwd ? v : -1, M, N, K0, K1, code, int4 ? RL_INT4_G64 : code);
        if (s.workspace_bytes > have && beyond++ == 0) first = v;
        if (!int4 && !(bwd && dA) && factors + s.workspace_bytes > runlora_vera_workspace_bytes(bwd ? -1 : v, bwd ? v : -1, M, N, K0, K1, code)) ++beyond_vera;
        if (!int4 && s.workspace_bytes != runlora_call_workspace_bytes(bwd ? -1 : v, bwd ? v : -1, M, N, K0, K1, code, choices)) ++inexact;
      });
      std::printf("%d %d %d %d\n", beyond, beyond_vera, inexact, first);
    } else if (std::strcmp(kind, "pair") == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: the launch of backward 1's dA, dB on 128x128 tiles or not, slices
      Schedule s;
      if (!build_backward(1, LayerDims{M, N, K0, K1, DT_BF16}, BwdOperands{}, nullptr, &s)) return 1;
      for (const Step& t : s.steps)
        if (t.is_mtpair && t.sk[0].a_strided) std::printf("%d %d %d\n", t.mtpair.wide ? 1 : 0, t.mtpair.splits[0], t.mtpair.splits[1]);
    } else if (std::strcmp(kind, "maskt") == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: T of forward 1 with dropout on tiles or not, slices
      LayerDims L{M, N, K0, K1, DT_BF16};
      L.drop_thr = 26;
      Schedule s;
      if (!build_forward(1, L, FwdOperands{}, nullptr, &s)) return 1;
      const Step& t = s.steps[0];
      std::printf("%d %d\n", t.nsk == 0 ? 1 : 0, t.nsk == 0 ? t.plan.splits : t.skplan.splits);
    } else if (std::strncmp(kind, "stream", 6) == 0) {  // M, N = r, K of T = X A, K1 = masked or not: slices, wavefronts, rows of a block
      SkinnyDesc d;
      d.M = M; d.N = N; d.K = K0;
      d.drop_thr = K1 != 0 ? 26 : 0;
      const SkinnyPlan p = skinny_plan(kind[6] == '3' ? DT_F32 : DT_BF16, 1, &d);
      std::printf("%d %d %d\n", p.splits, p.nwv, p.mr);
    } else if (std::strcmp(kind, "f32") == 0) {  // M, N, K: tile and slices by tile counts, and as the library runs the product
      GemmPlan p = gemm_plan(DT_F32, M, N, K0, K1);
      std::printf("%d %d ", p.cfg, p.splits);
      gemm_plan_f32(&p, M, N, K0, K1);
      std::printf("%d %d\n", p.cfg, p.splits);
    } else if (std::strcmp(kind, "masked") == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: backward 1 with dropout, dX = dY W^T and its masked update
      // as launches of their own: what they take, and what the call takes that brings so much
      LayerDims L{M, N, K0, K1, DT_BF16};
      L.drop_thr = 26;
      Schedule one, two, got;
      if (!build_backward(1, L, BwdOperands{}, nullptr, &one)) return 1;
      L.masked_product = false;
      if (!build_backward(1, L, BwdOperands{}, nullptr, &two)) return 1;
      L.masked_product = true;
      if (!fit_backward(1, L, BwdOperands{}, nullptr, two.workspace_bytes, &got)) return 1;
      std::printf("%zu %zu %zu %zu\n", one.workspace_bytes, two.workspace_bytes, got.workspace_bytes, got.steps.size());
    } else if (std::strcmp(kind, "static") == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: forward 1 with splits of its rank-r product and without
      LayerDims L{M, N, K0, K1, DT_BF16};
      Schedule s, t;
      if (!build_forward(1, L, FwdOperands{}, nullptr, &s)) return 1;
      L.rank_bytes = 0;
      if (!build_forward(1, L, FwdOperands{}, nullptr, &t)) return 1;
      std::printf("%zu %zu\n", s.workspace_bytes, t.workspace_bytes);
    } else if (std::strncmp(kind, "fit", 3) == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: forward 1 and backward 1 in full, in nothing, and in seven
      // amounts between: how often the schedule is beyond what was brought, and how often beyond its need with nothing
      LayerDims L{M, N, K0, K1, DT_BF16, kind[3] == '4'};
      int beyond = 0, uses_it = 0;
      for (int bwd = 0; bwd < 2; ++bwd) {
        Schedule s;
        auto fit = [&](size_t bytes) {
          if (bwd ? !fit_backward(1, L, BwdOperands{}, nullptr, bytes, &s) : !fit_forward(1, L, FwdOperands{}, nullptr, bytes, &s)) std::exit(1);
          return s.workspace_bytes;
        };
        const size_t full = fit((size_t)1 << 50), least = fit(0);
        for (int k = 0; k <= 8; ++k) {
          const size_t bytes = least + (full - least) * (size_t)k / 8;
          const size_t need = fit(bytes);
          if (full >= least && need > bytes) ++beyond;
          if (need > least) ++uses_it;
        }
      }
      std::printf("%d %d\n", beyond, uses_it);
    } else if (std::strcmp(kind, "few") == 0) {  // M = tokens, N = d_in, K0 = d_out, K1 = r: the few-token route's price and taken or not
      SkinnyDesc d;
      d.M = M; d.N = K1; d.K = N;
      const GemmPlan g = gemm_plan(DT_BF16, M, K0, N, K1);
      const SkinnyPlan t = skinny_plan(DT_BF16, 1, &d);
      const size_t bytes = t.partial_bytes > g.partial_bytes ? t.partial_bytes : g.partial_bytes;
      const FewPlan f = few_plan(M, N, K0, K1, bytes);
      GemmPlan rank;
      double t_us = 0;
      if (!rank_plan(DT_BF16, d, K1 > 32 && bytes < kRankScratch ? kRankScratch - ((size_t)M * (size_t)K1 * 2 + 255) / 256 * 256 : bytes, &rank, &t_us)) t_us = skinny_time_us(DT_BF16, 1, &d, t);
      Schedule sch;
      const bool ok = build_forward(1, LayerDims{M, N, K0, K1, DT_BF16}, FwdOperands{}, nullptr, &sch);
      std::printf("%d %d %.3f %.3f %zu\n", ok && sch.steps[0].is_few ? 1 : 0, f.splits, f.us,
                  t_us + plan_time_us(g, M, K0, N, K1) + kColdUsPerMB * 2e-6 * (double)(M * N + N * K0), sch.workspace_bytes);
    }
  }
  return 0;
}
