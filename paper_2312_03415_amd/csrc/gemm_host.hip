// Launch planning and dispatch for the tile GEMM engine.
#include "gemm.hpp"
#include "gemm_engine.hpp"
#include "skinny.hpp"
#include "merge.hpp"
#include "lora_finish.hpp"

namespace rl {

thread_local KernelEvents g_kernel_events;

// (ids 8..11 are no tile GEMMs)
static const int kTileBM[CFG_COUNT] = {256, 128, 128, 128, 32, 64, 256, 256, 0, 0, 0, 0, 128, 128, 256, 128, 64};
static const int kTileBN[CFG_COUNT] = {256, 128, 32, 64, 128, 128, 256, 256, 0, 0, 0, 0, 128, 128, 128, 64, 128};
static const int kTileBK16[CFG_COUNT] = {64, 64, 64, 64, 64, 64, 32, 64, 0, 0, 0, 0, 64, 64, 64, 64, 64};  // K tile, 16-bit types

// Slices of a contraction of length K for `tiles` output tiles of the matrix-core kernel (one 256x256 workgroup per
// compute unit).  In units of a whole tile's time (0.024 us per k): s slices take ceil(tiles * s / 256) rounds of 1 / s
// each; the reduce pass reads s fp32 partials per output at ~5.5 TB/s (2 tiles s / K) and is a launch of ~5 us (200 / K).
// 96 tiles at K = 4096 run best in two slices (192 work items, one round of half tiles), not in the three that fill 256
// slots and spill 32 items into a second round.
static int pick_splits(int64_t tiles, int64_t K, int smin) {
  int best = smin;
  double best_cost = 1e30;
  const double k = (double)(K > 0 ? K : 1);
  for (int s = smin; s <= 8; ++s) {
    const double rounds = (double)((tiles * s + 255) / 256);
    const double cost = rounds / s + (s > 1 ? 2.0 * (double)tiles * s / k + 200.0 / k : 0.0);
    if (cost < best_cost - 1e-9) { best_cost = cost; best = s; }
  }
  return best;
}

// What a launch of a 16-bit tile GEMM takes, in us, fitted to one sweep of tile shapes and K splits (534 products: M 33 .. 8192,
// N 40 .. 11008, K 512 .. 11008, NN / NT / TN; 17 800 timings with W from HBM, as in a model): `one` and `full` = one K tile
// with at most one workgroup on a compute unit and with all its slots taken, `fix` = launch, prologue and epilogue, `round` =
// every further round of workgroups, `store` = a million outputs, `split_lines` = what a K tile takes longer where rows are not
// whole 128-byte lines (a row's piece then touches two), `fabric` = KB per us that reach an XCD's L2 from outside it.
// One standard deviation is 7-11 %.  The plan these choose takes 2 % longer on average than the best one timed (26 % at worst),
// and for none of the 534 more than 2 % longer than the plan by tile counts in gemm_plan.  Constants from operands that the
// caches held, without the last three terms, lost 8 % on average, up to 22 % against that plan, and 48 % at 4096 x 2056 x 5464
// (182-201 us on 64x128 tiles, 123-137 on 256x256).
struct LaunchModel { int slots; double fix, one, full, round, store, split_lines, fabric; };
static LaunchModel launch_model(int cfg) {
  switch (cfg) {
    case CFG_MID: return {512, 3.8, 1.04, 1.26, 0.0, 0.51, 0.05, 1360};
    case CFG_TALL64: return {768, 2.7, 0.78, 1.13, 0.0, 0.59, 0.0, 1240};
    case CFG_WIDE32: return {768, 3.6, 0.35, 0.6, 0.0, 0.5, 0.09, 860};  // (priced for few_forward only)
    case CFG_WIDE64: return {768, 3.7, 0.89, 1.19, 2.8, 4.01, 0.09, 860};
    case CFG_MT128: return {512, 3.5, 0.66, 0.89, 0.0, 0.42, 0.18, 1130};
    case CFG_MT128D: return {256, 5.2, 0.42, 0.51, 1.8, 0.43, 0.15, 1380};
    case CFG_MT256: return {256, 6.2, 0.69, 0.81, 1.5, 0.69, 0.16, 1510};
    case CFG_MTN64: return {512, 3.8, 0.297, 0.637, 0.0, 0.26, 0.14, 1230};
    case CFG_MTM64: return {512, 4.1, 0.29, 0.586, 0.0, 0.35, 0.15, 1160};
    default: return {256, 5.0, 1.2, 1.32, 0.0, 0.48, 0.26, 1900};  // CFG_MC4: persistent, the next tile's loads run during an epilogue
  }
}

// Operand KB of a K tile that an XCD's resident workgroups want, each once: they hold a run of tiles in bands of eight tile rows
// (per K slice), of which those in a row share A and those in a column share B.
static double xcd_kbytes(int cfg, int64_t nbm, int64_t nbn, int64_t wgs, int64_t slots) {
  auto kb = [&](int64_t run) {
    const int64_t band = nbm < 8 ? nbm : 8, rows = run < band ? run : band, cols = (run + rows - 1) / rows;
    return (double)(rows * kTileBM[cfg] + cols * kTileBN[cfg]) * 0.128;
  };
  const int64_t per_xcd = (nbm * nbn + 7) / 8, most = slots / 8, resident = (wgs + 7) / 8 < most ? (wgs + 7) / 8 : most;
  return resident >= per_xcd ? (double)resident / (double)per_xcd * kb(per_xcd) : kb(resident);
}

double launch_time_us(int cfg, int64_t nbm, int64_t nbn, int splits, int64_t ktiles, double odd) {
  const LaunchModel m = launch_model(cfg);
  const int64_t tiles = nbm * nbn, wgs = tiles * splits, rounds = wgs / m.slots, rest = wgs % m.slots;
  const double bytes = xcd_kbytes(cfg, nbm, nbn, wgs, m.slots);
  const double feed = bytes * (1.0 + odd) / m.fabric;
  auto tile = [&](double t) { t += m.split_lines * odd; return t > feed ? t : feed; };
  double per_k = (double)rounds * tile(m.full);
  if (rest > 0) per_k += tile(rest <= 256 ? m.one : m.full);
  const double outs = splits > 1 ? 0.0 : (double)(tiles * kTileBM[cfg] * kTileBN[cfg]);
  return m.fix + (double)ktiles * per_k + m.round * (double)(rounds + (rest > 0 ? 1 : 0) - 1) + m.store * outs / 1e6;
}

// partials written, read back and reduced: 3 us, 5.5 TB/s, and 0.36 us for every slice beyond 16 (a thread of the reduce pass
// walks them one after the other)
double split_time_us(int64_t M, int64_t N, int splits) {
  return splits > 1 ? 3.0 + (double)M * (double)N * (8.0 * splits + 2.0) / 5.5e6 + 0.36 * (splits > 16 ? splits - 16 : 0) : 0.0;
}

// Tile shape and K split of a 16-bit product on the matrix-core kernels: the smallest modelled time among 256x256 (whole
// rounds with cut-off tail columns included), 256x128, 128x128 (two ways), 128x64 and 64x128, each with the contraction
// in 1 .. 64 slices of at least four K tiles.  cap = scratch bytes the plan may use for partials.
static bool mt_plan(GemmPlan* out, double* out_us, int64_t M, int64_t N, int64_t K0, int64_t K1, size_t cap, bool tail_ok) {
  static const int cfgs[] = {CFG_MC4, CFG_MT256, CFG_MT128, CFG_MT128D, CFG_MTN64, CFG_MTM64};
  const int64_t kt = (K0 + 63) / 64 + (K1 + 63) / 64;
  const double odd = odd_lines(N, K0);
  double best = 1e30;
  for (int cfg : cfgs) {
    const int64_t nbm = (M + kTileBM[cfg] - 1) / kTileBM[cfg], nbn = (N + kTileBN[cfg] - 1) / kTileBN[cfg], tiles = nbm * nbn;
    if (tiles > (1 << 30)) continue;
    for (int s = 1; s <= 64 && (s == 1 || kt / s >= 4); ++s) {
      const int64_t per = (kt + s - 1) / s;
      const int used = (int)((kt + per - 1) / per);  // no empty slice
      if (used != s) continue;
      const size_t bytes = s > 1 ? (size_t)s * (size_t)M * (size_t)N * sizeof(float) : 0;
      if (bytes > cap) break;
      const double us = launch_time_us(cfg, nbm, nbn, s, per, odd) + split_time_us(M, N, s);
      if (us < best) {
        best = us;
        *out = GemmPlan{};
        out->cfg = cfg;
        out->bk = 64;
        out->bm = kTileBM[cfg];
        out->bn = kTileBN[cfg];
        out->nbm = (int)nbm;
        out->nbn = (int)nbn;
        out->splits = s;
        out->tiles_per_split = (int)per;
        out->partial_bytes = bytes;
      }
    }
    // 256x256 tiles in whole rounds, the remaining tile columns as a launch of their own
    if (cfg == CFG_MC4 && tail_ok && tiles > 256 && kt >= 16) {
      for (int64_t t = nbn - 1; t >= 1 && t >= nbn - 16; --t) {
        if ((nbm * t) % 256 != 0) continue;
        GemmPlan tp;
        double tus = 0;
        if (!mt_plan(&tp, &tus, M, N - t * 256, K0, K1, cap, false)) break;
        const double us = launch_time_us(CFG_MC4, nbm, t, 1, kt, odd) + tus;
        if (us < best) {
          best = us;
          *out = GemmPlan{};
          out->cfg = CFG_MC4;
          out->bk = 64;
          out->bm = out->bn = 256;
          out->nbm = (int)nbm;
          out->nbn = (int)t;
          out->tiles_per_split = (int)kt;
          out->tail_n0 = t * 256;
          out->tail_cfg = tp.cfg;
          out->tail_splits = tp.splits;
          out->partial_bytes = tp.partial_bytes;
        }
        break;
      }
    }
  }
  *out_us = best;
  return best < 1e30;
}

bool long_operand(const GemmDesc& d) {
  for (int s = 0; s < d.nseg; ++s) {
    const int64_t a_rows = d.a_strided ? d.K[s] : d.M, b_rows = d.b_kcontig ? d.N : d.K[s];
    const int64_t a_cols = d.a_strided ? d.M : d.K[s], b_cols = d.b_kcontig ? d.K[s] : d.N;  // (planned without operands: ld 0)
    if (a_rows * (d.lda[s] > a_cols ? d.lda[s] : a_cols) >= (1LL << 30)) return true;
    if (!(s == 0 && d.b_int4) && b_rows * (d.ldb[s] > b_cols ? d.ldb[s] : b_cols) >= (1LL << 30)) return true;
  }
  return false;
}

// bf16 only: V = W + s A B rounded to f16 may overflow, or lose bits as a subnormal, where V diag(g), rounded after the scaling, does
// neither; in bf16 the two have the same range.
bool column_scale_ok(const GemmDesc& d, const GemmPlan& p) {
  auto built = [](int cfg, int splits) { return splits <= 1 && (cfg_is_mt(cfg) || cfg == CFG_MC4); };
  return d.dtype == DT_BF16 && d.nseg == 1 && !d.a_strided && !d.b_kcontig && !d.b_int4 && d.Bscale == nullptr && !d.has_addend && d.D == nullptr &&
         d.alpha == 1.f && d.drop_thr == 0 && !d.fuse_t && !long_operand(d) && built(p.cfg, p.splits) && (p.tail_n0 == 0 || built(p.tail_cfg, p.tail_splits));
}

bool masked_segment_ok(const GemmDesc& d, const GemmPlan& p) {
  auto built = [&](int cfg, int splits) { return cfg_is_mt(cfg) || (cfg == CFG_MC4 && splits <= 1 && d.K[0] <= 32); };
  return d.dtype != DT_F32 && d.nseg == 2 && !d.a_strided && d.b_kcontig && !d.b_int4 && d.Bscale == nullptr && !d.has_addend && d.D == nullptr &&
         d.bias == nullptr && d.alpha == 1.f && !d.fuse_t && !long_operand(d) && built(p.cfg, p.splits) && (p.tail_n0 == 0 || built(p.tail_cfg, p.tail_splits));
}

// What a launch of an fp32 tile GEMM takes, in us: a K tile of 32 takes a workgroup `one` alone on its compute unit, c workgroups on
// a unit c `sat` together, whatever runs next to what (128x128 512 GFLOP/s a unit, narrower tiles less: their operands are read
// more often).  Fitted to 16 products (200 .. 4096 rows, 512 .. 3000 columns, K 512 .. 4000), every tile and 1 .. 10 slices: within
// 10 % but for a few with many short slices.
static double f32_launch_us(int cfg, int64_t tiles, int splits, int64_t ktiles) {
  struct { double one, sat; } static const m[6] = {{8.1, 8.1}, {2.56, 2.26}, {1.02, 0.76}, {1.55, 1.2}, {1.02, 0.78}, {1.55, 1.25}};
  const double per = m[cfg].sat * (double)((tiles * splits + 255) / 256);
  return 4.0 + (double)ktiles * (per > m[cfg].one ? per : m[cfg].one);
}

static double f32_time_us(int cfg, int64_t tiles, int splits, int64_t ktiles, double outs) {
  return f32_launch_us(cfg, tiles, splits, ktiles) + (splits > 1 ? 4.0 + outs * (8.0 * splits + 4.0) / 5.5e6 : 0.0);
}

// Tile shape and K split of an fp32 product (more than 32 rows and columns) by that model, in the scratch of the plan by tile
// counts that comes in, which takes 128x128 tiles and as many slices as fill the chip: 256 x 768 x 768 21.8 us against 12.8 on 48 tiles of
// 32x128 in five slices, 4096 x 512 x 512 39.8 against 33 unsplit on 128x64, 1000 x 1024 x 1024 38 against 34.6, 300 x 2000 x 4000
// 102 against 67, 500 x 2048 x 2048 57 against 55.5.  Larger products keep the plan by tile counts: several workgroups of narrow
// tiles on every unit feed each other less than the model says (2000 x 768 x 3072 123 against 133, 3000 x 1800 x 1800 264 against
// 278, 950 x 3000 x 3000 235 against 243).  A plan on 128x128 tiles in 2 .. 16 slices has to be modelled more than 3 % slower: of 409 products (68 ..
// 6000 rows and columns, K 64 .. 6000) six are then slower than on the plan that comes in, by 4-8 %, where all take 0.8 of its time on
// average; without the 3 %, two more by 10 % (204 x 4008 x 4060 83.3 against 94.1, 212 x 3284 x 1944 45.3 against 50.2); with 5 %, none
// fewer and five gains of 4-16 % are lost.  Other plans are never kept: whole ones and those in many slices are modelled too fast (296 x
// 7496 x 32 3 us slower, 52 x 344 x 5992 6).
void gemm_plan_f32(GemmPlan* p, int64_t M, int64_t N, int64_t K0, int64_t K1) {
  if (M <= 32 || N <= 32 || (double)M * (double)N * (double)(K0 + K1) > 4e9) return;
  const int64_t kt = (K0 + p->bk - 1) / p->bk + (K1 + p->bk - 1) / p->bk;
  const size_t cap = p->partial_bytes;  // the scratch stays what is reported
  const double outs = (double)M * (double)N;
  double best = 1e30;
  if (p->cfg == CFG_MID && p->splits > 1 && p->splits <= 16) best = f32_time_us(p->cfg, (int64_t)p->nbm * p->nbn, p->splits, p->tiles_per_split, outs) / 1.03;
  for (int cfg = CFG_BIG; cfg <= CFG_WIDE64; ++cfg) {
    const int64_t nbm = (M + kTileBM[cfg] - 1) / kTileBM[cfg], nbn = (N + kTileBN[cfg] - 1) / kTileBN[cfg];
    if (nbm * nbn > (1 << 24)) continue;
    for (int s = 1; s <= 16 && (s == 1 || kt / s >= 4); ++s) {
      const int64_t per = (kt + s - 1) / s;
      if ((kt + per - 1) / per != s) continue;  // no empty slice
      if (s > 1 && (size_t)s * (size_t)M * (size_t)N * sizeof(float) > cap) break;
      const double us = f32_time_us(cfg, nbm * nbn, s, per, outs);
      if (us >= best) continue;
      best = us;
      p->cfg = cfg;
      p->bm = kTileBM[cfg];
      p->bn = kTileBN[cfg];
      p->nbm = (int)nbm;
      p->nbn = (int)nbn;
      p->splits = s;
      p->tiles_per_split = (int)per;
    }
  }
}

GemmPlan gemm_plan(int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1, int force_cfg,
                   int force_splits, bool b_int4, bool long_operand) {
  GemmPlan p;
  int cfg;
  if (b_int4 && force_cfg < 0) {
    // an int4 B runs on the matrix-core kernel (3-stage ring) when its 256x256 tiles fill the chip,
    // else on the generic engine's 128x128 tiles
    const int64_t big_tiles = ((M + 255) / 256) * ((N + 255) / 256);
    cfg = (big_tiles >= 160 || (big_tiles >= 80 && K0 + K1 >= 2048)) ? CFG_MC3 : CFG_MID;
  } else if (cfg_is_tile(force_cfg)) {
    cfg = force_cfg;
    if ((cfg == CFG_MC3 || cfg == CFG_MC4) && dtype == DT_F32) cfg = CFG_BIG;  // 16-bit only
    if (cfg_is_mt(cfg) && dtype == DT_F32) cfg = CFG_MID;
  } else if (M <= 32) {
    cfg = CFG_WIDE32;
  } else if (M <= 64) {
    cfg = CFG_WIDE64;
  } else if (N <= 32) {
    cfg = CFG_TALL32;
  } else if (N <= 64) {
    cfg = CFG_TALL64;
  } else {
    // the 256x256 tile needs enough tiles to occupy the 256 compute units; a grid between half
    // and full is filled by splitting the contraction in two
    const int64_t big_tiles = ((M + 255) / 256) * ((N + 255) / 256);
    const bool pipe_ok = dtype != DT_F32;
    if (big_tiles >= 160 || (big_tiles >= 80 && K0 + K1 >= 2048))
      cfg = pipe_ok ? CFG_MC4 : CFG_BIG;
    else
      cfg = CFG_MID;
  }
  p.cfg = cfg;
  p.bk = (dtype == DT_F32) ? 32 : kTileBK16[cfg];
  p.bm = kTileBM[cfg];
  p.bn = kTileBN[cfg];
  p.nbm = (int)((M + p.bm - 1) / p.bm);
  p.nbn = (int)((N + p.bn - 1) / p.bn);
  const int64_t tiles = (int64_t)p.nbm * p.nbn;
  const int ktiles = (int)((K0 + p.bk - 1) / p.bk + (K1 + p.bk - 1) / p.bk);
  int splits = 1;
  if (force_splits > 0) {
    splits = force_splits;
  } else if (cfg == CFG_MC3 || cfg == CFG_MC4 || cfg == CFG_BIG) {
    if (tiles < 160 && (int64_t)ktiles * p.bk >= 1024) splits = pick_splits(tiles, (int64_t)ktiles * p.bk, 1);
  } else if (tiles < 256 && ktiles >= 8) {
    // fill the chip (aim at ~512 workgroups) but keep >= 4 K tiles per slice
    int64_t want = (512 + tiles - 1) / tiles;
    int64_t cap = ktiles / 4;
    splits = (int)(want < cap ? want : cap);
    if (splits > 64) splits = 64;
    if (splits < 1) splits = 1;
  }
  if (splits > ktiles) splits = ktiles > 0 ? ktiles : 1;
  p.tiles_per_split = (ktiles + splits - 1) / splits;
  if (p.tiles_per_split < 1) p.tiles_per_split = 1;
  p.splits = (ktiles + p.tiles_per_split - 1) / p.tiles_per_split;  // no empty slice
  if (p.splits < 1) p.splits = 1;
  p.partial_bytes = p.splits > 1 ? (size_t)p.splits * (size_t)M * (size_t)N * sizeof(float) : 0;
  // Tile quantisation: with one 256x256 tile per compute unit and round, a grid of e.g. 32 x 43 tiles
  // ends on a round that is 3/8 full.  If whole tile columns can be cut off such that the rest is an
  // exact number of rounds and the cut-off part is small enough to be split along K, run that part
  // as a launch of its own (half a round with the contraction in two, plus its reduce).
  if (force_cfg < 0 && force_splits <= 0 && (p.cfg == CFG_MC4 || (b_int4 && p.cfg == CFG_MC3)) && p.splits == 1 &&
      tiles > 256 && (int64_t)ktiles * p.bk >= 2048) {
    for (int t = p.nbn - 1; t >= 1 && t >= p.nbn - 16; --t) {
      const int64_t main_tiles = (int64_t)p.nbm * t, tail_tiles = (int64_t)p.nbm * (p.nbn - t);
      if (tail_tiles > 128) break;
      if (main_tiles % 256 != 0 || tail_tiles < 32) continue;
      p.tail_n0 = (int64_t)t * p.bn;
      p.nbn = t;
      p.tail_cfg = p.cfg;
      p.tail_splits = pick_splits((int64_t)p.nbm * ((N - p.tail_n0 + p.bn - 1) / p.bn), K0 + K1, 2);
      p.partial_bytes = gemm_tail_plan(p, dtype, M, N, K0, K1).partial_bytes;
      break;
    }
  }
  // 16-bit products with more than 32 rows and columns run on the matrix-core kernels where those are modelled faster than
  // the plan above (256x256 tiles are among theirs), with no more scratch than it takes: its need stays the one that is
  // reported, the size of a workspace that callers keep is a matter of the product, not of the kernel it runs on.
  if (dtype != DT_F32 && !b_int4 && !long_operand && force_cfg < 0 && force_splits <= 0 && M > 32 && N > 32) {
    GemmPlan q;
    double us = 0;
    if (mt_plan(&q, &us, M, N, K0, K1, p.partial_bytes, true) && (p.cfg == CFG_MC4 || us < plan_time_us(p, M, N, K0, K1))) {
      q.partial_bytes = p.partial_bytes;
      return q;
    }
  }
  return p;
}

GemmPlan gemm_tail_plan(const GemmPlan& main, int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1) {
  return gemm_plan(dtype, M, N - main.tail_n0, K0, K1, main.tail_cfg, main.tail_splits);
}

double plan_time_us(const GemmPlan& p, int64_t M, int64_t N, int64_t K0, int64_t K1) {
  if (p.tail_n0 > 0) {
    GemmPlan main = p;
    main.tail_n0 = 0;
    return plan_time_us(main, M, p.tail_n0, K0, K1) + plan_time_us(gemm_tail_plan(p, DT_BF16, M, N, K0, K1), M, N - p.tail_n0, K0, K1);
  }
  const int64_t kt = p.splits > 1 ? p.tiles_per_split : (K0 + 63) / 64 + (K1 + 63) / 64;
  return launch_time_us(p.cfg, p.nbm, p.nbn, p.splits, kt, odd_lines(N, K0)) + split_time_us(M, N, p.splits);
}

GemmPlan gemm_plan_int4(int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1) {
  return gemm_plan(dtype, M, N, K0, K1, -1, 0, true);
}

// What the kernels that dequantise on the way to LDS take, in us (bf16; 4096 x 5120 x 13824: 557 us for three rounds of 256 tiles
// and 162 K tiles of 32, 492 for one of 434; 128x128 tiles of the generic engine, two to a compute unit: 247 us at 672 x 3208 x
// 12960 in four slices, 310 at 491 x 7408 x 11744 in three).  Layers timed on both routes, forward, r 16-64, us (direct / panels):
// 512 x 2048 -> 2048 38.8 / 30.7, 1024 x 4096 -> 4096 171 / 62.6, 2048 x 4096 -> 4096 124 / 92.6, 672 x 12960 -> 3208 266 / 183;
// 913 x 6240 -> 6232 135 / 159, 3748 x 12720 -> 7888 838 / 1156 (panels on the tiles chosen at the time).
static double int4_direct_us(const GemmPlan& p, int64_t M, int64_t N, int64_t K0, int64_t K1) {
  if (p.tail_n0 > 0) {
    GemmPlan main = p;
    main.tail_n0 = 0;
    const GemmPlan tail = gemm_tail_plan(p, DT_BF16, M, N, K0, K1);
    return int4_direct_us(main, M, p.tail_n0, K0, K1) + int4_direct_us(tail, M, N - p.tail_n0, K0, K1);
  }
  const double wgs = (double)p.nbm * p.nbn * p.splits;
  const int64_t kt = (K0 + p.bk - 1) / p.bk + (K1 + p.bk - 1) / p.bk;
  const double per = p.splits > 1 ? (double)p.tiles_per_split : (double)kt;
  if (p.cfg == CFG_MC3) {
    const double rounds = wgs <= 256.0 ? 1.0 : (double)(int64_t)(wgs / 256.0 + 0.999);
    return 10.0 + rounds * (per * 1.14 + 6.0) + split_time_us(M, N, p.splits);
  }
  // a K tile takes 1 us alone, 2.2 where two share a compute unit; a few workgroups of a last round take as long as a whole one
  const double rounds = wgs <= 512.0 ? 1.0 : (double)(int64_t)(wgs / 512.0 + 0.999);
  return 8.0 + rounds * (per * (wgs <= 256.0 ? 1.0 : 2.2) + 1.0) + split_time_us(M, N, p.splits);
}

Int4PanelPlan int4_panel_plan(int dtype, int64_t M, int64_t N, int64_t K0, int64_t K1) {
  Int4PanelPlan best;
  if (dtype == DT_F32 || M <= 32 || N <= 32 || K0 < 1) return best;
  const int64_t fit = (int64_t)(kInt4PanelBytes / (2 * (size_t)K0)) / 256 * 256;
  if (fit < 256) return best;
  // candidates: everything in one panel, the widest panel, and the widest whose 256x256 / 256x128 tiles are whole rounds
  int64_t cand[3] = {N <= fit ? N : fit, 0, 0};
  const int64_t nbm = (M + 255) / 256;
  for (int64_t w = fit; w >= 256 && cand[1] == 0; w -= 256)
    if (w < N && (nbm * (w / 256)) % 256 == 0) cand[1] = w;
  for (int64_t w = fit; w >= 256 && cand[2] == 0; w -= 256)
    if (w < N && (nbm * (w / 128)) % 256 == 0) cand[2] = w;
  best.us = int4_direct_us(gemm_plan_int4(dtype, M, N, K0, K1), M, N, K0, K1);
  for (int64_t w : cand) {
    if (w == 0) continue;
    const int64_t fulls = (N + w - 1) / w - 1, rest = N - fulls * w;
    Int4PanelPlan p;
    p.width = w;
    p.panel_bytes = ((size_t)w * (size_t)K0 * 2 + 255) / 256 * 256;
    // partials of a split product stay within what one panel may take
    const size_t cap = kInt4PanelBytes;
    double uf = 0, ul = 0;
    if (fulls > 0 && !mt_plan(&p.full, &uf, M, w, K0, K1, 0, true)) continue;
    if (!mt_plan(&p.last, &ul, M, rest, K0, K1, cap - (p.panel_bytes < cap ? p.panel_bytes : cap), true)) continue;
    if (fulls == 0) p.full = p.last;
    p.scratch_bytes = p.panel_bytes + p.last.partial_bytes;
    p.us = uf * (double)fulls + ul + 4.0 * (double)(fulls + 1) + (double)N * (double)K0 * 2.5 / 4.5e6;
    if (p.us < best.us) best = p;
  }
  return best;
}

hipError_t int4_panel_gemm(const GemmDesc& d, const Int4PanelPlan& plan, void* scratch, hipStream_t stream) {
  if (plan.width < 1 || scratch == nullptr || d.Bscale == nullptr || d.D != nullptr || d.drop_thr != 0 || d.a_strided) return hipErrorInvalidValue;
  char* const panel = static_cast<char*>(scratch);
  float* const partial = reinterpret_cast<float*>(panel + plan.panel_bytes);
  for (int64_t n0 = 0; n0 < d.N; n0 += plan.width) {
    const bool last = n0 + plan.width >= d.N;
    const int64_t w = last ? d.N - n0 : plan.width;
    GemmDesc s = d;
    s.b_int4 = false;
    s.Bscale = nullptr;
    s.ldbs = 0;
    s.N = w;
    s.B[0] = panel;
    s.ldb[0] = d.b_kcontig ? d.K[0] : w;
    hipError_t e = d.b_kcontig ? int4_panel_run(d.dtype, d.B[0], d.ldb[0], d.Bscale, d.ldbs, panel, d.K[0], n0, w, 0, d.K[0], stream)
                               : int4_panel_run(d.dtype, d.B[0], d.ldb[0], d.Bscale, d.ldbs, panel, w, 0, d.K[0], n0, w, stream);
    if (e != hipSuccess) return e;
    if (d.nseg > 1) s.B[1] = static_cast<const char*>(d.B[1]) + (size_t)(d.b_kcontig ? n0 * d.ldb[1] : n0) * 2;
    s.C = static_cast<char*>(d.C) + (size_t)n0 * 2;
    if (d.bias) s.bias = static_cast<const char*>(d.bias) + (size_t)n0 * 2;
    e = gemm_run(s, last ? plan.last : plan.full, partial, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

GemmPlan gemm_plan_fused(int dtype, int64_t M, int64_t N, int64_t K0, int64_t R) {
  // the shape rules of gemm_plan for the generic engine (those fp32 runs on); the workgroup that owns an output tile needs
  // the whole contraction of its rows of T: no split
  const int cfg = gemm_plan(DT_F32, M, N, K0, R).cfg;
  return gemm_plan(dtype, M, N, K0, R, cfg, 1);
}

hipError_t gemm_run(const GemmDesc& d, const GemmPlan& plan, float* scratch, hipStream_t stream) {
  if (d.M <= 0 || d.N <= 0) return hipErrorInvalidValue;
  if (plan.tail_n0 > 0) {
    // columns [0, tail_n0) with this plan, columns [tail_n0, N) as their own problem
    if (plan.tail_n0 >= d.N) return hipErrorInvalidValue;
    if (d.drop_thr != 0 && !d.mask_seg0) return hipErrorInvalidValue;  // the mask is indexed by the full product's columns (K = r: never cut)
    const size_t esz = d.dtype == DT_F32 ? 4 : 2;
    GemmDesc dm = d, dt = d;
    GemmPlan pm = plan;
    pm.tail_n0 = 0;
    pm.partial_bytes = 0;
    dm.N = plan.tail_n0;
    dt.N = d.N - plan.tail_n0;
    dt.drop_n4 = d.drop_n4 + (uint32_t)(plan.tail_n0 / 4);
    for (int s = 0; s < d.nseg; ++s) {
      const int64_t off = d.b_kcontig ? plan.tail_n0 * d.ldb[s] : plan.tail_n0;
      if (s == 0 && d.Bscale != nullptr) {
        // int4: two weights per byte; the scales of columns (B stored [K,N]) or of row groups
        // (B stored [N,K]; tail_n0 is a multiple of 64) move along
        dt.B[0] = static_cast<const char*>(d.B[0]) + (size_t)off / 2;
        const int64_t soff = d.b_kcontig ? (plan.tail_n0 / 64) * d.ldbs : plan.tail_n0;
        dt.Bscale = static_cast<const char*>(d.Bscale) + (size_t)soff * 2;
      } else {
        dt.B[s] = static_cast<const char*>(d.B[s]) + (size_t)off * esz;
      }
    }
    dt.C = static_cast<char*>(d.C) + (size_t)plan.tail_n0 * esz;
    if (d.D) dt.D = static_cast<const char*>(d.D) + (size_t)plan.tail_n0 * esz;
    if (d.bias) dt.bias = static_cast<const char*>(d.bias) + (size_t)plan.tail_n0 * esz;
    if (d.cscale) dt.cscale = d.cscale + plan.tail_n0;
    hipError_t e = gemm_run(dm, pm, nullptr, stream);
    if (e != hipSuccess) return e;
    const GemmPlan pt = gemm_tail_plan(plan, d.dtype, d.M, d.N, d.K[0], d.nseg > 1 ? d.K[1] : 0);
    if (pt.tail_n0 > 0 || pt.partial_bytes > plan.partial_bytes) return hipErrorInvalidValue;
    return gemm_run(dt, pt, pt.splits > 1 ? scratch : nullptr, stream);
  }
  if (plan.splits > 1 && scratch == nullptr) return hipErrorInvalidValue;
  if (d.cscale != nullptr && !column_scale_ok(d, plan)) return hipErrorInvalidValue;
  if (d.mask_a && (d.drop_thr == 0 || d.nseg != 1 || plan.cfg != CFG_MTN64 || d.b_kcontig || d.dtype == DT_F32 || long_operand(d))) return hipErrorInvalidValue;
  if (d.mask_seg0 && (d.drop_thr == 0 || !masked_segment_ok(d, plan))) return hipErrorInvalidValue;
  if (d.fuse_t) {
    const bool ok = d.LA != nullptr && d.nseg == 2 && d.K[1] >= 1 && d.K[1] <= kFuseMaxR && d.K[0] >= 1 && !d.a_strided &&
                    !d.b_kcontig && plan.splits == 1 && d.D == nullptr && d.Bscale == nullptr && d.drop_thr == 0 &&
                    plan.cfg != CFG_MC3 && plan.cfg != CFG_MC4 && !cfg_is_mt(plan.cfg);
    if (!ok) return hipErrorInvalidValue;
  }
  int cfg = plan.cfg;
  if (d.Bscale != nullptr && cfg != CFG_BIG && cfg != CFG_MID && cfg != CFG_MC3) return hipErrorInvalidValue;  // see gemm_plan_int4
  if (d.Bscale != nullptr && d.a_strided) return hipErrorInvalidValue;
  if (cfg == CFG_MC3 || cfg == CFG_MC4) {
    // the matrix-core kernel addresses each operand with 32-bit byte offsets into a buffer descriptor whose
    // extent is the operand's bytes plus 3 KB (gemm_mc.hpp, kBias): the 16-bit elements of an operand, rows x ld,
    // must stay below 2^31 - 2048 so that neither wraps; it also clamps a strided operand's last columns to
    // [dim-8, dim) and wants every K slice to hold at least one K tile
    bool ok = d.dtype != DT_F32 && plan.bk == (cfg == CFG_MC4 ? 64 : 32);
    constexpr int64_t kMaxElems = (1LL << 31) - 2048;
    for (int s = 0; s < d.nseg; ++s) {
      const int64_t a_rows = d.a_strided ? d.K[s] : d.M, b_rows = d.b_kcontig ? d.N : d.K[s];
      if (a_rows * d.lda[s] >= kMaxElems || b_rows * d.ldb[s] >= kMaxElems) ok = false;
    }
    if ((d.a_strided && d.M < 8) || (!d.b_kcontig && d.N < 8)) ok = false;
    if (!ok) cfg = CFG_BIG;
  }
  int nbm = plan.nbm, nbn = plan.nbn;
  if (cfg_is_mt(cfg)) {
    // gemm_mt.hpp addresses each operand with 31-bit byte offsets; a forced id with a larger one runs on the generic engine
    // (same K tile)
    if (d.dtype == DT_F32 || plan.bk != 64 || long_operand(d)) {
      cfg = CFG_MID;
      nbm = (int)((d.M + kTileBM[cfg] - 1) / kTileBM[cfg]);
      nbn = (int)((d.N + kTileBN[cfg] - 1) / kTileBN[cfg]);
    }
  }
  GemmArgs a{};
  for (int s = 0; s < 2; ++s) {
    const bool on = s < d.nseg;
    a.A[s] = on ? d.A[s] : nullptr;
    a.B[s] = on ? d.B[s] : nullptr;
    a.lda[s] = on ? d.lda[s] : 0;
    a.ldb[s] = on ? d.ldb[s] : 0;
    a.K[s] = on ? (int)d.K[s] : 0;
  }
  a.C = d.C;
  a.ldc = d.ldc;
  a.D = plan.splits > 1 ? nullptr : d.D;
  a.ldd = d.ldd;
  a.partial = plan.splits > 1 ? scratch : nullptr;
  a.M = (int)d.M;
  a.N = (int)d.N;
  a.tiles_per_split = plan.splits > 1 ? plan.tiles_per_split : (1 << 30);
  a.nbm = nbm;
  a.nbn = nbn;
  a.splits = plan.splits;
  a.Bscale = d.Bscale;
  a.ldbs = d.ldbs;
  a.alpha = d.alpha;
  a.bias = plan.splits > 1 ? nullptr : d.bias;
  a.drop_thr = d.drop_thr;
  a.drop_key = d.drop_key;
  a.drop_cpr = d.drop_cpr;
  a.mask_seg0 = d.mask_seg0 ? 1 : 0;
  a.mask_a = d.mask_a ? 1 : 0;
  a.drop_n4 = d.drop_n4;
  a.cscale = d.cscale;
  a.rotate = d.rotate;
  a.LA = d.fuse_t ? d.LA : nullptr;
  a.ldla = d.ldla;
  a.R = d.fuse_t ? (int)d.K[1] : 0;
  a.t_alpha = d.t_alpha;
  dim3 grid((unsigned)(nbm * nbn), (unsigned)plan.splits, 1);
  const int al = d.a_strided ? 1 : 0, bl = d.b_kcontig ? 1 : 0;
  hipError_t e;
  switch (d.dtype) {
    case DT_BF16: e = gemm_launch_bf16(cfg, al, bl, a, grid, stream); break;
    case DT_F16: e = gemm_launch_f16(cfg, al, bl, a, grid, stream); break;
    case DT_F32: e = gemm_launch_f32(cfg, al, bl, a, grid, stream); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (plan.splits > 1)
    e = splitk_reduce_launch(d.dtype, scratch, plan.splits, (int)d.M, (int)d.N, d.C, d.ldc, d.D, d.ldd, d.alpha,
                             d.bias, d.mask_seg0 || d.mask_a ? DropMask{} : DropMask{d.drop_thr, d.drop_key, d.drop_cpr}, stream);
  return e;
}

hipError_t splitk_reduce_launch(int dtype, const float* partial, int splits, int M, int N, void* C,
                                int64_t ldc, const void* D, int64_t ldd, float alpha, const void* bias,
                                DropMask drop, hipStream_t s) {
  const int64_t quads = (int64_t)M * N / 4;
  int blocks = (int)((quads + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  switch (dtype) {
    case DT_BF16:
      launch_timed(splitk_reduce_kernel<__bf16>, dim3(blocks), dim3(256), 0, s, partial, splits, M, N,
                         static_cast<__bf16*>(C), ldc, static_cast<const __bf16*>(D), ldd, alpha,
                         static_cast<const __bf16*>(bias), drop.thr, drop.key, drop.cpr);
      break;
    case DT_F16:
      launch_timed(splitk_reduce_kernel<_Float16>, dim3(blocks), dim3(256), 0, s, partial, splits, M, N,
                         static_cast<_Float16*>(C), ldc, static_cast<const _Float16*>(D), ldd, alpha,
                         static_cast<const _Float16*>(bias), drop.thr, drop.key, drop.cpr);
      break;
    case DT_F32:
      launch_timed(splitk_reduce_kernel<float>, dim3(blocks), dim3(256), 0, s, partial, splits, M, N,
                         static_cast<float*>(C), ldc, static_cast<const float*>(D), ldd, alpha,
                         static_cast<const float*>(bias), drop.thr, drop.key, drop.cpr);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---- few-token forward ---------------------------------------------------------------------------------

// What few_run's two launches take, us, fitted to 2100 of them timed (301 layers, n 1 .. 256, 512 .. 11008 wide, r 8 .. 128, W from HBM, in
// every slicing; standard deviation 9 %).  The first: K tiles of one, two, ... workgroups on a compute unit, W once from HBM and once more
// from the caches for every further 64 rows, the partials, and what a second workgroup on some of the units costs while the others wait
// (64 x 8192 -> 8192: 195 workgroups 29 us, 260 40, 455 32).  The second (lora_finish.hpp): trips to memory, the partials, and what waves read
// of others' operands: X A's slices once for every block of columns and B once for every 16 rows, which is most of it for many rows at
// a high rank (48 x 4096 -> 11008 r 32 in two slices 4.0 us, 256 x 4096 -> 11008 r 128 17).  Over those layers the route taken is 1.9 % slower
// than the best of both routes and all slicings (4.6 % where neither W's further passes nor B's were counted: 245 x 4608 -> 9648 r 128 74.2 us for 51.4).
static double few_time_us(int64_t n, int64_t i, int64_t o, int64_t r, int splits, int64_t ktiles) {
  const int64_t nbm = (n + 63) / 64, nbn = (o + 127) / 128 + (r + 127) / 128, wgs = nbm * nbn * splits, rounds = wgs / 512, rest = wgs % 512;
  const double uneven = wgs > 256 && wgs < 512 ? (double)(512 - wgs) / 256.0 : 0.0;
  const double load = 2.0 * (double)rounds + (rest == 0 ? 0.0 : (rest <= 256 ? 1.0 : 2.0)), wmb = 2e-6 * (double)(i * o);
  const double first = 3.1 + wmb * (0.1 + 0.028 * (double)(nbm - 1) + 0.009 * uneven) + 0.42e-6 * (double)(n * i) +
                       (double)ktiles * (0.29 * load + 0.0044 * (double)(nbm - 1)) + 0.81e-6 * (double)n * (double)(o + r) * splits;
  const FinishShape f = finish_shape(n, o, r, splits);
  const double trips = (double)((splits + f.u - 1) / f.u);
  const double second = 2.8 + 0.93 * (trips - 1.0) + (r > 64 ? 0.9 : 0.0) + 0.62e-6 * (double)(n * o) * (splits + 1.0) +
                        0.28e-6 * (double)(n * r) * splits * (double)((o + f.cols - 1) / f.cols) + 0.2e-6 * (double)(r * o) * (double)((n + 15) / 16);
  return first + second;
}

// The slicing of the first launch whose partials fit the scratch the call has anyway.
FewPlan few_plan(int64_t n, int64_t i, int64_t o, int64_t r, size_t scratch_bytes) {
  FewPlan best;
  if (n < 1 || n > kFewMaxRows || r > kFewMaxR || n > (1LL << 30)) return best;
  const int64_t kt = (i + 63) / 64;
  for (int s = 1; s <= 16 && (s == 1 || kt / s >= 6); ++s) {
    const int64_t per = (kt + s - 1) / s;
    if ((kt + per - 1) / per != s) continue;  // no empty slice
    if ((size_t)s * (size_t)n * (size_t)(o + r) * sizeof(float) > scratch_bytes) break;
    const double us = few_time_us(n, i, o, r, s, per);
    if (best.splits == 0 || us < best.us) {
      best.splits = s;
      best.tiles_per_split = (int)per;
      best.us = us;
    }
  }
  return best;
}

hipError_t few_run(int dtype, const FewDesc& d, const FewPlan& plan, float* scratch, hipStream_t stream) {
  if (dtype == DT_F32 || plan.splits < 1 || scratch == nullptr || d.n < 1 || d.n > kFewMaxRows || d.r < 1 || d.r > kFewMaxR)
    return hipErrorInvalidValue;
  GemmArgs a{};
  a.A[0] = d.X; a.lda[0] = d.ldx;
  a.B[0] = d.W; a.ldb[0] = d.ldw;
  a.K[0] = (int)d.i;
  a.M = (int)d.n; a.N = (int)d.o;
  a.partial = scratch;
  a.partial_t = scratch + (size_t)plan.splits * (size_t)d.n * (size_t)d.o;
  a.tiles_per_split = plan.tiles_per_split;
  a.nbm = (int)((d.n + 63) / 64);
  a.nbn = (int)((d.o + 127) / 128);
  a.splits = plan.splits;
  a.alpha = 1.f;
  a.LA = d.A; a.ldla = d.lda; a.R = (int)d.r;
  const dim3 grid((unsigned)(a.nbm * (a.nbn + (a.R + 127) / 128)), (unsigned)plan.splits, 1);
  hipError_t e = dtype == DT_BF16 ? gemm_launch_bf16(CFG_MTM64, 0, 0, a, grid, stream) : gemm_launch_f16(CFG_MTM64, 0, 0, a, grid, stream);
  if (e != hipSuccess) return e;
  FinishArgs f{};
  f.partial = a.partial; f.partial_t = a.partial_t;
  f.B = d.B; f.ldb = d.ldb; f.bias = d.bias;
  f.C = d.Y; f.ldc = d.ldy; f.T = d.T; f.ldt = d.ldt;
  f.M = a.M; f.N = a.N; f.R = a.R; f.splits = plan.splits;
  f.t_alpha = d.t_alpha;
  return dtype == DT_BF16 ? finish_launch_bf16(f, stream) : finish_launch_f16(f, stream);
}

// ---- streaming kernel for the rank-r products -----------------------------------------------------

SkinnyPlan skinny_plan(int dtype, int nprob, const SkinnyDesc* d, size_t cap) {
  SkinnyPlan p;
  const int bk = dtype == DT_F32 ? 32 : 64;
  int64_t min_ktiles = 1 << 30, outs = 0, maxn = 0;
  for (int w = 0; w < nprob; ++w)
    if (d[w].N > maxn) maxn = d[w].N;
  p.rt = maxn <= 32 ? 1 : (maxn <= 64 ? 2 : 4);
  const bool masked = d[0].drop_thr != 0 || (nprob == 2 && d[1].drop_thr != 0);
  auto count = [&](int mb) {
    int64_t b = 0;
    for (int w = 0; w < nprob; ++w) b += (d[w].M + mb - 1) / mb;
    return b;
  };
  for (int w = 0; w < nprob; ++w) {
    const int64_t kt = (d[w].K + bk - 1) / bk;
    if (kt < min_ktiles) min_ktiles = kt;
    outs += d[w].M * d[w].N;
  }
  // 64-row workgroups (see skinny.hpp) where they fill more than half of the compute units, or where the contraction can be
  // split over them.  dA, dB in us, 64 rows / 32 rows: 2048 x (2048 + 2048) 12.4 / 8.9, 2048 x (4096 + 4096) 13.4 / 10.3, 4096
  // x (4096 + 4096) 18.8 / 15.6, 8192 x (4096 + 4096) 34 / 30.6, 8192 x (1024 + 4096) 27.7 (four slices) / 22.9; with more
  // blocks 2048 x (2048 + 8192) 15.1 / 16.6, 4096 x (2048 + 8192) 21.1 / 25.4, 8192 x (4096 + 6144) 33 / 48; with few and a long
  // contraction 8192 x (768 + 3072) 21.4 (four slices) / 24.0.  Masked ones (LoRA dropout) alike: 4096 x (8192 + 2048) 28.7 / 36.8, 8192 x (11008
  // + 4096) 59.0 / 75.4 (operands from HBM; plain 27.1 / 36.7 and 59.1 / 75.9).
  if (nprob == 2 && d[0].a_strided && d[1].a_strided && p.rt <= 2) {
    const int64_t b64 = count(64);
    if (b64 > 128 || (b64 <= 64 && min_ktiles >= 64)) p.mr = 2;
  }
  const int64_t blocks = count(32 * p.mr);
  // A masked problem of the [M,K] orientation whose chains of K tiles are the launch: alone, or next to an unmasked one of at most twice its
  // contraction where the blocks leave it half a compute unit or more.
  const SkinnyDesc& m = d[0].drop_thr != 0 ? d[0] : d[nprob - 1];
  const bool chains = masked && !d[0].a_strided && p.rt == 1 && (nprob == 1 || (blocks <= 256 && 2 * m.K >= (d[0].drop_thr != 0 ? d[1] : d[0]).K));
  // Split K over workgroups only when there are fewer workgroups than compute units, and keep >= 8 K tiles per wave and slice (T of
  // 5 x 3744, fp32, masked: 20.9 us in three slices, 30.8 whole), but twice as many for a masked pair that fills a quarter of the chip
  // whole ({Z1, T} of 2048 x (4096 + 4096) 15.1 in two slices, 14.2 whole).
  // (64-row workgroups: 128-160 of them without a split beat twice as many plus the reduce pass, and so do 32-row ones of a
  // pair that 64-row blocks do not fill.)
  // In the [M,K] orientation a launch of 16-bit or masked blocks of up to 32 columns takes no more slices than leave every workgroup a
  // compute unit: T r 16 of 5000 x 5464 19.2 us whole, 22.7 in two, 3232 x 8192 16.1 in two, 21.6 in three, 2560 x 8192 15.5 in three, 18.2
  // in four (in fp32 and with wider blocks a few beyond are no worse: {Z1, T} of 950 x (3000 + 3000), fp32, 17.3 in five, 22.7 whole).
  // 32 and more unmasked ones stay whole up to 64 K tiles: T of 2048 x 4096 12.7 us, 13.2 in two slices, {Z1, T} 12.0 and 13.1;
  // with more the reduce pass pays: Z1 of 1776 x 4536 19.3 us, 16.4 in two, T of 1240 x 5464 19.6 and 16.1, 2048 x 8192 18.4 in two, 16.9 in four.
  int64_t splits = 1;
  const bool half = nprob == 2 && d[0].a_strided && d[1].a_strided && p.rt <= 2;
  if (blocks < (half ? 128 : 224)) {
    const bool one_each = !d[0].a_strided && p.rt == 1 && (dtype != DT_F32 || chains);
    splits = one_each ? 256 / blocks : (256 + blocks - 1) / blocks;
    int64_t slice_max = min_ktiles / (chains && nprob == 2 && blocks >= 64 ? 64 : 32);
    if (slice_max < 1 || (one_each && !chains && blocks >= 32 && min_ktiles <= 64)) slice_max = 1;
    if (splits > slice_max) splits = slice_max;
    if (splits > 16) splits = 16;
  }
  while (splits > 1 && (size_t)splits * (size_t)outs * sizeof(float) > cap) --splits;
  p.splits = (int)splits;
  // 16 waves for masked chains of at least 48 K tiles that are not split, 4 for every other launch.  us on 16 and 4 waves, of 90 T and 67
  // {Z1, T} with 24 K tiles and more: T of 6795 x 10496 r 16 28.3 and 33.1, 490 x 3184 r 8 11.1 and 13.1; {Z1, T} of 2212 x (10496 + 768) 22.9
  // and 28.9, 104 x (3424 + 2048) 11.3 and 12.8.  Shorter or in slices: T of 6262 x 2704 r 32 13.3 and 12.0, 3822 x 4928 r 32 in two slices 18.5
  // and 16.5, 263 x 2304 fp32 in two 20.2 and 17.9.  All of them: 16 waves 2485 us, 4 waves 2553, so 2424.
  if (chains && splits == 1 && (m.K + bk - 1) / bk >= 48) p.nwv = 16;
  p.partial_bytes = splits > 1 ? (size_t)splits * (size_t)outs * sizeof(float) : 0;
  return p;
}

// T = (X o m) A alone with r > 32 (LoRA dropout), streaming kernel: a workgroup's chain of K tiles, one workgroup to a compute unit, never
// below the bytes at 4.8 TB/s.  Fitted to 287 launches (n 64 .. 7816, 512 .. 11008 wide, r 40 .. 128, 16 bits; standard deviation 6 %): 1954 x
// 1280 r 64 10.5 us (10.2 modelled), 3074 x 2304 r 48 13.0 (13.7), 280 x 2304 r 64 12.3 (13.7), 700 x 3000 r 96 23.7 (24.4).
static double masked_t_us(const SkinnyDesc& d, const SkinnyPlan& plan) {
  const int64_t wgs = (d.M + 31) / 32 * plan.splits;
  const double tiles = (double)(((d.K + 63) / 64 + 4 * plan.splits - 1) / (4 * plan.splits)), outs = (double)d.M * (double)d.N;
  const double chain = (plan.rt > 2 ? 9.3 + 1.26 * tiles : 5.8 + 0.88 * tiles) * (double)((wgs + 255) / 256);
  const double floor_us = 5.0 + 2.0 * ((double)d.M * d.K + (double)d.K * d.N + outs) / 4.8e6;
  return (chain > floor_us ? chain : floor_us) + (plan.splits > 1 ? 5.4 + outs * 8.0 * plan.splits / 7.5e6 : 0.0);
}

double skinny_time_us(int dtype, int nprob, const SkinnyDesc* d, const SkinnyPlan& plan) {
  if (nprob == 1 && dtype != DT_F32 && d[0].drop_thr != 0 && !d[0].a_strided && plan.rt > 1) return masked_t_us(d[0], plan);
  // Rates in TB/s of algorithmic bytes, measured (bf16): up to 32 columns the big operand streams; with 64 and 128 the
  // waves' re-reads of the short operand bind (paired launches at 8192 x (4096 + 11008) r 128: 118 us; at 4096 x (5120 +
  // 13824) r 64: 58 us), single launches fill less of the chip.
  const double e = dtype == DT_F32 ? 4.0 : 2.0;
  double bytes = 0, outs = 0;
  for (int w = 0; w < nprob; ++w) {
    bytes += e * ((double)d[w].M * d[w].K + (double)d[w].K * d[w].N + (double)d[w].M * d[w].N);
    outs += (double)d[w].M * d[w].N;
  }
  double rate = plan.rt == 1 ? (d[0].a_strided ? 4.4 : 4.8) : (plan.rt == 2 ? 2.8 : 2.1);
  if (nprob == 1) rate *= plan.rt == 1 ? 0.65 : 0.8;
  double us = (plan.rt == 1 || nprob == 1 ? 5.0 : 9.0) + bytes / (rate * 1e6);
  if (nprob == 1 && dtype != DT_F32 && !d[0].a_strided) {
    // few rows: a workgroup's four waves walk their K tiles one after the other, 0.35 / 0.62 / 1.27 us each with up to 32 / 64 /
    // 128 columns (T of 1 .. 256 rows: 4.7 / 5.7 / 7.7 us at K 512, 6.6 / 9.9 / 15.4 at 2048)
    const double tiles = (double)(((d[0].K + 63) / 64 + 4 * plan.splits - 1) / (4 * plan.splits));
    const double chain = plan.rt == 1 ? 4.4 + 0.35 * tiles : (plan.rt == 2 ? 5.8 + 0.62 * tiles : 6.9 + 1.27 * tiles);
    if (chain > us) us = chain;
  }
  const bool masked = d[0].drop_thr != 0 || (nprob == 2 && d[1].drop_thr != 0);
  for (int w = 0; w < nprob && masked && plan.rt > 1; ++w) {
    // The chains of a pair with a masked problem, whose own is longer, its mask arithmetic included.  Shorter by 20-30 % since skinny_body's
    // loads go stage after stage; but with launches priced as they are now ({Z1, T} of 3074 x (2304 + 1792) r 48 13.7 us, dA, dB of 8192 x
    // (4096 + 4096) r 64 41.6) and tiles as masked_tile_us prices them, 120 layers that neither was fitted to ran {Z1, T} in 2462 us in place
    // of 2482, dA, dB in 1984 of 1987, some of them 6 us slower (the best plan for each: 2388, 1903).
    const double tiles = (double)(((d[w].K + 63) / 64 + 4 * plan.splits - 1) / (4 * plan.splits));
    double chain = 0.0;
    if (d[w].drop_thr == 0) chain = d[w].a_strided ? 0.0 : (plan.rt == 2 ? 5.8 + 0.62 * tiles : 6.9 + 1.27 * tiles);
    else if (d[w].a_strided) chain = plan.rt == 2 ? 6.0 + 1.8 * tiles : 8.0 + 3.2 * tiles;
    else chain = plan.rt == 2 ? 5.8 + 1.4 * tiles : 6.9 + 2.2 * tiles;
    if (chain > us) us = chain;
  }
  return us + (plan.splits > 1 ? 4.0 + outs * 8.0 * plan.splits / 7.5e6 : 0.0);
}

// ---- rank-r products with r > 32 on the middle-sized kernel ------------------------------------------------------

// a streaming-kernel problem as the tile GEMM sees it: C^T = op(B)^T op(A) is turned back into C
GemmDesc rank_desc(int dtype, const SkinnyDesc& d) {
  GemmDesc g;
  g.dtype = dtype;
  g.alpha = d.alpha;
  g.C = d.C;
  g.ldc = d.ldc;
  g.K[0] = d.K;
  const bool t = d.trans_out != 0;  // both operands stored [K, .]
  g.a_strided = d.a_strided;
  g.b_kcontig = t ? 0 : d.b_kcontig;
  g.A[0] = t ? d.B : d.A; g.lda[0] = t ? d.ldb : d.lda;
  g.B[0] = t ? d.A : d.B; g.ldb[0] = t ? d.lda : d.ldb;
  g.M = t ? d.N : d.M;
  g.N = t ? d.M : d.N;
  g.rotate = g.a_strided ? 0 : 5;
  g.mask_a = d.drop_thr != 0;
  g.drop_thr = d.drop_thr; g.drop_key = d.drop_key; g.drop_cpr = d.drop_cpr;
  return g;
}

// One launch of narrow tiles over operands that come from HBM: 0.53 us per K tile and workgroup (0.45 where a tile's rows
// are whole lines of a [K, .] operand), twice that where two share a compute unit (see gemm_mt_pair_kernel); never below
// the operands' bytes at 4.8 TB/s.  Operands that the caches still hold (the activations of a short batch) arrive twice as
// fast: dA, dB of 1024 x 4096 r 64 take 9.7 us here, 17.5 on the streaming kernel.  Masked pairs (LoRA dropout; streaming kernel / here, reduce
// included): {Z1, T} of 700 x 3000 r 96 23.8 / 16 us, of 8192 x (4096 + 4096) r 64 35.5 / 35, dA, dB of that 41.6 / 36.
static double rank_time_us(bool a_strided, bool masked, int64_t wgs, int64_t ktiles, double bytes) {
  const int64_t rounds = wgs / 512, rest = wgs % 512;
  double tk = bytes < 32e6 ? 0.28 : (a_strided ? 0.45 : 0.53);
  if (masked) tk = 0.7;  // (priced as unmasked, {dA, dB} of 8192 x (4096 + 4096) r 64 take 41.9 us for 35.5, in fewer slices)
  const double us = (bytes < 32e6 ? 5.0 : 7.5) + (double)ktiles * tk * (double)(2 * rounds + (rest > 256 ? 2 : (rest > 0 ? 1 : 0)));
  const double floor_us = 5.0 + bytes / 4.8e6;
  return us > floor_us ? us : floor_us;
}

// The same for a pair on 128x128 tiles, one workgroup to a compute unit: they read the long operand once where 128x64 ones read it for every 64
// columns.  A K tile is 32 KB, 0.65 us at the 50 bytes a ns that a unit fetches (0.45 from the caches).
static double wide_rank_us(bool a_strided, bool masked, int64_t wgs, int64_t ktiles, double bytes) {
  const double tk = masked ? 0.8 : (bytes < 32e6 ? 0.45 : (a_strided ? 0.6 : 0.65));  // ({Z1, T} of 800 x (1024 + 1024) r 128, masked: 20.7 us whole)
  const double us = 7.5 + (double)((wgs + 255) / 256) * (double)ktiles * tk, floor_us = 5.0 + bytes / 4.8e6;
  return us > floor_us ? us : floor_us;
}

// T = (X o m) A alone on 128x64 tiles (LoRA dropout): K tiles of a workgroup, 1.7 times that where two share a compute unit, never below the bytes
// at 5.3 TB/s, and what its slices cost.  Fitted to 2000 launches of the layers that masked_t_us was (standard deviation 3 %): 700 x 3000 r 96 in
// ten slices 12.9 us, 23.7 on the streaming kernel; 1954 x 1280 r 64 in five 12.3 and 10.5, 3074 x 2304 r 48 in eight 13.9 and 13.0.
static double masked_tile_us(int64_t M, int64_t N, int64_t wgs, int64_t ktiles, int splits, double bytes) {
  const int64_t rounds = wgs / 512, rest = wgs % 512;
  const double us = 4.9 + (double)ktiles * 0.68 * (1.7 * (double)rounds + (rest > 256 ? 1.7 : (rest > 0 ? 1.0 : 0.0))), floor_us = 5.0 + bytes / 5.3e6;
  return (us > floor_us ? us : floor_us) + (splits > 1 ? 5.2 + (double)M * (double)N * (8.0 * splits + 2.0) / 5.4e6 : 0.0);
}

static bool rank_shape_ok(int dtype, const SkinnyDesc& d) {
  return dtype != DT_F32 && d.N > 32 && d.M > 32 && (d.drop_thr == 0 || (!d.b_kcontig && !d.trans_out));
}

bool rank_plan(int dtype, const SkinnyDesc& d, size_t cap, GemmPlan* plan, double* plan_us, double slice_us) {
  if (!rank_shape_ok(dtype, d)) return false;
  const GemmDesc g = rank_desc(dtype, d);
  const int cfg = g.N == d.N ? CFG_MTN64 : CFG_MTM64;
  const int64_t nbm = (g.M + kTileBM[cfg] - 1) / kTileBM[cfg], nbn = (g.N + kTileBN[cfg] - 1) / kTileBN[cfg];
  const int64_t kt = (g.K[0] + 63) / 64;
  const double bytes = 2.0 * ((double)g.M * g.K[0] + (double)g.K[0] * g.N + (double)g.M * g.N);
  double best = skinny_time_us(dtype, 1, &d, skinny_plan(dtype, 1, &d));
  bool found = false;
  for (int s = 1; s <= 16 && (s == 1 || kt / s >= 4); ++s) {
    const int64_t per = (kt + s - 1) / s;
    if ((kt + per - 1) / per != s) continue;  // no empty slice
    const size_t part = s > 1 ? (size_t)s * (size_t)g.M * (size_t)g.N * sizeof(float) : 0;
    if (part > cap) break;
    const double us = (d.drop_thr != 0 && !g.a_strided ? masked_tile_us(g.M, g.N, nbm * nbn * s, per, s, bytes)
                                                       : rank_time_us(g.a_strided != 0, d.drop_thr != 0, nbm * nbn * s, per, bytes) + split_time_us(g.M, g.N, s)) +
                      (s > 1 ? slice_us : 0.0);
    if (us >= best) continue;
    best = us;
    found = true;
    *plan = GemmPlan{};
    plan->cfg = cfg;
    plan->bk = 64;
    plan->bm = kTileBM[cfg];
    plan->bn = kTileBN[cfg];
    plan->nbm = (int)nbm;
    plan->nbn = (int)nbn;
    plan->splits = s;
    plan->tiles_per_split = (int)per;
    plan->partial_bytes = part;
  }
  if (found && plan_us != nullptr) *plan_us = best;
  return found;
}

bool mt_pair_plan(int dtype, const SkinnyDesc* d, size_t cap, MtPairPlan* plan, double alone_us, double slice_us) {
  if (!rank_shape_ok(dtype, d[0]) || !rank_shape_ok(dtype, d[1])) return false;
  int64_t tiles[2], kt[2];
  double bytes = 0, best = 1e30;
  for (int w = 0; w < 2; ++w) {
    const GemmDesc g = rank_desc(dtype, d[w]);
    plan->cfg[w] = g.N == d[w].N ? CFG_MTN64 : CFG_MTM64;
    tiles[w] = ((g.M + kTileBM[plan->cfg[w]] - 1) / kTileBM[plan->cfg[w]]) * ((g.N + kTileBN[plan->cfg[w]] - 1) / kTileBN[plan->cfg[w]]);
    kt[w] = (g.K[0] + 63) / 64;
    bytes += 2.0 * ((double)g.M * g.K[0] + (double)g.K[0] * g.N + (double)g.M * g.N);
  }
  // the launches the kernel is built for (gemm_launch.inc)
  const bool z = !d[0].a_strided && !d[1].a_strided && d[0].b_kcontig && !d[1].b_kcontig && !d[0].trans_out && !d[1].trans_out;
  const bool g = d[0].a_strided && d[1].a_strided && plan->cfg[0] == CFG_MTN64 && plan->cfg[1] == CFG_MTM64;
  if (!z && !g) return false;
  const int64_t longest = kt[0] > kt[1] ? kt[0] : kt[1];
  for (int s = 1; s <= 16 && (s == 1 || longest / s >= 4); ++s) {
    const int64_t per = (longest + s - 1) / s;
    int64_t sp[2], tps[2];
    size_t part = 0;
    double us = 0;
    int64_t wgs = 0;
    for (int w = 0; w < 2; ++w) {
      sp[w] = (kt[w] + per - 1) / per;
      tps[w] = (kt[w] + sp[w] - 1) / sp[w];
      sp[w] = (kt[w] + tps[w] - 1) / tps[w];
      wgs += tiles[w] * sp[w];
      if (sp[w] > 1) {
        part += (size_t)sp[w] * (size_t)d[w].M * (size_t)d[w].N * sizeof(float);
        us += (double)d[w].M * (double)d[w].N * (8.0 * sp[w] + 2.0) / 7.5e6;
      }
    }
    if (part > cap) break;
    us += rank_time_us(d[0].a_strided != 0, d[0].drop_thr != 0 || d[1].drop_thr != 0, wgs, per, bytes) + (part > 0 ? 3.0 + slice_us : 0.0);
    if (us < best) {
      best = us;
      plan->partial_bytes = part;
      for (int w = 0; w < 2; ++w) { plan->splits[w] = (int)sp[w]; plan->tiles_per_split[w] = (int)tps[w]; }
    }
  }
  // r > 64: 128x128 tiles, each product cut into about as many slices as make its workgroups equally long: {Z1, Z2} of 8192 x (11008 +
  // 4096) r 128 96.5 us on 128x64 tiles, 74.4 so; 4096 x (2048 + 8192) 36.7 and 33.7; dA, dB of 8192 x (4096 + 4096) 41.6 and 35.6.
  // (A lone product gains nothing: T of 8192 x 4096 27.8 and 28.7, of 8192 x 11008 62.2 and 61.6.)  dA, dB over fewer than 44 MB stay on
  // the narrow ones, which want half the slices: 41 such layers from 32 MB on took 722 us so and 769 on 128x128 (1480 x (5808 + 4920)
  // r 72 12.5 and 15.3; the other way at most 18.1 and 16.3), 47 of 44 .. 64 MB 1048 and 1038.
  if (d[0].N > 64 && d[1].N > 64 && (z || bytes >= 44e6)) {
    int64_t wide[2];
    for (int w = 0; w < 2; ++w) wide[w] = ((d[w].M + 127) / 128) * ((d[w].N + 127) / 128);
    for (int s = 1; s <= 16 && (s == 1 || longest / s >= 8); ++s) {
      const int64_t per = (longest + s - 1) / s;
      int64_t sp[2], tps[2], wgs = 0, most = 0;
      size_t part = 0;
      double us = 0;
      for (int w = 0; w < 2; ++w) {
        sp[w] = (kt[w] + per / 2) / per;
        if (sp[w] < 1) sp[w] = 1;
        tps[w] = (kt[w] + sp[w] - 1) / sp[w];
        sp[w] = (kt[w] + tps[w] - 1) / tps[w];  // no empty slice
        wgs += wide[w] * sp[w];
        if (tps[w] > most) most = tps[w];
        if (sp[w] > 1) {
          part += (size_t)sp[w] * (size_t)d[w].M * (size_t)d[w].N * sizeof(float);
          us += (double)d[w].M * (double)d[w].N * (8.0 * sp[w] + 2.0) / 7.5e6;
        }
      }
      if (part > cap) break;
      us += wide_rank_us(d[0].a_strided != 0, d[0].drop_thr != 0 || d[1].drop_thr != 0, wgs, most, bytes) + (part > 0 ? 3.0 + slice_us : 0.0);
      if (us < best) {
        best = us;
        plan->wide = true;
        plan->partial_bytes = part;
        for (int w = 0; w < 2; ++w) { plan->splits[w] = (int)sp[w]; plan->tiles_per_split[w] = (int)tps[w]; }
      }
    }
  }
  plan->us = best;
  return best < (alone_us > 0.0 ? alone_us : skinny_time_us(dtype, 2, d, skinny_plan(dtype, 2, d)));
}

hipError_t mt_pair_run(int dtype, const SkinnyDesc* d, const MtPairPlan& plan, float* scratch, hipStream_t stream) {
  if (dtype == DT_F32) return hipErrorInvalidValue;
  GemmArgs a[2] = {};
  SkinnyArgs r{};
  r.nprob = 2;
  r.mr = 1;
  r.nwv = 4;
  float* part = scratch;
  unsigned grid = 0;
  int al = 0, bl[2] = {0, 0};
  for (int w = 0; w < 2; ++w) {
    const GemmDesc g = rank_desc(dtype, d[w]);
    const int64_t a_rows = g.a_strided ? g.K[0] : g.M, b_rows = g.b_kcontig ? g.N : g.K[0];
    if (a_rows * g.lda[0] >= (1LL << 30) || b_rows * g.ldb[0] >= (1LL << 30)) return hipErrorInvalidValue;  // callers check sk_ok
    a[w].A[0] = g.A[0]; a[w].B[0] = g.B[0];
    a[w].lda[0] = g.lda[0]; a[w].ldb[0] = g.ldb[0];
    a[w].K[0] = (int)g.K[0];
    a[w].M = (int)g.M; a[w].N = (int)g.N;
    a[w].C = g.C; a[w].ldc = g.ldc;
    a[w].alpha = g.alpha;
    a[w].rotate = g.a_strided ? 0 : 5;
    a[w].mask_a = g.mask_a ? 1 : 0;
    a[w].drop_thr = g.drop_thr; a[w].drop_key = g.drop_key; a[w].drop_cpr = g.drop_cpr;
    a[w].splits = plan.splits[w];
    a[w].tiles_per_split = plan.tiles_per_split[w];
    const int64_t bm = plan.wide ? 128 : kTileBM[plan.cfg[w]], bn = plan.wide ? 128 : kTileBN[plan.cfg[w]];
    a[w].nbm = (int)((g.M + bm - 1) / bm);
    a[w].nbn = (int)((g.N + bn - 1) / bn);
    al = g.a_strided;
    bl[w] = g.b_kcontig;
    grid += (unsigned)(a[w].nbm * a[w].nbn * a[w].splits);
    SkinnyProblem& P = r.p[w];  // the reduce pass: [slices][M][N] -> C, scaled
    P.C = g.C; P.ldc = g.ldc;
    P.M = (int)g.M; P.N = (int)g.N;
    P.alpha = g.alpha;
    if (plan.splits[w] > 1) {
      if (scratch == nullptr) return hipErrorInvalidValue;
      a[w].partial = part;
      P.partial = part;
      part += (size_t)plan.splits[w] * (size_t)g.M * (size_t)g.N;
    }
  }
  hipError_t e = dtype == DT_BF16 ? mt_pair_launch_bf16(al, bl[0], bl[1], plan.wide, a[0], a[1], grid, stream)
                                  : mt_pair_launch_f16(al, bl[0], bl[1], plan.wide, a[0], a[1], grid, stream);
  if (e != hipSuccess || (plan.splits[0] <= 1 && plan.splits[1] <= 1)) return e;
  return dtype == DT_BF16 ? skinny_reduce_launch_bf16(r, plan.splits[0], plan.splits[1], stream)
                          : skinny_reduce_launch_f16(r, plan.splits[0], plan.splits[1], stream);
}

hipError_t skinny_run(int dtype, int nprob, const SkinnyDesc* d, const SkinnyPlan& plan, float* scratch,
                      hipStream_t stream) {
  if (nprob < 1 || nprob > 2) return hipErrorInvalidValue;
  if (plan.splits > 1 && scratch == nullptr) return hipErrorInvalidValue;
  const int bk = dtype == DT_F32 ? 32 : 64;
  SkinnyArgs a{};
  a.nprob = nprob;
  a.mr = plan.mr;
  a.nwv = plan.nwv;
  if (plan.mr != 1 && !(plan.mr == 2 && nprob == 2 && d[0].a_strided && d[1].a_strided && plan.rt <= 2)) return hipErrorInvalidValue;
  float* part = scratch;
  for (int w = 0; w < nprob; ++w) {
    SkinnyProblem& P = a.p[w];
    if (d[w].N > 32 * plan.rt || d[w].M < 1 || d[w].K < 1) return hipErrorInvalidValue;
    P.A = d[w].A; P.B = d[w].B; P.C = d[w].C;
    P.lda = d[w].lda; P.ldb = d[w].ldb; P.ldc = d[w].ldc;
    P.M = (int)d[w].M; P.N = (int)d[w].N; P.K = (int)d[w].K;
    P.a_strided = d[w].a_strided; P.b_kcontig = d[w].b_kcontig; P.trans_out = d[w].trans_out;
    P.alpha = d[w].alpha;
    P.drop_thr = d[w].drop_thr; P.drop_key = d[w].drop_key; P.drop_cpr = d[w].drop_cpr;
    const int mb = 32 * plan.mr;
    P.row_blocks = (int)((d[w].M + mb - 1) / mb);
    {
      const int64_t esz = dtype == DT_F32 ? 4 : 2;
      const int64_t a_rows = d[w].a_strided ? d[w].K : d[w].M, a_cols = d[w].a_strided ? d[w].M : d[w].K;
      const int64_t b_rows = d[w].b_kcontig ? d[w].N : d[w].K, b_cols = d[w].b_kcontig ? d[w].K : d[w].N;
      const int64_t ab = ((a_rows - 1) * d[w].lda + a_cols) * esz, bb = ((b_rows - 1) * d[w].ldb + b_cols) * esz;
      if (ab >= (1LL << 31) || bb >= (1LL << 31)) return hipErrorInvalidValue;  // callers check skinny_fits()
      P.a_bytes = (int)ab;
      P.b_bytes = (int)bb;
    }
    const int64_t kt = (d[w].K + bk - 1) / bk;
    P.tiles_per_split = (int)((kt + plan.splits - 1) / plan.splits);
    P.partial = nullptr;
    if (plan.splits > 1) {
      P.partial = part;
      part += (size_t)plan.splits * (size_t)d[w].M * (size_t)d[w].N;
    }
  }
  // one slot list per XCD: ceil(R0/8) + ceil(R1/8) workgroups on each (see skinny_kernel)
  int64_t per_xcd = 0;
  for (int w = 0; w < nprob; ++w) per_xcd += (a.p[w].row_blocks + 7) / 8;
  dim3 grid((unsigned)(8 * per_xcd), (unsigned)plan.splits, 1);
  switch (dtype) {
    case DT_BF16: return skinny_launch_bf16(plan.rt, a, grid, plan.splits, stream);
    case DT_F16: return skinny_launch_f16(plan.rt, a, grid, plan.splits, stream);
    case DT_F32: return skinny_launch_f32(plan.rt, a, grid, plan.splits, stream);
    default: return hipErrorInvalidValue;
  }
}

// ---- M = W + A B ------------------------------------------------------------------------------------

hipError_t merge_run(int dtype, const MergeDesc& d, hipStream_t stream) {
  if (!merge_ok(dtype, d.R) || d.I < 1 || d.O < 1 || d.R < 1) return hipErrorInvalidValue;
  MergeArgs a{};
  a.W = d.W; a.A = d.A; a.B = d.B; a.M = d.M;
  a.ldw = d.ldw; a.lda = d.lda; a.ldb = d.ldb; a.ldm = d.ldm;
  a.I = (int)d.I; a.O = (int)d.O; a.R = (int)d.R;
  a.blocks_per_wg = 1;
  a.alpha = d.alpha;
  a.b_trans = d.b_trans;
  a.wcol = d.wcol;
  a.sq_partial = d.sq_partial;
  a.drop_thr = d.drop_thr; a.drop_key = d.drop_key; a.drop_cpr = d.drop_cpr;
  return dtype == DT_BF16 ? merge_launch_bf16(a, stream) : merge_launch_f16(a, stream);
}

}  // namespace rl
