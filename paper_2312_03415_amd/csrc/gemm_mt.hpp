// Matrix-core kernel for the middle-sized contractions of the LoRA layer (16-bit types): the products whose 256x256 tiles
// would leave compute units idle (a few hundred to a few thousand tokens) and the rank-r products with r > 32, in every
// operand layout of Eq. 1 / Eq. 3 (X W, dY W^T, X^T dY and their K-concatenated forms; arxiv 2312.03415).
//
// What bounds it.  A 128x128 tile needs 32 KB of operands per K tile of 64 and 512 cycles of v_mfma_f32_16x16x32 per
// wave: the compute unit's path from L1 to LDS (64 bytes a cycle) and its LDS reads (128 bytes a cycle) are then as busy
// as the matrix cores, where the generic engine (gemm_engine.hpp) also passes every operand byte through registers,
// issues half-size products and waits for memory once per K tile.  A K tile of a 128x128 tile takes a workgroup alone on the chip
// 0.31 .. 0.39 us against 0.21 of products (44 bytes a cycle fetched), one of 256 0.51, which is why 256x128 wins as soon as its tiles
// fill the chip.  It is not LDS (waves that split K instead of the tile read and write 64 KB of it per K tile instead of 96: 45.3 /
// 44.6 us against 42.1 / 41.0 at 1024 x 4096 x 4096 NN / NT) and with operands from HBM not power (42 us on zeros too; from the caches
// 37-42 and 33-34 on zeros).
// Measured (us a launch, bf16, N(0,1); this kernel / generic engine / 256x256 kernel, each at its best K split):
// 1024 x 4096 x 4096 NN 40.7 / 65.4 / 51.3, NT 36.2 / 59.1 / 47.5; 512 x 4096 x 4096 24.2 / 39.8 / 35.4;
// 1237 x 2056 x 5464 46.3 / 53.4 / 52.9; 4096 x 256 x 8192 28.8 / 38.5 / 36.6; 4096 x 2048 x 8192 112 / 183 / 117.
//
//  - Output tile BM x BN per workgroup, 4 wavefronts (2 x 2), K tile 64.  LDS is a ring of NS stages filled by 16-byte
//    LDS-DMA loads (global memory straight to LDS, no registers); NS - 1 K tiles are in flight.
//  - A K tile is two K steps of 32.  The fragments of the next K step are read while the current one is multiplied
//    (double-buffered registers), across the barrier too: behind the first MFMAs of K step 1 the wave waits for its own
//    loads of the next tile and for the workgroup, reads the next tile's first fragments, and refills the stage that has
//    just been released, its loads spread between the MFMAs.
//  - Everything outside the matrices (rows beyond M / N, k beyond K, tiles beyond the last) is fetched from an offset past
//    the end of the buffer descriptor: the range check returns zeros, so there is no masking and every K tile issues the
//    same number of loads (the waits count them).
//  - LDS-DMA writes lane l's 16 bytes at base + 16 l: rows cannot be padded, so bank conflicts are avoided by an XOR
//    swizzle on the global-address side:
//      K-contiguous tile [rows][8 chunks]: chunk c of row q in slot c ^ ((q >> 1) & 7)
//      K-strided tile [64 k-rows][BX / 8 chunks]: chunk c of k-row q in slot c ^ f(q), f distinct over the eight k-rows
//      that 32 lanes of a transposing read touch
//  - The LDS reads are inline assembly (reads the compiler tracks would wait for all outstanding LDS-DMA loads); between
//    their issue and the wait for them there is no branch, and their results are combined only behind the wait.
//  - XA build: the few-token forward (lora_finish.hpp).  The adapter's A stands next to W as more tile columns, so that one
//    launch reads X and W once and leaves the fp32 partials of X W and of T = X A.
//  - Epilogue: the accumulators of 16 rows at a time pass through wave-private LDS (the ring, drained), so that a lane
//    owns eight consecutive columns of a row: every option (scale, dropout mask, addend, bias) works on those, and a store
//    instruction writes whole 128-byte lines.
#pragma once
#include <type_traits>
#include <utility>

#include "gemm_mc64.hpp"

namespace rl {

template <int AL, int BL, int BM_, int BN_, int NS_>
struct MtTile {
  static constexpr int BM = BM_, BN = BN_, NS = NS_, BK = 64;
  static constexpr int NT = 256;
  static constexpr bool A_STR = (AL == 1), B_STR = (BL == 0);
  static constexpr int WTM = BM / 2, WTN = BN / 2;  // a wave's sub-tile
  static constexpr int TM = WTM / 16, TN = WTN / 16;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int IA = A_BYTES / 4096, IB = B_BYTES / 4096;  // 1 KB loads per wave and K tile
  static constexpr int LPT = IA + IB;
  static constexpr int EPI_LD = WTN + 4;                           // fp32 row of the epilogue's staging area
  static constexpr int EPI_BYTES = 4 * 16 * EPI_LD * 4;
  static constexpr int RING_BYTES = NS * STAGE_BYTES;
  static constexpr int LDS_BYTES = RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
  static_assert((NS - 1) * LPT < 64, "the load counter holds 63");
};

// swizzle of a K-strided tile with BX columns: 16-byte chunk index of k-row q is XORed with this
template <int BX>
__device__ __forceinline__ int mt_swz(int q) {
  if constexpr (BX == 64) return 2 * (((q >> 1) & 1) | (((q >> 3) & 1) << 1));  // 128-byte rows: the parity of q is a bank bit already
  else return 2 * ((q & 3) | (((q >> 3) & 1) << 2));
}

template <typename T> struct Mma16;
template <> struct Mma16<__bf16> {
  static __device__ __forceinline__ f32x4 mma(i32x4 rowop, i32x4 colop, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, rowop), __builtin_bit_cast(bf16x8, colop), c, 0, 0, 0);
  }
};
template <> struct Mma16<_Float16> {
  static __device__ __forceinline__ f32x4 mma(i32x4 rowop, i32x4 colop, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, rowop), __builtin_bit_cast(f16x8, colop), c, 0, 0, 0);
  }
};

// A 16-wide operand fragment as the LDS reads deliver it: one 16-byte read, or two transposing 8-byte reads that are put
// together only behind the wait (a register copy before it would copy what has not arrived)
template <bool STRIDED> struct MtFrag;
template <> struct MtFrag<false> {
  i32x4 v;
  __device__ __forceinline__ i32x4 get() const { return v; }
  __device__ __forceinline__ void touch() { asm volatile("" : "+v"(v)); }
};
template <> struct MtFrag<true> {
  i32x2 lo, hi;
  __device__ __forceinline__ i32x4 get() const { return i32x4{lo[0], lo[1], hi[0], hi[1]}; }
  __device__ __forceinline__ void touch() { asm volatile("" : "+v"(lo), "+v"(hi)); }
};

// SEGMASK: dX = m o (Z1 A^T) + dY W^T of a layer with LoRA dropout in one launch.  Segment 0 is the rank-r one; behind its last K
// tile (of this K slice) the dropped accumulators are zeroed (a lane holds four consecutive columns of a row: one hash), and
// the other segment is added to what is left.
// COLSCALE: C = (the products) diag(cscale) + bias, see gemm_mc64.hpp
// MASKA: A is the input X of a layer with LoRA dropout (T = (X o m) A, dA = (X o m)^T Z1; r > 32).  A wave masks the chunks that it
// loaded itself, in LDS, between its wait for them and the barrier that hands them over: two hashes a chunk, each formed once.
template <typename T, int AL, int BL, int BM, int BN, int NS, bool XA, bool SEGMASK = false, bool COLSCALE = false, bool MASKA = false>
__device__ __forceinline__ void gemm_mt_body(const GemmArgs& g, const int bx, const int by) {
  static_assert(!XA || (AL == 0 && BL == 0), "X [M,K], W and A [K,.]");
  static_assert(!MASKA || (BM == 128 && !XA && !SEGMASK), "four chunks of X per lane");
  using P = MtTile<AL, BL, BM, BN, NS>;
  constexpr int BK = P::BK, TM = P::TM, TN = P::TN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  unsigned char* const smem = smem_raw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int s16 = lane & 15, grp = lane >> 4;

  // ---- workgroup -> output tile: a contiguous run of tiles per XCD (own L2), walked in bands of 8 tile rows
  int m0, n0;
  [[maybe_unused]] bool t_tile = false;  // XA: this tile's columns are A's
  {
    const int nbn = XA ? g.nbn + (g.R + BN - 1) / BN : g.nbn;
    const int total = g.nbm * nbn;
    const int x = bx & 7, slot = bx >> 3, q = total >> 3, rem = total & 7;
    const int id = x * q + (x < rem ? x : rem) + slot;
    constexpr int BAND = 8;
    const int per_band = BAND * nbn;
    const int band = id / per_band, first_m = band * BAND;
    const int band_rows = (g.nbm - first_m) < BAND ? (g.nbm - first_m) : BAND;
    const int in_band = id - band * per_band;
    m0 = (first_m + in_band % band_rows) * BM;
    int tile_n = in_band / band_rows;
    if constexpr (XA) {
      t_tile = tile_n >= g.nbn;
      if (t_tile) tile_n -= g.nbn;
    }
    n0 = tile_n * BN;
  }
  const int N = XA && t_tile ? g.R : g.N;
  const void* const B0 = XA && t_tile ? g.LA : g.B[0];
  const int64_t ldb0 = XA && t_tile ? g.ldla : g.ldb[0];
  // ---- this workgroup's K tiles (over both segments; `by` slices them)
  const int K0 = g.K[0], K1 = g.K[1];
  const int nt0 = (K0 + BK - 1) / BK, nt1 = (K1 + BK - 1) / BK;
  const int u0 = by * g.tiles_per_split;
  int u1 = u0 + g.tiles_per_split;
  if (u1 > nt0 + nt1) u1 = nt0 + nt1;

  // ---- load cursor.  Per-lane byte offsets, one per load; OOB lanes hold an offset past every descriptor's end
  // (operands are smaller than 2 GiB, checked on the host, so that adding steps to it cannot wrap into range).
  constexpr uint32_t OOB = 0x80000000u;
  auto extent_bytes = [&](bool strided, int rows_or_cols, int K, int64_t ld) -> int {
    if (K <= 0) return 0;
    const int64_t e = strided ? ((int64_t)(K - 1) * ld + rows_or_cols) : ((int64_t)(rows_or_cols - 1) * ld + K);
    return (int)(e * 2);
  };
  auto make_rsrc = [&](const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
  };
  __amdgpu_buffer_rsrc_t rsA = make_rsrc(g.A[0], 0), rsB = rsA;
  uint32_t offA[P::IA], offB[P::IB], stepA = 0, stepB = 0;
  // next tile to load, tiles still to load, tile at which the state below must be rebuilt.  The walk may start inside the
  // range and wrap around (GemmArgs::rotate): row blocks of a rank-r product that all read the same columns of a
  // power-of-two wide matrix at once crowd a few memory channels.
  int left = u1 - u0, cu = u0, cnext = u0;
  if (g.rotate != 0 && left > 0) cu += (int)((uint32_t)(m0 / BM * g.rotate) % (uint32_t)left);
  auto cursor_setup = [&]() {
    if (left <= 0) {  // beyond the last tile: loads of nothing
      stepA = stepB = 0;
#pragma unroll
      for (int j = 0; j < P::IA; ++j) offA[j] = OOB;
#pragma unroll
      for (int j = 0; j < P::IB; ++j) offB[j] = OOB;
      cnext = 0x7fffffff;
      return;
    }
    const int seg = cu < nt0 ? 0 : 1;
    const int Ks = seg ? K1 : K0;
    const int k0 = (cu - (seg ? nt0 : 0)) * BK;
    const int kvalid = Ks - k0;
    const uint32_t lda = (uint32_t)(seg ? g.lda[1] : g.lda[0]), ldb = (uint32_t)(seg ? g.ldb[1] : ldb0);
    rsA = make_rsrc(seg ? g.A[1] : g.A[0], extent_bytes(P::A_STR, g.M, Ks, lda));
    rsB = make_rsrc(seg ? g.B[1] : B0, extent_bytes(P::B_STR, N, Ks, ldb));
    stepA = 2u * (P::A_STR ? (uint32_t)BK * lda : (uint32_t)BK);
    stepB = 2u * (P::B_STR ? (uint32_t)BK * ldb : (uint32_t)BK);
    auto offset = [&](bool strided, int cpr_strided, int swz_strided_row, int p, int base, int dim, uint32_t ld) -> uint32_t {
      if (!strided) {
        const int row = p >> 3, col = ((p & 7) ^ ((row >> 1) & 7)) << 3;
        return (base + row < dim && col < kvalid) ? 2u * ((uint32_t)(base + row) * ld + (uint32_t)(k0 + col)) : OOB;
      }
      const int row = p / cpr_strided, col = ((p % cpr_strided) ^ swz_strided_row) << 3;
      return (row < kvalid && base + col < dim) ? 2u * ((uint32_t)(k0 + row) * ld + (uint32_t)(base + col)) : OOB;
    };
#pragma unroll
    for (int j = 0; j < P::IA; ++j) {
      const int p = (wave * P::IA + j) * 64 + lane;
      offA[j] = offset(P::A_STR, BM / 8, mt_swz<BM>(p / (BM / 8)), p, m0, g.M, lda);
    }
#pragma unroll
    for (int j = 0; j < P::IB; ++j) {
      const int p = (wave * P::IB + j) * 64 + lane;
      offB[j] = offset(P::B_STR, BN / 8, mt_swz<BN>(p / (BN / 8)), p, n0, N, ldb);
    }
    // rebuilt at the end, at a segment switch, in front of a segment's partial last tile and behind it
    cnext = u1;
    if (kvalid < BK) {
      cnext = cu + 1;
    } else {
      const int seg_end = seg ? nt0 + nt1 : nt0;
      if (seg_end < cnext) cnext = seg_end;
      if (Ks % BK != 0 && seg_end - 1 < cnext) cnext = seg_end - 1;
    }
    if (cu + left < cnext) cnext = cu + left;
  };
  auto cursor_advance = [&]() {
    ++cu;
    --left;
    if (__builtin_expect(cu == cnext, 0)) {
      if (cu == u1) cu = u0;
      cursor_setup();
    } else {
#pragma unroll
      for (int j = 0; j < P::IA; ++j) offA[j] += stepA;
#pragma unroll
      for (int j = 0; j < P::IB; ++j) offB[j] += stepB;
    }
  };
  // load j (a constant) of the cursor's tile into stage st: first the A half's, then the B half's
  auto issue_load = [&](int st, auto j_c) {
    constexpr int j = decltype(j_c)::value;
    constexpr bool isB = j >= P::IA;
    constexpr int jj = isB ? j - P::IA : j;
    unsigned char* dst = smem + st * P::STAGE_BYTES + (isB ? P::A_BYTES + wave * (P::IB * 1024) : wave * (P::IA * 1024)) + jj * 1024;
    if constexpr (isB) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (mc_lds_void_t*)dst, 16, offB[jj], 0, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (mc_lds_void_t*)dst, 16, offA[jj], 0, 0, 0);
  };

  // ---- fragment addresses (bytes inside a stage).  MFMA 16x16x32: lane l carries row / column l % 16 of its block and the
  // eight k 8 (l / 16) .. + 7 of the K step (see gemm_mc64.hpp for both orientations)
  constexpr int NFA = P::A_STR ? TM : 2, NFB = P::B_STR ? TN : 2;
  uint32_t fragA[NFA], fragB[NFB];
  {
    const int sw = (s16 >> 1) & 7, kr = 8 * grp + (s16 >> 2);
    if constexpr (!P::A_STR) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) fragA[ks] = (uint32_t)((wm * P::WTM + s16) * 128 + (((4 * ks + grp) ^ sw) << 4));
    } else {
#pragma unroll
      for (int b = 0; b < TM; ++b)
        fragA[b] = (uint32_t)(kr * (BM * 2) + ((wm * (P::WTM / 8) + 2 * b + ((s16 & 3) >> 1)) ^ mt_swz<BM>(kr)) * 16 + 8 * (s16 & 1));
    }
    if constexpr (!P::B_STR) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) fragB[ks] = (uint32_t)(P::A_BYTES + (wn * P::WTN + s16) * 128 + (((4 * ks + grp) ^ sw) << 4));
    } else {
#pragma unroll
      for (int b = 0; b < TN; ++b)
        fragB[b] = (uint32_t)(P::A_BYTES + kr * (BN * 2) + ((wn * (P::WTN / 8) + 2 * b + ((s16 & 3) >> 1)) ^ mt_swz<BN>(kr)) * 16 + 8 * (s16 & 1));
    }
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)((mc_lds_void_t*)smem);

  MtFrag<P::A_STR> fa[2][TM];
  MtFrag<P::B_STR> fb[2][TN];
  auto read_one = [&](auto& out, const auto& fr, uint32_t soff, auto strided_c, auto bx_c, auto blk_c, auto ks_c) {
    constexpr bool strided = decltype(strided_c)::value;
    constexpr int bx = decltype(bx_c)::value, blk = decltype(blk_c)::value, ks = decltype(ks_c)::value;
    if constexpr (!strided) {
      const uint32_t addr = lds_base + soff + fr[ks];
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(out.v) : "v"(addr), "i"(blk * 2048));
    } else {
      const uint32_t addr = lds_base + soff + fr[blk];
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(out.lo) : "v"(addr), "i"(ks * 64 * bx));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(out.hi) : "v"(addr), "i"(ks * 64 * bx + 8 * bx));
    }
  };
  // read number r (a constant) of K step ks's fragments into buffer buf: A and B fragments in turn
  constexpr int NR = TM + TN;
  auto read_frag_n = [&](auto buf_c, auto r_c, auto ks_c, uint32_t soff) {
    constexpr int buf = decltype(buf_c)::value, r = decltype(r_c)::value;
    // B fragments first (the first row of products needs all of them and one of A)
    if constexpr (r < TN)
      read_one(fb[buf][r], fragB, soff, std::bool_constant<P::B_STR>{}, std::integral_constant<int, BN>{}, std::integral_constant<int, r>{}, ks_c);
    else
      read_one(fa[buf][r - TN], fragA, soff, std::bool_constant<P::A_STR>{}, std::integral_constant<int, BM>{}, std::integral_constant<int, r - TN>{}, ks_c);
  };
  auto wait_frags = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int a = 0; a < TM; ++a) fa[buf][a].touch();
#pragma unroll
    for (int b = 0; b < TN; ++b) fb[buf][b].touch();
  };

  // MASKA: the dropped elements of this lane's chunks of X zeroed, K tile t of the (one) segment in stage st, which have arrived
  [[maybe_unused]] int tile_k = cu;  // the tile that is handed over next (in the order of the load cursor)
  auto mask_tile = [&](int st) {
    if constexpr (MASKA) {
      const uint32_t addr = lds_base + (uint32_t)(st * P::STAGE_BYTES + wave * (P::IA * 1024) + lane * 16);
      i32x4 c[4];
      asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:1024\n\tds_read_b128 %2, %4 offset:2048\n\t"
                   "ds_read_b128 %3, %4 offset:3072\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(c[0]), "=&v"(c[1]), "=&v"(c[2]), "=&v"(c[3]) : "v"(addr) : "memory");
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = (wave * P::IA + j) * 64 + lane;
        uint32_t lane_g, tile_g;  // the chunk's group of columns: row drop_cpr + column / 4
        if constexpr (!P::A_STR) {
          const int row = p >> 3;
          lane_g = (uint32_t)(m0 + row) * g.drop_cpr + (uint32_t)(((p & 7) ^ ((row >> 1) & 7)) << 1);
          tile_g = (uint32_t)(tile_k * (BK / 4));
        } else {
          const int row = p / (BM / 8);
          lane_g = (uint32_t)row * g.drop_cpr + ((uint32_t)m0 >> 2) + (uint32_t)(((p % (BM / 8)) ^ mt_swz<BM>(row)) << 1);
          tile_g = (uint32_t)(tile_k * BK) * g.drop_cpr;
        }
        c[j] = drop_chunk<T>(c[j], lane_g + tile_g, g.drop_key, g.drop_thr);
      }
      asm volatile("ds_write_b128 %4, %0\n\tds_write_b128 %4, %1 offset:1024\n\tds_write_b128 %4, %2 offset:2048\n\t"
                   "ds_write_b128 %4, %3 offset:3072\n\ts_waitcnt lgkmcnt(0)"
                   :: "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(addr) : "memory");
      if (++tile_k == u1) tile_k = u0;
    }
  };

  f32x4 acc[TM][TN];  // lane l: row l % 16, columns 4 (l / 16) .. + 3 of each 16x16 block
  static_for<TM * TN>([&](auto e) { acc[decltype(e)::value / TN][decltype(e)::value % TN] = f32x4{0.f, 0.f, 0.f, 0.f}; });

#define MT_FENCE() __builtin_amdgcn_sched_barrier(0)
  constexpr int Q = TM * TN;                      // MFMAs per K step
  constexpr int SY = Q >= 16 ? 4 : (Q >= 4 ? 1 : 0);  // K step 1: MFMAs issued ahead of the wait and the barrier
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto mma = [&](auto buf_c, auto q_c) {
    constexpr int buf = decltype(buf_c)::value, q = decltype(q_c)::value;
    // left to the compiler, a workgroup whose waves may use more than 256 registers keeps the accumulators in the
    // accumulation registers and copies each to a vector register and back around its product: those are tied by hand
    if constexpr (TM * TN > 16) Elem16<T>::mma(acc[q / TN][q % TN], fb[buf][q % TN].get(), fa[buf][q / TN].get());
    else acc[q / TN][q % TN] = Mma16<T>::mma(fb[buf][q % TN].get(), fa[buf][q / TN].get(), acc[q / TN][q % TN]);
    MT_FENCE();
  };
  // MFMAs [FROM, Q) of a K step out of buffer buf, with the next K step's reads spread over the first three quarters of
  // them and, if LOADS, a K tile's loads over all of them
  auto kstep = [&](auto buf_c, auto from_c, auto ks_next_c, uint32_t soff, auto loads_c, int st) {
    constexpr int FROM = decltype(from_c)::value, W = Q - FROM, RW = W >= 4 ? (W * 3) / 4 : W;
    using NB = std::integral_constant<int, 1 - decltype(buf_c)::value>;
    static_for<W>([&](auto w_c) {
      constexpr int w = decltype(w_c)::value;
      mma(buf_c, std::integral_constant<int, FROM + w>{});
      constexpr int r0 = w < RW ? NR * w / RW : NR, r1 = w < RW ? NR * (w + 1) / RW : NR;
      static_for<r1 - r0>([&](auto r_c) { read_frag_n(NB{}, std::integral_constant<int, r0 + decltype(r_c)::value>{}, ks_next_c, soff); });
      if constexpr (decltype(loads_c)::value) {
        constexpr int l0 = P::LPT * w / W, l1 = P::LPT * (w + 1) / W;
        static_for<l1 - l0>([&](auto l_c) { issue_load(st, std::integral_constant<int, l0 + decltype(l_c)::value>{}); });
      }
      MT_FENCE();
    });
  };

  if (u0 < u1) {
    // ---- prologue: NS tiles on their way, the first landed for everyone, its first fragments in registers
    cursor_setup();
    for (int s = 0; s < NS; ++s) {
      static_for<P::LPT>([&](auto j) { issue_load(s, j); });
      cursor_advance();
    }
    MT_FENCE();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(mc_wait_imm((NS - 1) * P::LPT, true));  // loads return in order
    mask_tile(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    MT_FENCE();
    static_for<NR>([&](auto r) { read_frag_n(I0{}, r, I0{}, 0u); });
    wait_frags(I0{});
    MT_FENCE();
    int st = 0;
    for (int u = u0; u < u1; ++u) {
      const int stn = st + 1 == NS ? 0 : st + 1;
      const uint32_t soff = (uint32_t)(st * P::STAGE_BYTES), soffn = (uint32_t)(stn * P::STAGE_BYTES);
      // K step 0: MFMAs and the reads of K step 1
      kstep(I0{}, I0{}, I1{}, soff, std::false_type{}, 0);
      // K step 1: the next tile has landed and this tile's stage is free behind the barrier
      wait_frags(I1{});
      MT_FENCE();
      static_for<SY>([&](auto q) { mma(I1{}, q); });
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(mc_wait_imm((NS - 2) * P::LPT, true));
      mask_tile(stn);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      MT_FENCE();
      kstep(I1{}, std::integral_constant<int, SY>{}, I0{}, soffn, std::true_type{}, st);
      // no LDS read is in flight across a branch (the cursor's, the loop's)
      wait_frags(I0{});
      MT_FENCE();
      cursor_advance();
      if constexpr (SEGMASK) {
        if (u < nt0 && (u == nt0 - 1 || u == u1 - 1)) {  // wave-uniform: the last tile of segment 0 in this slice
          if constexpr (TM * TN > 16) asm volatile("s_nop 7\n\ts_nop 7");
          MT_FENCE();
          // (opaque: nothing of this is worth keeping in registers around the K loop)
          uint32_t group = (uint32_t)(m0 + wm * P::WTM + s16) * g.drop_cpr + g.drop_n4 + (uint32_t)((n0 + wn * P::WTN) >> 2) + (uint32_t)grp;
          asm volatile("" : "+v"(group));
          static_for<TM * TN>([&](auto e) {
            constexpr int a = decltype(e)::value / TN, b = decltype(e)::value % TN;
            acc[a][b] = drop_acc4(acc[a][b], group + 4 * b, g.drop_key, g.drop_thr);
            if constexpr (b == TN - 1) {
              group += 16u * g.drop_cpr;
              asm volatile("" : "+v"(group));
            }
            MT_FENCE();
          });
          if constexpr (TM * TN > 16) asm volatile("s_nop 7");
          MT_FENCE();
        }
      }
      st = stn;
    }
  }
  // the stage loads of nothing may still be in flight: the ring becomes the epilogue's staging area behind this
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(mc_wait_imm(0, true));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  MT_FENCE();

  if constexpr (TM * TN > 16) asm volatile("s_nop 7\n\ts_nop 7");  // the last products' results (not the compiler's to guard)
  MT_FENCE();
  // ---- epilogue: 16 rows of the wave at a time through LDS (fp32), then eight columns of a row per lane
  constexpr int LD = P::EPI_LD, LPR = P::WTN / 8, RPP = 64 / LPR;  // lanes per row, rows per pass
  float* const stg = reinterpret_cast<float*>(smem) + wave * (16 * LD);
  const int prow = lane / LPR, pcol = (lane % LPR) * 8;
  const int n = n0 + wn * P::WTN + pcol;
  const bool n_ok = n < N;  // N is a multiple of 8: the eight columns are valid together
  float* const part = XA && t_tile ? g.partial_t : g.partial;
  const bool split = XA || part != nullptr;
  float b8[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) b8[e] = 0.f;
  if (g.bias != nullptr && !split && n_ok) {
    const i32x4 v = *reinterpret_cast<const i32x4*>(static_cast<const T*>(g.bias) + n);
    const T* t8 = reinterpret_cast<const T*>(&v);
#pragma unroll
    for (int e = 0; e < 8; ++e) b8[e] = (float)t8[e];
  }
  [[maybe_unused]] f32x4 c8[2];
  if constexpr (COLSCALE) {
    c8[0] = c8[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (n_ok) {
      c8[0] = *reinterpret_cast<const f32x4*>(g.cscale + n);
      c8[1] = *reinterpret_cast<const f32x4*>(g.cscale + n + 4);
    }
  }
#pragma unroll
  for (int a = 0; a < TM; ++a) {
#pragma unroll
    for (int b = 0; b < TN; ++b) *reinterpret_cast<f32x4*>(stg + s16 * LD + 16 * b + 4 * grp) = acc[a][b];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
    for (int p = 0; p < 16 / RPP; ++p) {
      const int r = p * RPP + prow, m = m0 + wm * P::WTM + a * 16 + r;
      f32x4 v0 = *reinterpret_cast<const f32x4*>(stg + r * LD + pcol);
      f32x4 v1 = *reinterpret_cast<const f32x4*>(stg + r * LD + pcol + 4);
      if (m < g.M && n_ok) {
        if (split) {
          float* dst = part + ((int64_t)by * g.M + m) * N + n;
          *reinterpret_cast<f32x4*>(dst) = v0;
          *reinterpret_cast<f32x4*>(dst + 4) = v1;
        } else {
          if constexpr (COLSCALE) { v0 *= c8[0]; v1 *= c8[1]; }
          if (g.alpha != 1.f) { v0 *= g.alpha; v1 *= g.alpha; }
          if (!SEGMASK && !MASKA && g.drop_thr != 0u) {
            uint32_t k0[4], k1[4];
            const uint32_t grp4 = (uint32_t)m * g.drop_cpr + (uint32_t)(n >> 2);
            drop_keep4(grp4, g.drop_key, g.drop_thr, k0);
            drop_keep4(grp4 + 1, g.drop_key, g.drop_thr, k1);
#pragma unroll
            for (int e = 0; e < 4; ++e) { v0[e] = k0[e] ? v0[e] : 0.f; v1[e] = k1[e] ? v1[e] : 0.f; }
          }
          if (g.D != nullptr) {
            const i32x4 dv = *reinterpret_cast<const i32x4*>(static_cast<const T*>(g.D) + (int64_t)m * g.ldd + n);
            const T* d8 = reinterpret_cast<const T*>(&dv);
#pragma unroll
            for (int e = 0; e < 4; ++e) { v0[e] += (float)d8[e]; v1[e] += (float)d8[4 + e]; }
          }
          T o8[8];
#pragma unroll
          for (int e = 0; e < 4; ++e) { o8[e] = from_f32<T>(v0[e] + b8[e]); o8[4 + e] = from_f32<T>(v1[e] + b8[4 + e]); }
          *reinterpret_cast<i32x4*>(static_cast<T*>(g.C) + (int64_t)m * g.ldc + n) = *reinterpret_cast<const i32x4*>(o8);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  }
#undef MT_FENCE
}

template <typename T, int AL, int BL, int BM, int BN, int NS, bool XA = false>
__global__ __launch_bounds__(256, (BM * BN <= 128 * 128 ? 2 : 1)) void gemm_mt_kernel(GemmArgs g) {
  gemm_mt_body<T, AL, BL, BM, BN, NS, XA>(g, (int)blockIdx.x, (int)blockIdx.y);
}

template <typename T, int AL, int BL, int BM, int BN, int NS>
__global__ __launch_bounds__(256, (BM * BN <= 128 * 128 ? 2 : 1)) void gemm_mt_colscale_kernel(GemmArgs g) {
  gemm_mt_body<T, AL, BL, BM, BN, NS, false, false, true>(g, (int)blockIdx.x, (int)blockIdx.y);
}
template <typename T, int AL, int BL, int BM, int BN, int NS>
__global__ __launch_bounds__(256, 2) void gemm_mt_maska_kernel(GemmArgs g) {
  gemm_mt_body<T, AL, BL, BM, BN, NS, false, false, false, true>(g, (int)blockIdx.x, (int)blockIdx.y);
}
template <typename T, int AL, int BL, int BM, int BN, int NS>
__global__ __launch_bounds__(256, (BM * BN <= 128 * 128 ? 2 : 1)) void gemm_mt_segmask_kernel(GemmArgs g) {
  gemm_mt_body<T, AL, BL, BM, BN, NS, false, true>(g, (int)blockIdx.x, (int)blockIdx.y);
}

// Two products in one launch (Z1 = dY B^T with Z2 = X A, dA = X^T Z1 with dB = Z2^T dY; r > 32): each fills a part of the
// chip only, so they run side by side.  Workgroups [0, tiles0 splits0) belong to the first.  Tiles of 128x64 for a
// product with r columns, 64x128 for one with r rows; beyond r = 64 also 128x128 for both (mt_pair_plan), which fetch the long
// operand once.  Bound by what a compute unit fetches from HBM: ~45 bytes a ns
// however many stages are in flight (three and six measure the same), so that a K tile's 24 KB take 0.53 us.  The streaming
// kernel (skinny.hpp), whose waves re-read the short operand for every 32 rows, against this one: dA, dB of 8192 x (4096 +
// 11008) r 128 129 / 61 us, Z1, Z2 120 / 97; dA, dB of 4096 x (5120 + 13824) r 64 59 / 29, of 1024 x 4096 r 64 17.5 / 9.7.
// DROPM: bit w = the A operand of product w is X under LoRA dropout
template <typename T, int AL, int BL0, int BL1, int BM0, int BN0, int BM1, int BN1, int DROPM>
__device__ __forceinline__ void gemm_mt_pair_body(const GemmArgs& g0, const GemmArgs& g1) {
  const int tiles0 = g0.nbm * g0.nbn, c0 = tiles0 * g0.splits;
  const int id = (int)blockIdx.x;
  if (id < c0) {
    gemm_mt_body<T, AL, BL0, BM0, BN0, 3, false, false, false, (DROPM & 1) != 0>(g0, id % tiles0, id / tiles0);
  } else {
    const int tiles1 = g1.nbm * g1.nbn, j = id - c0;
    gemm_mt_body<T, AL, BL1, BM1, BN1, 3, false, false, false, (DROPM & 2) != 0>(g1, j % tiles1, j / tiles1);
  }
}
template <typename T, int AL, int BL0, int BL1, int BM0, int BN0, int BM1, int BN1>
__global__ __launch_bounds__(256, 2) void gemm_mt_pair_kernel(GemmArgs g0, GemmArgs g1) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass has no use for the body and instantiates it twice over (gemm_mt_kernel's)
  gemm_mt_pair_body<T, AL, BL0, BL1, BM0, BN0, BM1, BN1, 0>(g0, g1);
#endif
}
template <typename T, int AL, int BL0, int BL1, int BM0, int BN0, int BM1, int BN1, int DROPM>
__global__ __launch_bounds__(256, 2) void gemm_mt_pair_maska_kernel(GemmArgs g0, GemmArgs g1) {
#if defined(__HIP_DEVICE_COMPILE__)
  gemm_mt_pair_body<T, AL, BL0, BL1, BM0, BN0, BM1, BN1, DROPM>(g0, g1);
#endif
}

}  // namespace rl
