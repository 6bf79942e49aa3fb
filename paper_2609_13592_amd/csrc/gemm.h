#pragma once
// Matrix-core GEMM, y[b, n] = sum_k W[n, k] x[b, k] for a batch of rows b: W
// and x streamed into LDS by direct-to-LDS loads.
//
// The unit is RTL 16-row tiles of each of G consecutive pages and one slice of
// K.  K is walked in stages of 64 columns; W's rows and x's rows of a stage go
// from memory straight into two rings of stages in LDS (buffer_load ... lds:
// no register holds data in flight).  Half of the wavefronts load W and half
// load x: a wavefront's loads complete in order, so one that loaded both would
// wait for W, which comes from HBM, whenever it needs x, which comes from L2.
// One load instruction moves 1 KiB: lane i writes LDS bytes [16 i, 16 i + 16)
// of the block at M0, and chooses which global 16 bytes it fetches, so an
// instruction reads 8 whole 128-byte rows of a stage and lays them out
// swizzled: row r (0..15) of a tile keeps its 16-byte chunk c at position
// c ^ (r >> 1) of its 128 bytes, so that the lanes which a 16-byte LDS read
// serves together (0-3, 12-15, 20-23 and 24-27 of 32, and the others) find
// their rows on distinct banks (an earlier layout, c ^ r, cost four conflict
// cycles a read).  The compiler does not see these loads (inline assembly: it
// would otherwise wait for all of them before any LDS read); the waits on
// them are explicit, in issue order.  Out-of-range lanes (rows past the page,
// columns outside the page or the slice, batch rows past B) write zeros into
// LDS, as out-of-range register loads return zeros.
//
// The wavefronts form a grid over the unit's row tiles and batch tiles, each
// with the full sums of its tiles over the slice, so there is no
// cross-wavefront reduction.  Rows cut by a page boundary and split-K slices
// go through partial buffers that launch_sums (or the consumer) adds in order.
//
// What bounds it: W's stream up to about 32 batch rows (28672 x 4096: 41-42
// us, 5.7 TB/s at 4..32 rows in cold weights, against 46 at 8 and 50 at 16 for
// 16-row units that staged W through registers), then the requests that a
// compute unit's L1 keeps in flight, of which x takes 2 BT and W 2 G RTL KiB a
// stage (the same matrix at 64 / 128 / 256 rows: 44 / 55 / 77 us; 59 / 69 / 90
// before the two roles, the start columns, the step-ahead fragment reads and
// the conflict-free layout).  So a unit holds as many rows as the grid allows:
// two pages of 8192 columns (57344 x 8192, 256 rows: 257 us, 287 with one
// page), four of 28672 (8192 x 28672, 64 rows: 94-100 us; 145 with 64-row units).
#include <algorithm>
#include <type_traits>

#include "gemm_plan.h"
#include "gemv_common.h"
#include "lds_dma.h"

namespace bst {
namespace gv {
namespace {

// The 2-D arrangement of the NW wavefronts over a unit's G pages of RTL row
// tiles and BT batch tiles (16 row groups + batch groups): the one with the
// fewest products per wavefront, then the fewest fragments read per 32-column
// step; a row group lies on one page.
template <int BT, int RTL, int G, int NW>
constexpr int dma_wave_grid() {
  int best = -1, cost = 1 << 30;
  for (int wr = NW; wr >= 1; --wr)
    for (int wb = NW / wr; wb >= 1; --wb) {
      if (wr % G || RTL % (wr / G) || BT % wb) continue;
      const int rw = G * RTL / wr, bw = BT / wb, c = 64 * rw * bw + rw + bw;
      if (c < cost) best = 16 * wr + wb, cost = c;
    }
  return best;
}
// Whether a wavefront of `tiles` 16 x 16 tiles keeps its sums in blocks: a
// second set of sums, for which 24 and 32 tiles leave no registers.
constexpr bool gemm_block_sums(int tiles) { return tiles <= 16; }
template <int BT, int RTL, int G, int NW>
struct GemmCfg {
  static constexpr int kWStage = 2 * G * RTL * kDmaBlk, kXStage = 2 * BT * kDmaBlk;
  static constexpr int kXs = gemm_x_stages(BT, G * RTL), kWs = gemm_w_stages(BT, G * RTL);
  static constexpr int kWRing = kWs * kWStage, kXRing = kXs * kXStage;
  static constexpr int kGrid = dma_wave_grid<BT, RTL, G, NW>();
  static constexpr int WR = kGrid / 16, WB = kGrid % 16;
  // sums in blocks, in the unit and, the same order being owed, in its host
  // sub-units
  static constexpr bool kBlocks = gemm_block_sums(G * RTL / WR * (BT / WB));
  // batch groups of a host sub-unit (one row tile)
  static constexpr int kHostWB = BT < NW ? BT : NW;
  static_assert(kGrid > 0 && kWs >= 2, "no wavefront grid or ring fits the unit");
  static_assert(kHostSpans * kSpan * 2 * kDmaBlk <= kWRing, "a host sub-unit's ring");
};
// Wait until at most `stages` (0 .. M) stages of Q loads each are outstanding
// for this wavefront (0 for fewer).
template <int M, int Q>
__device__ __forceinline__ void wait_stages(int stages) {
  if constexpr (M <= 0) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm<0>());
  } else {
    if (stages >= M)
      __builtin_amdgcn_s_waitcnt(vmcnt_imm<M * Q>());
    else
      wait_stages<M - 1, Q>(stages);
  }
}


typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ bf16x8_t lds16(lds_char* p) {
  return *(__attribute__((address_space(3))) bf16x8_t*)(p);
}

// One unit of the GEMM, on NW wavefronts.  With G > 1 every page fits one unit
// (G pages, one unit), and pages of the other tier are left out of it.
//
// HOST: the unit is one 16-row tile of one page of a unit (sub-unit unit_in % RTL of unit
// unit_in / RTL), so a page read over the host link, whose loads wait far
// longer than HBM's, spreads over RTL times more workgroups; every output
// still sums the same columns in the same order, so the results do not depend
// on which pages are on the host.
template <int BT, int RTL, int G, int NW, bool HOST>
__device__ __forceinline__ void gemm_dma_unit(const GemvParams& P, int page_in, int unit_in,
                                              lds_char* smem) {
  using C = GemmCfg<BT, RTL, G, NW>;
  constexpr int H = NW / 2;           // wavefronts that load W, and that load x
  constexpr int HW = HOST ? H : H / G;     // of which load one page's W
  constexpr int kWb = HOST ? 2 * kSpan : 2 * RTL;  // W blocks of a stage (span) and page
  constexpr int kXb = 2 * BT;              // x blocks of a stage
  constexpr int kWStage = kWb * (HOST ? 1 : G) * kDmaBlk;
  constexpr int kWs = HOST ? kHostSpans : C::kWs;  // stages (spans) of W's ring
  constexpr int kWRing = kWs * kWStage;
  constexpr int kWq = (kWb + HW - 1) / HW, kXq = (kXb + H - 1) / H;  // loads of one, at most
  const int page0 = __builtin_amdgcn_readfirstlane(page_in);  // HOST: the page, else the first
  const int uin = __builtin_amdgcn_readfirstlane(unit_in);
  const int unit = HOST ? uin / RTL : uin;
  const int j = unit / P.S, slice = unit % P.S;
  const int64_t K = P.K;
  const int64_t total = static_cast<int64_t>(P.N) * K;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int lrow = lane & 15, lgrp = lane >> 4;
  // the rows of page page0 + g in this unit: [rbase, r_hi], of which the page
  // holds elements [pe0, pe1); none (rbase > r_hi) past the last page, and for
  // a page of the other tier
  struct Rows {
    int64_t pe0, pe1, r_lo, r_hi, rbase;
  };
  auto rows_of = [&](int g) {
    Rows r;
    const int page = page0 + g;
    r.pe0 = static_cast<int64_t>(page) * kPageElems;
    r.pe1 = min(r.pe0 + kPageElems, total);
    r.r_lo = r.pe0 / K;
    r.r_hi = (r.pe1 - 1) / K;  // inclusive
    r.rbase = r.r_lo + static_cast<int64_t>(j) * (16 * RTL) + (HOST ? 16 * (uin % RTL) : 0);
    if (G > 1 && !HOST &&
        (page >= P.n_pages || (!P.address_order && page_tier(P, page) == BOOST_TIER_HOST)))
      r.rbase = r.r_hi + 1;
    return r;
  };
  if constexpr (G == 1 || HOST) {
    const Rows r = rows_of(0);
    if (r.rbase > r.r_hi) return;  // uniform over the workgroup
  } else {
    bool any = false;
    for (int g = 0; g < G; ++g) {
      const Rows r = rows_of(g);
      any = any || r.rbase <= r.r_hi;
    }
    if (!any) return;  // uniform over the workgroup
  }

  const int64_t ksl = (K + P.S - 1) / P.S;
  const int64_t kslice = (ksl + 63) / 64 * 64;
  const int k_beg = static_cast<int>(min(K, slice * kslice));
  const int width = static_cast<int>(min(K, k_beg + kslice)) - k_beg;
  const int nst = (width + 63) / 64;
  // First stage of this unit: units start at different columns and wrap.  The
  // rows of a matrix lie a power of two apart, so units that all walked the
  // same columns together would meet on the same few memory channels.
  const int rot = nst > 0 ? ((page0 / G) * P.units_per_page + unit) % nst : 0;
  // the order in which W is loaded: the stages from rot on, wrapping; on host
  // the spans that hold them (the span of rot comes first with its columns from
  // rot on, and once more at the end with those before)
  const int spans = (nst + kSpan - 1) / kSpan;
  const int w_loads = HOST ? spans + (rot % kSpan != 0) : nst;

  // loads: half of the wavefronts load W, the others x, so that each waits for
  // its own operand's stages only (a wavefront's loads complete in order).
  // Lane i of an instruction for block b fetches row i / 8 of the block and
  // the chunk that it stores at position i % 8 (the swizzle above).
  const bool wl = wave < H;  // uniform
  const int lg = wl && G > 1 && !HOST ? wave / HW : 0;  // page of a W-loading wavefront
  const int lw = wl ? wave - lg * HW : wave - H;        // its place among those of the same blocks
  const Rows lr = rows_of(lg);
  const bool some = lr.rbase <= lr.r_hi;  // else nothing is read (a resource of no bytes)
  const __amdgpu_buffer_rsrc_t rs =
      wl ? make_rsrc_uniform(page_addr(P, some ? page0 + lg : page0),
                             some ? static_cast<uint32_t>((lr.pe1 - lr.pe0) * 2) : 0)
         : make_rsrc_uniform(P.x, static_cast<uint32_t>(static_cast<int64_t>(P.B) * K * 2));
  constexpr int kQ = kWq > kXq ? kWq : kXq;
  // blocks per stage (uniform; may be 0)
  const int mine = wl ? (kWb - lw + HW - 1) / HW : (kXb - lw + H - 1) / H;
  const int brow = lane >> 3;
  // the lane's first column in a stage for a block of even number (odd: ^ 32)
  const int col0 = 8 * ((lane & 7) ^ (brow >> 1));
  static_assert(H % 2 == 0 && (HW % 2 == 0 || HW == 1), "block parity of a load");
  auto col = [&](int i) {  // of a wavefront's i-th load
    return col0 ^ (32 * ((HW == 1 && wl ? i : lw) & 1));
  };
  // host W: block b holds rows 2 b and 2 b + 1 of the tile, 32 chunks of each;
  // chunk c of row r at position c ^ r
  auto host_row = [&](int i) { return 2 * (lw + HW * i) + (lane >> 5); };
  auto host_col = [&](int i) { return 8 * ((lane & 31) ^ host_row(i)); };
  uint32_t off[kQ];
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    // row of the unit, or batch row
    const int64_t r8 = HOST && wl ? host_row(i) : 8 * (lw + (wl ? HW : H) * i) + brow;
    const int c = HOST && wl ? host_col(i) : col(i);
    // a row begun on the previous page gets a wrapped (huge) offset, so its
    // columns before the page read as zero
    if (wl)
      off[i] = lr.rbase + r8 > lr.r_hi
                   ? kOOB
                   : static_cast<uint32_t>(((lr.rbase + r8) * K - lr.pe0 + k_beg + c) * 2);
    else
      off[i] = r8 >= P.B ? kOOB : static_cast<uint32_t>((r8 * K + k_beg + c) * 2);
  }
  const uint32_t ring0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem)) +
                         (wl ? lg * kWb * kDmaBlk : C::kWRing) + lw * kDmaBlk;
  const uint32_t ring1 = ring0 + (wl ? kWRing : C::kXRing);
  uint32_t to = ring0;
  int at = HOST && wl ? rot / kSpan : rot;  // the stage (span) that the next issue loads
  int span = 0;                             // host: its number in the order
  auto issue = [&] {
    if (HOST && wl) {
      const int c = 64 * kSpan * at;
      const int lo = span == 0 ? 64 * rot : 0, hi = span == spans ? 64 * rot : width;
#pragma unroll
      for (int i = 0; i < kWq; ++i) {
        const int k = c + host_col(i);
        load16_lds(rs, (off[i] + static_cast<uint32_t>(2 * c)) | (k >= lo && k < hi ? 0u : kOOB),
                   to + i * HW * kDmaBlk);
      }
      ++span;
      at = at + 1 == spans ? 0 : at + 1;
      to = to + kWStage == ring1 ? ring0 : to + kWStage;
      return;
    }
    const uint32_t c = 64 * at;
    // past the slice: zeros
    const uint32_t oob0 = static_cast<int>(c) + col(0) < width ? 0u : kOOB;
    const uint32_t oob1 = HW > 1 ? oob0 : (static_cast<int>(c) + col(1) < width ? 0u : kOOB);
    if (wl) {
      if (P.w_once) {
#pragma unroll
        for (int i = 0; i < kWq; ++i) {
          if (kWb % HW != 0 && i >= mine) break;  // uniform
          load16_lds_nt(rs, (off[i] + 2 * c) | (i & 1 ? oob1 : oob0), to + i * HW * kDmaBlk);
        }
      } else {
#pragma unroll
        for (int i = 0; i < kWq; ++i) {
          if (kWb % HW != 0 && i >= mine) break;  // uniform
          load16_lds(rs, (off[i] + 2 * c) | (i & 1 ? oob1 : oob0), to + i * HW * kDmaBlk);
        }
      }
      to += kWStage;
    } else {
#pragma unroll
      for (int i = 0; i < kXq; ++i) {
        if (kXb % H != 0 && i >= mine) break;  // uniform
        load16_lds(rs, (off[i] + 2 * c) | oob0, to + i * H * kDmaBlk);
      }
      to += C::kXStage;
    }
    at = at + 1 == nst ? 0 : at + 1;
    to = to == ring1 ? ring0 : to;
  };
  // wait until `left` stages of this wavefront's operand may be outstanding
  auto landed = [&](int left) {
    if (wl) {
      if (kWb % HW == 0 || mine == kWq)
        wait_stages<kWs - 1, kWq>(left);
      else if (kWq > 1 && mine > 0)
        wait_stages<kWs - 1, (kWq > 1 ? kWq - 1 : 1)>(left);
    } else {
      if (kXb % H == 0 || mine == kXq)
        wait_stages<C::kXs - 1, kXq>(left);
      else if (kXq > 1 && mine > 0)
        wait_stages<C::kXs - 1, (kXq > 1 ? kXq - 1 : 1)>(left);
    }
  };
  const int depth = wl ? kWs : C::kXs, loads = wl ? w_loads : nst;

  // fragment reads: lane l takes row l % 16 of a tile (block 2 tile + h,
  // h = l % 16 / 8, block row l % 8) and 8 columns at chunk 4 sub + l / 16
  // of the stage, at position chunk ^ (l % 16 / 2)
  const int r8 = lrow & 7, hb = lrow >> 3;
  const int fx = hb * kDmaBlk + r8 * 128 + ((lgrp ^ (lrow >> 1)) << 4);  // sub 1: ^ 64
  // products: the NW wavefronts form a WR x WB grid over the unit's G RTL row
  // tiles and BT batch tiles; wavefront w takes row tiles [RW (w / WB), + RW)
  // and batch tiles [BW (w % WB), + BW)  (a host sub-unit: one row tile, the
  // batch tiles over WB wavefronts; the others only load)
  constexpr int WR = HOST ? 1 : C::WR;
  constexpr int WB = HOST ? C::kHostWB : C::WB;
  constexpr int RT = HOST ? 1 : G * RTL, RW = RT / WR, BW = BT / WB;
  static_assert(RW * WR == RT && BW * WB == BT && (HOST || RTL % RW == 0), "wavefront grid");
  const int t_row = RW * (wave / WB), t_bat = BW * (wave % WB);
  const bool computes = WR * WB == NW || wave < WR * WB;  // uniform over the wavefront
  const int wa = 2 * t_row * kDmaBlk + fx;
  const int xa = C::kWRing + 2 * t_bat * kDmaBlk + fx;

  f32x4_t acc[RW][BW];
#pragma unroll
  for (int a = 0; a < RW; ++a)
#pragma unroll
    for (int t = 0; t < BW; ++t) acc[a][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  struct Frags {
    bf16x8_t w[RW], x[BW];
  };
  // (host: row l % 16 of the span, chunk 8 (stage % 4) + 4 sub + l / 16)
  const int hx = lrow * 128 * kSpan + ((lgrp ^ lrow) << 4);
  auto read = [&](Frags& f, uint32_t ws, uint32_t xs, int sub, int stage) {
    lds_char* const pw =
        smem + ws + (HOST ? hx ^ ((stage % kSpan) * 128 + sub * 64) : wa ^ (sub * 64));
    lds_char* const px = smem + xs + (xa ^ (sub * 64));
#pragma unroll
    for (int a = 0; a < RW; ++a) f.w[a] = lds16(pw + a * 2 * kDmaBlk);
#pragma unroll
    for (int t = 0; t < BW; ++t) f.x[t] = lds16(px + t * 2 * kDmaBlk);
  };
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (int t = 0; t < BW; ++t)
#pragma unroll
      for (int a = 0; a < RW; ++a)
        acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[a], f.x[t], acc[a][t], 0, 0, 0);
  };
  // Sums in blocks of `block` stages: the running sums of a
  // block are added to `sum` and begun anew, since one chain over a long slice
  // rounds at the size of the whole sum at every step (8192 x 28672 at 8 rows:
  // relative error 7.5e-7 as one chain).  P.parts blocks and slices a row in
  // all, of 512 columns at least: with sqrt(n) blocks of the n steps, sums of 64
  // columns err half as much and cost 4-6 % of the time at 17 rows and more,
  // these 1 %.  One batch tile (two or three tiles a wavefront) adds every stage
  // to sums of 64 bits, so that the error does not grow with K at all: the GEMV,
  // which takes the smaller batches, sums over 64 lanes and errs no more (4096
  // columns: 9e-8; 6.5e-8 here).  That costs 1 %.
  constexpr bool kBlocks = C::kBlocks, kWide = BT == 1;
  using sum_t = typename std::conditional<kWide, f64x4_t, f32x4_t>::type;
  sum_t sum[kBlocks ? RW : 1][kBlocks ? BW : 1];
  if constexpr (kBlocks) {
#pragma unroll
    for (int a = 0; a < RW; ++a)
#pragma unroll
      for (int t = 0; t < BW; ++t) sum[a][t] = sum_t(0.f);
  }
  auto close_block = [&] {
    if constexpr (kBlocks) {
#pragma unroll
      for (int a = 0; a < RW; ++a)
#pragma unroll
        for (int t = 0; t < BW; ++t) {
          sum[a][t] += __builtin_convertvector(acc[a][t], sum_t);
          acc[a][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
  };
  const int block = kBlocks && !kWide ? max(8, (nst * P.S + P.parts - 1) / P.parts) : nst;

  // A stage is two 32-column steps; the fragments of a step are read while
  // the matrix cores work on the step before it (two register sets), and the
  // one barrier of a stage stands between its two steps: by then the stage's
  // second fragments are in registers, so its slot takes the next loads, and
  // the next stage has landed for every wavefront.
  const int first = min(depth, loads);
  for (int s = 0; s < first; ++s) issue();
  landed(first - 1);
  __syncthreads();
  Frags f0, f1;
  uint32_t ws = 0, xs = 0;
  int stage = rot;  // the stage being multiplied
  int used = 0;     // ring slots of this wavefront's operand used up
  if (computes) read(f0, ws, xs, 0, stage);
  // (blocks in a loop around the stages': a condition among them cost the small
  // units up to 14 %)
#pragma unroll 1
  for (int s0 = 0; s0 < nst; s0 += block) {
    const int s1 = min(nst, s0 + block);
#pragma unroll 1
    for (int s = s0; s < s1; ++s) {
      if (computes) {
        read(f1, ws, xs, 1, stage);
        __builtin_amdgcn_sched_barrier(0);
        mma(f0);
      }
      __builtin_amdgcn_sched_barrier(0);
      ++stage;
      // whether W's next stage is in its next slot, and this operand's
      const bool w_next = !HOST || stage % kSpan == 0 || stage == nst, next = w_next || !wl;
      stage = stage == nst ? 0 : stage;
      if (next) landed(min(depth, loads - used) - 2);
      __syncthreads();
      if (w_next) ws = ws + kWStage == kWRing ? 0 : ws + kWStage;
      xs = xs + C::kXStage == C::kXRing ? 0 : xs + C::kXStage;
      if (computes) read(f0, ws, xs, 0, stage);  // (after the last stage: not used)
      if (next && used + depth < loads) issue();
      used += next;
      __builtin_amdgcn_sched_barrier(0);
      if (computes) {
        if (kWide) close_block();  // (the products of f0 have had the barrier's wait)
        mma(f1);
      }
    }
    if (!kWide && computes) close_block();
  }
  if constexpr (kBlocks) {
#pragma unroll
    for (int a = 0; a < RW; ++a)
#pragma unroll
      for (int t = 0; t < BW; ++t)
        acc[a][t] = __builtin_convertvector(
            sum[a][t] + __builtin_convertvector(acc[a][t], sum_t), f32x4_t);
  }
  __syncthreads();  // LDS is reused by the next unit of a persistent worker

  if (!computes) return;
  // this wavefront's rows, all of one page; rows [p_lo, p_hi] lie whole on it,
  // the others are cut and go to the boundary's partial sums
  const int tg = G == 1 || HOST ? 0 : t_row / RTL;
  const int page = page0 + tg;
  const Rows wr = rows_of(tg);
  const int64_t rbase = wr.rbase + 16 * (t_row - tg * RTL), r_hi = wr.r_hi;
  if (G > 1 && wr.rbase > r_hi) return;  // (uniform over the wavefront)
  const int64_t p_lo = wr.r_lo + (wr.r_lo * K < wr.pe0), p_hi = r_hi - ((r_hi + 1) * K > wr.pe1);
  float* const outf = P.S == 1 ? (P.y_bf16 ? nullptr : static_cast<float*>(P.y))
                               : P.ws + static_cast<int64_t>(slice) * P.B * P.N;
  const bool vec = P.vec_out && rbase % 4 == 0;  // four rows in one 16-byte store
#pragma unroll
  for (int a = 0; a < RW; ++a) {
    const int64_t rt = rbase + 16 * a, r0 = rt + 4 * lgrp;
    const bool plain = rt >= p_lo && rt + 15 <= p_hi;  // uniform
#pragma unroll
    for (int t = 0; t < BW; ++t) {
      const int b = 16 * (t_bat + t) + lrow;
      if (b >= P.B) continue;
      if (plain && outf && vec) {
        *reinterpret_cast<f32x4_t*>(outf + static_cast<int64_t>(b) * P.N + r0) = acc[a][t];
        continue;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t r = r0 + e;
        if (r > r_hi) continue;
        const float v = acc[a][t][e];
        const int side = r < p_lo ? 1 : (r > p_hi ? 0 : -1);  // cut row: its part's side
        if (side < 0) {
          if (outf)
            outf[static_cast<int64_t>(b) * P.N + r] = v;
          else
            store_y(P, b, r, v);
        } else if (P.S == 1) {
          P.partial[(static_cast<int64_t>(page + 1 - side) * 2 + side) * kMaxGemvBatch + b] = v;
        } else {
          P.ws[static_cast<int64_t>(P.S) * P.B * P.N +
               ((static_cast<int64_t>(page + 1 - side) * 2 + side) * P.S + slice) * P.B + b] = v;
        }
      }
    }
  }
}

template <int BT, int RTL, int G, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_dma_kernel(GemvParams P) {
  using C = GemmCfg<BT, RTL, G, NW>;
  __shared__ __attribute__((aligned(16))) char smem[C::kWRing + C::kXRing];
  lds_char* const ring = (lds_char*)smem;
  const int bid = blockIdx.x;
  const int U = P.units_per_page;
  if (!P.address_order && bid < P.host_workers) {
    const int Uh = U * RTL;  // 16-row sub-units per host page
    const int n_host_sub = P.n_host_pages * Uh;
    for (int v = bid; v < n_host_sub; v += P.host_workers)
      gemm_dma_unit<BT, RTL, G, NW, true>(P, host_page(P, v / Uh), v % Uh, ring);
    return;
  }
  const int u = P.address_order ? bid : bid - P.host_workers;
  const int first = G > 1 ? (u / U) * G : (P.address_order ? u / U : hbm_page(P, u / U));
  gemm_dma_unit<BT, RTL, G, NW, false>(P, first, u % U, ring);
}

template <int BT, int RTL, int G>
int launch_gemm_shape(GemvParams& P, int n_pages, bool need_fixup, const boost_ctx* ctx,
                      hipStream_t s) {
  constexpr int NW = gemm_waves(BT, RTL, G);
  const int64_t groups = (n_pages + G - 1) / G;
  P.vec_out = P.N % 4 == 0 && (reinterpret_cast<uintptr_t>(P.S > 1 ? P.ws : P.y) & 15) == 0;
  P.w_once = P.K % 64 == 0;
  // sums a row: the kernels before cut K, into up to eight slices, where it was
  // longer than 16 K or where 64-row units were fewer than three quarters of the
  // compute units; twice as many here
  P.parts = n_pages < ctx->n_cu * 3 / 8 || P.K > 65536 ? 16 : 4;
  int64_t grid;
  if (P.address_order || P.n_host_pages == 0) {
    P.address_order = 1;
    P.host_workers = 0;
    grid = groups * P.units_per_page;
  } else {
    // host pages run as 16-row sub-units (RTL per unit)
    const int64_t host_sub = static_cast<int64_t>(P.n_host_pages) * P.units_per_page * RTL;
    P.host_workers = host_worker_count(ctx, host_sub, true);
    grid = P.host_workers + (G > 1 ? groups : P.n_hbm_pages) * P.units_per_page;
  }
  if (grid > 0x7fffffff) return fail(BOOST_EINVAL, "grid too large");
  hipLaunchKernelGGL((gemm_dma_kernel<BT, RTL, G, NW>), dim3(static_cast<unsigned>(grid)),
                     dim3(NW * 64), 0, s, P);
  BOOST_HIP(hipGetLastError());
  return launch_sums(P, n_pages, need_fixup, s);
}

}  // namespace

template <int BT>
int launch_gemm(GemvParams& P, const Route& route, int n_pages, bool need_fixup,
                const boost_ctx* ctx, hipStream_t s) {
  switch (route.shape) {
    case 0: return launch_gemm_shape<BT, 8, 1>(P, n_pages, need_fixup, ctx, s);
    case 1: return launch_gemm_shape<BT, 8, 2>(P, n_pages, need_fixup, ctx, s);
    case 2: return launch_gemm_shape<BT, 3, 4>(P, n_pages, need_fixup, ctx, s);
    case 3: return launch_gemm_shape<BT, 5, 1>(P, n_pages, need_fixup, ctx, s);
    case 4: return launch_gemm_shape<BT, 4, 1>(P, n_pages, need_fixup, ctx, s);
    default: return launch_gemm_shape<BT, 2, 1>(P, n_pages, need_fixup, ctx, s);
  }
}

}  // namespace gv
}  // namespace bst
