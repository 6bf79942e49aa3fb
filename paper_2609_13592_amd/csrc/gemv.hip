// a4: decode GEMV over tiered pages, y[b, n] = sum_k W[n, k] x[b, k].
//
// W is an [N, K] row-major bf16 matrix placed page by page on HBM or host
// (§3.1 modulo placement).  The work unit of a workgroup is a group of rows
// restricted to ONE page, so a workgroup reads one tier for its whole life
// (§3.2 CTA-level confinement: a workgroup never mixes tiers; the GEMM's units
// of several pages keep to it under CAP, not in address order).  A row that
// straddles a page boundary is split-K across the two workgroups of those
// pages; each stores its partial sum and a small second kernel adds them in a
// fixed order (part of the earlier page first), so results are bitwise
// reproducible and independent of the placement.
//
// Schedules (which workgroup takes which unit):
//   address order -- workgroup i takes unit i, blind to tiers (the
//     transparent kernel of §3.1; CAP then depends on where host pages fall);
//   CAP -- the first `host_workers` workgroups (dispatched first, spread over
//     the XCDs) stream all host-page units in a persistent loop while every
//     other workgroup takes one HBM-page unit, so the host link and HBM are
//     busy together in every wave (§3 CAP; §3.2 CTA specialisation).
//
// Inside a unit each wavefront owns RW rows and walks K with 16-byte loads:
// lane l reads columns [8l + 512i, 8l + 512i + 8) of every row, so one load
// instruction of a wavefront covers 1 KiB of one row contiguously.  The x
// chunk is loaded once per column step and reused for the RW rows.  Partial
// sums are reduced across the 64 lanes by a fixed xor butterfly.
#include <algorithm>

#include "gemv_common.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
using namespace bst::gv;

__device__ __forceinline__ float lo_bf16(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t v) {
  return __uint_as_float(v & 0xffff0000u);
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
// a.lo * b.lo + a.hi * b.hi + c for two packed bf16 pairs (products of bf16
// values are exact in fp32; the sum is accumulated in fp32)
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                         __builtin_bit_cast(bf16x2_t, b), c, false);
}

// 8-element dot product of two 16-byte bf16 vectors, accumulated into acc in
// element order
__device__ __forceinline__ float dot8(const uint4& w, const uint4& x, float acc) {
  acc = dot2(w.x, x.x, acc);
  acc = dot2(w.y, x.y, acc);
  acc = dot2(w.z, x.z, acc);
  acc = dot2(w.w, x.w, acc);
  return acc;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// A row cut by page boundary `bnd` (between pages bnd-1 and bnd) is summed by
// two workgroups, one per page; each stores its partial sum here (side 0 = the
// part on the earlier page) and split_fixup adds them after the main kernel.
template <int B>
__device__ __forceinline__ void store_split(const GemvParams& P, int bnd, int side,
                                            const float* v) {
  float* slot = P.partial + (static_cast<int64_t>(bnd) * 2 + side) * bst::kMaxGemvBatch;
#pragma unroll
  for (int b = 0; b < B; ++b) slot[b] = v[b];
}

// Accumulate this wavefront's columns [k_beg, k_end) of its RW rows from
// the page behind resource wr; row i's column 0 sits at byte offset ro[i]
// (offsets outside the page read as zero).
template <int B, int RW, int UN>
__device__ __forceinline__ void accumulate(__amdgpu_buffer_rsrc_t wr,
                                           __amdgpu_buffer_rsrc_t xr, const uint32_t* ro,
                                           int64_t K, int64_t k_beg, int64_t k_end, int lane,
                                           float (*acc)[B]) {
  constexpr int kStep = 64 * 8;  // columns covered by one load of a wavefront
  for (int64_t kb = k_beg; kb < k_end; kb += kStep * UN) {
    uint4 wv[UN][RW], xv[UN][B];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t kc = kb + u * kStep + lane * 8;
      const uint32_t oob = kc < k_end ? 0u : kOOB;
      const uint32_t kc2 = static_cast<uint32_t>(kc * 2);
#pragma unroll
      for (int b = 0; b < B; ++b)
        xv[u][b] = load16(xr, (static_cast<uint32_t>(b * K * 2) + kc2) | oob);
#pragma unroll
      for (int i = 0; i < RW; ++i) wv[u][i] = load16<BOOST_W_AUX>(wr, (ro[i] + kc2) | oob);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int b = 0; b < B; ++b) acc[i][b] = dot8(wv[u][i], xv[u][b], acc[i][b]);
  }
}

// One unit: a group of rows of page `page`, restricted to the page's bytes.
// The wavefronts of the workgroup form (kWaves / KS) row slots of RW rows;
// the KS wavefronts of a slot split K into KS contiguous column ranges
// (split-K inside the workgroup) and combine their partial sums through LDS
// in a fixed order.  The page's buffer resource covers exactly its valid
// bytes, so columns of a cut row that lie on the neighbouring page, and
// columns past K, read as zero without a branch.
//
// A row cut by a page boundary belongs to the earlier page's unit when both
// pages are in the same tier (it reads the next page too and adds the two
// parts itself); when the tiers differ each page's unit stores its part and
// split_fixup adds them, so no workgroup ever reads two tiers.
template <int B, int RW, int UN, int KS>
__device__ void gemv_unit(const GemvParams& P, int page, int j, float* lds) {
  constexpr int kSlots = kWaves / KS;
  constexpr int kRowsWg = kSlots * RW;
  const int64_t K = P.K;
  const int64_t total = static_cast<int64_t>(P.N) * K;
  const int64_t pe0 = static_cast<int64_t>(page) * kPageElems;
  const int64_t pe1 = min(pe0 + kPageElems, total);
  const int64_t r_lo = pe0 / K;
  const int64_t r_hi = (pe1 - 1) / K;  // inclusive
  const int64_t rbase = r_lo + static_cast<int64_t>(j) * kRowsWg;
  if (rbase > r_hi) return;  // uniform over the workgroup
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int slot = wave / KS, part = wave % KS;
  const int64_t r0 = rbase + slot * RW;
  // tiers are read only by the (few) units that hold a row cut by a page
  // boundary, so the common unit starts its loads without waiting on them
  const bool cut_first = rbase == r_lo && r_lo * K < pe0;
  const bool cut_last = rbase + kRowsWg > r_hi && (r_hi + 1) * K > pe1;
  bool prev_same = false, next_same = false;
  if (cut_first || cut_last) {
    const uint8_t tier = page_tier(P, page);
    prev_same = cut_first && page_tier(P, page - 1) == tier;
    next_same = cut_last && page + 1 < P.n_pages && page_tier(P, page + 1) == tier;
  }

  const __amdgpu_buffer_rsrc_t wr =
      make_rsrc(page_addr(P, page), static_cast<uint32_t>((pe1 - pe0) * 2));
  const __amdgpu_buffer_rsrc_t xr =
      make_rsrc(P.x, static_cast<uint32_t>(B * K * 2));
  // 0 = whole row here, 1 = tail of a row begun on the previous page,
  // 2 = head of a row ending on the next page, 3 = skipped
  int kind[RW];
  uint32_t ro[RW], ro2[RW];
  bool join = false;
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const int64_t r = r0 + i;
    const int64_t e0 = r * K;
    kind[i] = r > r_hi ? 3 : (e0 < pe0 ? (prev_same ? 3 : 1) : (e0 + K > pe1 ? 2 : 0));
    ro[i] = kind[i] == 3 ? kOOB : static_cast<uint32_t>((e0 - pe0) * 2);
    ro2[i] = kOOB;
    if (kind[i] == 2 && next_same) {
      ro2[i] = static_cast<uint32_t>((e0 - pe1) * 2);  // wraps: columns before pe1 read 0
      join = true;
    }
  }

  float acc[RW][B], acc2[RW][B];
#pragma unroll
  for (int i = 0; i < RW; ++i)
#pragma unroll
    for (int b = 0; b < B; ++b) acc[i][b] = acc2[i][b] = 0.f;

  constexpr int kStep = 64 * 8;
  // this wavefront's columns: [k_beg, k_end), k_beg a multiple of kStep
  const int64_t kper = (((K + KS - 1) / KS) + kStep - 1) / kStep * kStep;
  const int64_t k_beg = part * kper;
  const int64_t k_end = min(K, k_beg + kper);
  accumulate<B, RW, UN>(wr, xr, ro, K, k_beg, k_end, lane, acc);
  if (join) {  // uniform over the slot (same rows, same page): the next page's part
    const int64_t pe2 = min(pe1 + kPageElems, total);
    const __amdgpu_buffer_rsrc_t wr2 =
        make_rsrc(page_addr(P, page + 1), static_cast<uint32_t>((pe2 - pe1) * 2));
    accumulate<B, RW, UN>(wr2, xr, ro2, K, k_beg, k_end, lane, acc2);
  }

  float v[RW][B], v2[RW][B];
#pragma unroll
  for (int i = 0; i < RW; ++i)
#pragma unroll
    for (int b = 0; b < B; ++b) {
      v[i][b] = wave_sum(acc[i][b]);
      v2[i][b] = join ? wave_sum(acc2[i][b]) : 0.f;
    }

  if constexpr (KS > 1) {
    // partial sums of the KS column ranges meet in LDS; the slot's first
    // wavefront adds them in range order (each page part separately)
    float* l1 = lds;
    float* l2 = lds + kWaves * RW * B;
    if (lane == 0)
#pragma unroll
      for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int b = 0; b < B; ++b) {
          l1[(wave * RW + i) * B + b] = v[i][b];
          l2[(wave * RW + i) * B + b] = v2[i][b];
        }
    __syncthreads();
    if (part == 0 && lane == 0)
#pragma unroll
      for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int b = 0; b < B; ++b) {
          float s1 = l1[(wave * RW + i) * B + b], s2 = l2[(wave * RW + i) * B + b];
#pragma unroll
          for (int q = 1; q < KS; ++q) {
            s1 += l1[((wave + q) * RW + i) * B + b];
            s2 += l2[((wave + q) * RW + i) * B + b];
          }
          v[i][b] = s1;
          v2[i][b] = s2;
        }
    __syncthreads();  // LDS is reused by the next unit of a persistent worker
  }
  if (part != 0 || lane != 0) return;
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const int64_t r = r0 + i;
    if (kind[i] == 0) {
#pragma unroll
      for (int b = 0; b < B; ++b) store_y(P, b, r, v[i][b]);
    } else if (kind[i] == 1) {
      store_split<B>(P, page, 1, v[i]);  // tail of a row begun on a page of the other tier
    } else if (kind[i] == 2) {
      if (ro2[i] != kOOB) {
#pragma unroll
        for (int b = 0; b < B; ++b) store_y(P, b, r, v[i][b] + v2[i][b]);
      } else {
        store_split<B>(P, page + 1, 0, v[i]);  // head of a row ending on the other tier
      }
    }
  }
}

// Unit `idx` of a list of n pages (the HBM pages in page order, or with
// all_pages every page) with U units each.  Normally page idx / U, unit idx % U.  With tail_first the first n
// indices are the last non-empty unit of every page and the rest the other
// units in page order: the last unit of a page holds the row cut by the page
// boundary, which it sums over both pages when they are in one tier, so it
// reads twice as many steps as the others; dispatched first it overlaps
// them instead of running alone at the end of the launch.
template <int kRowsWg>
__device__ __forceinline__ void unit_of(const GemvParams& P, bool all_pages, int n, int U,
                                        int idx, int& page, int& j) {
  if (!P.tail_first) {
    page = all_pages ? idx / U : hbm_page(P, idx / U);
    j = idx % U;
    return;
  }
  const int i = idx < n ? idx : (idx - n) / (U - 1);
  page = all_pages ? i : hbm_page(P, i);
  const int64_t total = static_cast<int64_t>(P.N) * P.K;
  const int64_t pe0 = static_cast<int64_t>(page) * kPageElems;
  const int64_t pe1 = min(pe0 + kPageElems, total);
  const int last = static_cast<int>(((pe1 - 1) / P.K - pe0 / P.K) / kRowsWg);
  if (idx < n) {
    j = last;
  } else {
    const int k = (idx - n) % (U - 1);
    j = k < last ? k : k + 1;
  }
}

template <int B, int RW, int UN, int KS>
__global__ __launch_bounds__(kThreads) void gemv_kernel(GemvParams P) {
  __shared__ float lds[2 * kWaves * RW * B];
  constexpr int kRowsWg = (kWaves / KS) * RW;
  const int bid = blockIdx.x;
  const int U = P.units_per_page;
  int page, j;
  if (P.address_order) {
    unit_of<kRowsWg>(P, true, P.n_pages, U, bid, page, j);
    gemv_unit<B, RW, UN, KS>(P, page, j, lds);
  } else if (bid < P.host_workers) {
    const int n_host_units = P.n_host_pages * U;
    for (int v = bid; v < n_host_units; v += P.host_workers)
      gemv_unit<B, RW, UN, KS>(P, host_page(P, v / U), v % U, lds);
  } else {
    unit_of<kRowsWg>(P, false, P.n_hbm_pages, U, bid - P.host_workers, page, j);
    gemv_unit<B, RW, UN, KS>(P, page, j, lds);
  }
}

// y of every row cut by a page boundary: part on the earlier page plus part
// on the later page, in that order.  One lane per (boundary, batch row).
__global__ __launch_bounds__(256) void split_fixup(GemvParams P, int n_pages, int B) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int bnd = 1 + t / B, b = t % B;
  if (bnd >= n_pages) return;
  const int64_t e = static_cast<int64_t>(bnd) * kPageElems;
  if (e % P.K == 0) return;  // this boundary falls between rows
  if (P.join && page_tier(P, bnd - 1) == page_tier(P, bnd)) return;  // summed by one workgroup
  const float* s0 = P.partial + static_cast<int64_t>(bnd) * 2 * bst::kMaxGemvBatch;
  store_y(P, b, e / P.K, s0[b] + s0[bst::kMaxGemvBatch + b]);
}

// ---------------------------------------------------------------------------
// Up to 16 batch rows: RT 16-row tiles of a page and one K slice per workgroup,
// the slice split over its four wavefronts and their partial tiles summed in
// LDS in wavefront order, in 64 bits.  Which calls it takes, and why:
// gemm_plan.h.
//
// Units, schedules and cut rows as in the GEMV; with K split over S workgroups
// every part goes to the workspace.  Each wavefront streams its rows
// row-contiguously (one load instruction = 512 bytes of each of two rows),
// writes the 16 RT x 256 column chunk into a private LDS tile (16-byte chunks
// XOR-swizzled by row, so that neither the writes nor the fragment reads meet
// on a bank) and reads the A fragments of v_mfma_f32_16x16x32_bf16 back from
// there; x's B fragments come straight from memory, once for the RT tiles.
constexpr int kMfmaCols = 256;                          // columns per chunk
constexpr int kMfmaTileFloats = 16 * kMfmaCols * 2 / 4;  // one wavefront's tile
template <int RT>
constexpr int mfma_sum_floats() { return 16 * (16 * RT + 1); }  // [batch][row], padded

template <int RT>
__device__ void mfma_unit(const GemvParams& P, int page, int unit, float* lds) {
  const int j = unit / P.S, slice = unit % P.S;
  const int64_t K = P.K;
  const int64_t total = static_cast<int64_t>(P.N) * K;
  const int64_t pe0 = static_cast<int64_t>(page) * kPageElems;
  const int64_t pe1 = min(pe0 + kPageElems, total);
  const int64_t r_lo = pe0 / K;
  const int64_t r_hi = (pe1 - 1) / K;  // inclusive
  const int64_t rbase = r_lo + static_cast<int64_t>(j) * (16 * RT);
  if (rbase > r_hi) return;  // uniform over the workgroup
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int lrow = lane & 15, lgrp = lane >> 4;

  const __amdgpu_buffer_rsrc_t wr =
      make_rsrc(page_addr(P, page), static_cast<uint32_t>((pe1 - pe0) * 2));
  const __amdgpu_buffer_rsrc_t xr =
      make_rsrc(P.x, static_cast<uint32_t>(static_cast<int64_t>(P.B) * K * 2));
  const uint32_t xo = lrow < P.B ? static_cast<uint32_t>(lrow * K * 2) : kOOB;
  // sums of two steps, added up in 64 bits (as the GEMM's one batch tile)
  f64x4_t sum[RT];
#pragma unroll
  for (int a = 0; a < RT; ++a) sum[a] = f64x4_t(0.);

  constexpr int kStep = 32;
  // this unit's K slice, then this wavefront's quarter of it
  const int64_t ksl = (K + P.S - 1) / P.S;
  const int64_t kslice = (ksl + kWaves * kStep - 1) / (kWaves * kStep) * (kWaves * kStep);
  const int64_t s_beg = slice * kslice;
  const int64_t s_end = min(K, s_beg + kslice);
  const int64_t kper = kslice / kWaves;
  const int64_t k_beg = min(s_end, s_beg + wave * kper);
  const int64_t k_end = min(s_end, k_beg + kper);

  uint4* tile = reinterpret_cast<uint4*>(lds + kWaves * mfma_sum_floats<RT>() +
                                         wave * (RT * kMfmaTileFloats));
  // load instruction i: rows 2i and 2i+1 (lanes 0-31 / 32-63), 16 bytes each;
  // a row begun on the previous page gets a wrapped (huge) offset, so its
  // columns before the page read as zero
  constexpr int kLd = 8 * RT;
  uint32_t lo[kLd];
#pragma unroll
  for (int i = 0; i < kLd; ++i) {
    const int64_t r = rbase + 2 * i + (lane >> 5);
    lo[i] = r > r_hi ? kOOB : static_cast<uint32_t>((r * K - pe0) * 2);
  }
  const int wr_chunk = lane & 31;
  uint4 wv[kLd];
  auto load_chunk = [&](int64_t kb) {
    const int64_t kc = kb + 8 * wr_chunk;
    const uint32_t oob = kc < k_end ? 0u : kOOB;
    const uint32_t kc2 = static_cast<uint32_t>(kc * 2);
#pragma unroll
    for (int i = 0; i < kLd; ++i) wv[i] = load16(wr, (lo[i] + kc2) | oob);
  };
  if (k_beg < k_end) load_chunk(k_beg);
  constexpr int kChunkSteps = kMfmaCols / kStep;
#pragma unroll 1
  for (int64_t kb = k_beg; kb < k_end; kb += kMfmaCols) {
#pragma unroll
    for (int i = 0; i < kLd; ++i) {
      const int rr = 2 * i + (lane >> 5);
      tile[rr * 32 + (wr_chunk ^ (rr & 15))] = wv[i];
    }
    // this chunk's x fragments, then the next chunk's weights: the MFMAs
    // below wait only for the former (the wait counter is in order)
    uint4 xv[kChunkSteps];
#pragma unroll
    for (int st = 0; st < kChunkSteps; ++st) {
      const int64_t kc = kb + st * kStep + 8 * lgrp;
      const uint32_t oob = kc < k_end ? 0u : kOOB;
      xv[st] = load16(xr, (xo + static_cast<uint32_t>(kc * 2)) | oob);
    }
    load_chunk(kb + kMfmaCols);
    __builtin_amdgcn_sched_barrier(0);
    f32x4_t acc[RT][kChunkSteps / 2];
#pragma unroll
    for (int st = 0; st < kChunkSteps; ++st)
#pragma unroll
      for (int a = 0; a < RT; ++a) {
        const uint4 w = tile[(16 * a + lrow) * 32 + ((4 * st + lgrp) ^ lrow)];
        const f32x4_t c = st % 2 ? acc[a][st / 2] : f32x4_t{0.f, 0.f, 0.f, 0.f};
        acc[a][st / 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, xv[st]), c, 0, 0, 0);
      }
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
      for (int st = 0; st < kChunkSteps / 2; ++st)
        sum[a] += __builtin_convertvector(acc[a][st], f64x4_t);
  }

  // output element (row 16 a + 4 lgrp + e, batch row lrow); LDS holds the
  // [batch][row] tile of every wavefront, added up in wavefront order and
  // rounded once
  constexpr int R = 16 * RT, LS = R + 1;
#pragma unroll
  for (int a = 0; a < RT; ++a)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      lds[wave * mfma_sum_floats<RT>() + lrow * LS + 16 * a + 4 * lgrp + e] =
          static_cast<float>(sum[a][e]);
  __syncthreads();
#pragma unroll
  for (int idx = threadIdx.x; idx < 16 * R; idx += kThreads) {
    const int b = idx / R, i = idx % R;
    const int64_t r = rbase + i;
    if (b >= P.B || r > r_hi) continue;
    double all = 0.;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) all += lds[w * mfma_sum_floats<RT>() + b * LS + i];
    const float v = static_cast<float>(all);
    const int64_t e0 = r * K;
    const int side = e0 < pe0 ? 1 : (e0 + K > pe1 ? 0 : -1);  // cut row: its part's side
    const int64_t bnd = side == 1 ? page : page + 1;
    if (side < 0 && P.S == 1)
      store_y(P, b, r, v);
    else if (side < 0)
      P.ws[(static_cast<int64_t>(slice) * P.B + b) * P.N + r] = v;
    else if (P.S == 1)
      P.partial[(bnd * 2 + side) * bst::kMaxGemvBatch + b] = v;
    else
      P.ws[static_cast<int64_t>(P.S) * P.B * P.N + ((bnd * 2 + side) * P.S + slice) * P.B + b] = v;
  }
  __syncthreads();  // LDS is reused by the next unit of a persistent worker
}

template <int RT>
__global__ __launch_bounds__(kThreads) void mfma_kernel(GemvParams P) {
  __shared__ float lds[kWaves * (mfma_sum_floats<RT>() + RT * kMfmaTileFloats)];
  const int bid = blockIdx.x;
  const int U = P.units_per_page;
  if (P.address_order) {
    mfma_unit<RT>(P, bid / U, bid % U, lds);
  } else if (bid < P.host_workers) {
    const int n_host_units = P.n_host_pages * U;
    for (int v = bid; v < n_host_units; v += P.host_workers)
      mfma_unit<RT>(P, host_page(P, v / U), v % U, lds);
  } else {
    const int u = bid - P.host_workers;
    mfma_unit<RT>(P, hbm_page(P, u / U), u % U, lds);
  }
}

// y of a split-K call: the S slice partials of every (batch row, row) in
// slice order; a row cut by a page boundary adds its earlier page's slices,
// then its later page's.
//
// One lane per (b, V consecutive n): V = 4 where rows of y and of the slices
// are 16-byte aligned and four rows end on at most one other page (6144 x 4096
// at 256 rows, four slices: 6.1 us, and 7.1 with one n a lane for half the
// slices), else 1.  Every load goes out before the sums (a loop over a run-time
// S would wait for each in turn; a cut row found by division and loaded after
// the others cost 4096 x 14336 at 24 rows 29.2 us a call against 27.8).
template <int V>
__global__ __launch_bounds__(256) void split_reduce(GemvParams P) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int nv = P.N / V;
  if (t >= static_cast<int64_t>(P.B) * nv) return;
  const int b = static_cast<int>(t / nv);
  const int64_t r0 = (t - static_cast<int64_t>(b) * nv) * V;
  typedef __attribute__((ext_vector_type(V))) float vec_t;
  vec_t part[kMaxSlices];
#pragma unroll
  for (int s = 0; s < kMaxSlices; ++s)
    part[s] = s < P.S ? *reinterpret_cast<const vec_t*>(
                            P.ws + (static_cast<int64_t>(s) * P.B + b) * P.N + r0)
                      : vec_t(0.f);
  // the one page that begins inside these rows, if any: `in` elements after
  // their start, in the row `cut` unless it begins with a row
  const int64_t e0 = r0 * P.K, p = e0 / kPageElems + 1;
  const int64_t in = p * kPageElems - e0;
  int cut = -1;
  float part0[kMaxSlices], part1[kMaxSlices];
  if (in < static_cast<int64_t>(V) * P.K) {
    const int d = static_cast<int>(in);
    int i = 0;
#pragma unroll
    for (int k = 1; k < V; ++k) i += d >= k * P.K;
    if (d != i * P.K) {
      cut = i;
      const float* q = P.ws + static_cast<int64_t>(P.S) * P.B * P.N + p * 2 * P.S * P.B + b;
#pragma unroll
      for (int s = 0; s < kMaxSlices; ++s) {
        part0[s] = s < P.S ? q[static_cast<int64_t>(s) * P.B] : 0.f;
        part1[s] = s < P.S ? q[static_cast<int64_t>(P.S + s) * P.B] : 0.f;
      }
    }
  }
  vec_t v = vec_t(0.f);
#pragma unroll
  for (int s = 0; s < kMaxSlices; ++s)
    if (s < P.S) v += part[s];
  if (cut >= 0) {
    float v0 = 0.f, v1 = 0.f;
#pragma unroll
    for (int s = 0; s < kMaxSlices; ++s)
      if (s < P.S) {
        v0 += part0[s];
        v1 += part1[s];
      }
#pragma unroll
    for (int e = 0; e < V; ++e)
      if (e == cut) v[e] = v0 + v1;
  }
  if (V == 4 && !P.y_bf16) {
    *reinterpret_cast<vec_t*>(static_cast<float*>(P.y) + static_cast<int64_t>(b) * P.N + r0) = v;
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e) store_y(P, b, r0 + e, v[e]);
  }
}

#ifndef BOOST_GEMV_UN1
#define BOOST_GEMV_UN1 8
#endif
// Rows per wavefront and loads in flight per row, by batch size.
// Rows per wavefront (an x chunk is reused for every row) and load steps in
// flight, by batch size: more rows per wavefront as the batch grows keeps the
// x loads per weight load, and the registers, bounded.
// Batch 1 with a row split over four wavefronts (rows longer than 12K
// columns): each wavefront's x slice differs from its neighbours', so x misses
// the L1 cache (counters: as many L2 requests for x as for the weights) and
// would be fetched from L2 once per row; two rows per wavefront reuse one x
// slice from registers (8B down projection 22.2 -> 21.2 us, 70B 44.0 ->
// 42.1 us; with a row over two wavefronts it did not pay), with eight load
// steps in flight per row (four: 21.8 us, eight: 21.4, sixteen: 30.4 at
// half the occupancy).
#ifndef BOOST_GEMV_RW1_LONG
#define BOOST_GEMV_RW1_LONG 2
#endif
#ifndef BOOST_GEMV_UN1_LONG
#define BOOST_GEMV_UN1_LONG 8
#endif
#ifndef BOOST_GEMV_RW1
#define BOOST_GEMV_RW1 1
#endif
template <int B, int KS>
struct Shape {
  static constexpr int RW = B == 1 ? (KS > 2 ? BOOST_GEMV_RW1_LONG : BOOST_GEMV_RW1)
                                   : (B == 2 ? 2 : 4);
  static constexpr int UN = B == 1 ? (KS > 2 ? BOOST_GEMV_UN1_LONG : BOOST_GEMV_UN1)
                                   : 2;
};

// Wavefronts per row (split-K inside the workgroup) for a row of K columns:
// enough that each wavefront reads a few KiB of a row, so long rows do not
// serialise many round trips in one wavefront.
#ifndef BOOST_GEMV_KS_MAX
#define BOOST_GEMV_KS_MAX 4
#endif
#ifndef BOOST_GEMV_KS2_ABOVE
#define BOOST_GEMV_KS2_ABOVE 6144
#endif
#ifndef BOOST_GEMV_KS4_ABOVE
#define BOOST_GEMV_KS4_ABOVE 12288
#endif
inline int k_splits(int K) {
  const int ks = K <= BOOST_GEMV_KS2_ABOVE ? 1 : (K <= BOOST_GEMV_KS4_ABOVE ? 2 : 4);
  return ks < BOOST_GEMV_KS_MAX ? ks : BOOST_GEMV_KS_MAX;
}

}  // namespace

namespace bst {
namespace gv {

// Host workers for host_units units on host pages: n_cu / 16 by default.  The
// matrix-core kernels, whose workgroups keep fewer bytes in flight, take up to
// n_cu / 8, as many as give every worker the same number of units.  The GEMV's
// workgroups already keep the link busy; more of them slowed the HBM units
// beside them (2 GiB tensor, 8 host pages: 360 -> 432 us).  Never more workers
// than host units.
int host_worker_count(const boost_ctx* ctx, int64_t host_units, bool matrix_core) {
  int64_t h = std::max(1, ctx->n_cu / 16);
  if (matrix_core) {
    const int64_t most = std::max(1, ctx->n_cu / 8), rounds = (host_units + most - 1) / most;
    h = std::max(h, (host_units + rounds - 1) / std::max<int64_t>(1, rounds));
  }
  if (ctx->gemv_host_workers > 0) h = ctx->gemv_host_workers;
  return static_cast<int>(std::min(h, host_units));
}

int64_t rows_met(const GemvParams& P, int n_pages) {
  const int64_t K = P.K, total = static_cast<int64_t>(P.N) * K;
  if (kPageElems % K == 0) return std::min<int64_t>(P.N, kPageElems / K);
  int64_t most = 0;
  for (int p = 0; p < n_pages; ++p) {
    const int64_t pe0 = static_cast<int64_t>(p) * kPageElems;
    const int64_t pe1 = std::min(pe0 + kPageElems, total);
    most = std::max(most, (pe1 - 1) / K - pe0 / K + 1);
  }
  return most;
}

int launch_sums(GemvParams& P, int n_pages, bool need_fixup, hipStream_t s) {
  if (P.S > 1) {
    if (P.slices) return BOOST_OK;  // the consumer sums the slices
    const bool vec = P.N % 4 == 0 && P.K <= kPageElems / 4 &&
                     (P.y_bf16 || (reinterpret_cast<uintptr_t>(P.y) & 15) == 0);
    const int64_t lanes = static_cast<int64_t>(P.B) * (vec ? P.N / 4 : P.N);
    const dim3 grid(static_cast<unsigned>((lanes + 255) / 256));
    if (vec)
      hipLaunchKernelGGL(split_reduce<4>, grid, dim3(256), 0, s, P);
    else
      hipLaunchKernelGGL(split_reduce<1>, grid, dim3(256), 0, s, P);
    BOOST_HIP(hipGetLastError());
  } else if (need_fixup) {
    const int lanes = (n_pages - 1) * P.B;
    hipLaunchKernelGGL(split_fixup, dim3((lanes + 255) / 256), dim3(256), 0, s, P, n_pages, P.B);
    BOOST_HIP(hipGetLastError());
  }
  return BOOST_OK;
}

}  // namespace gv
}  // namespace bst

namespace {

// Grid of a kernel whose workgroups take one unit each (P.units_per_page set);
// fills in P.host_workers and P.address_order.  Returns -1 if it is too large.
int64_t plan_grid(GemvParams& P, int n_pages, const boost_ctx* ctx, bool matrix_core) {
  int64_t grid;
  if (P.address_order || P.n_host_pages == 0) {
    P.address_order = 1;
    P.host_workers = 0;
    grid = static_cast<int64_t>(n_pages) * P.units_per_page;
  } else {
    P.host_workers = host_worker_count(
        ctx, static_cast<int64_t>(P.n_host_pages) * P.units_per_page, matrix_core);
    grid = P.host_workers + static_cast<int64_t>(P.n_hbm_pages) * P.units_per_page;
  }
  return grid > 0x7fffffff ? -1 : grid;
}

#ifndef BOOST_GEMV_TAIL_FIRST
#define BOOST_GEMV_TAIL_FIRST 1
#endif
template <int B, int KS>
int launch(GemvParams& P, int n_pages, bool need_fixup, const boost_ctx* ctx, hipStream_t s) {
  constexpr int RW = Shape<B, KS>::RW, UN = Shape<B, KS>::UN;
  constexpr int kRowsWg = RW * (kWaves / KS);
  // units per page: enough for the page that meets the most rows
  P.units_per_page = static_cast<int>((rows_met(P, n_pages) + kRowsWg - 1) / kRowsWg);
  const int64_t grid = plan_grid(P, n_pages, ctx, false);
  if (grid < 0) return bst::fail(BOOST_EINVAL, "grid too large");
  // rows cut by page boundaries: their units go first (see unit_of)
  P.tail_first = kPageElems % P.K != 0 && P.units_per_page >= 2 ? BOOST_GEMV_TAIL_FIRST : 0;
  hipLaunchKernelGGL((gemv_kernel<B, RW, UN, KS>), dim3(static_cast<unsigned>(grid)),
                     dim3(kThreads), 0, s, P);
  BOOST_HIP(hipGetLastError());
  return launch_sums(P, n_pages, need_fixup, s);
}

template <int RT>
int launch_mfma(GemvParams& P, int n_pages, bool need_fixup, const boost_ctx* ctx,
                hipStream_t s) {
  const int S = P.S;
  P.units_per_page = static_cast<int>((rows_met(P, n_pages) + 16 * RT - 1) / (16 * RT));
  // host workers are counted over the units of whole rows
  int64_t grid = plan_grid(P, n_pages, ctx, true);
  if (grid < 0) return bst::fail(BOOST_EINVAL, "grid too large");
  P.units_per_page *= S;
  grid = P.host_workers +
         static_cast<int64_t>(P.address_order ? n_pages : P.n_hbm_pages) * P.units_per_page;
  if (grid > 0x7fffffff) return bst::fail(BOOST_EINVAL, "grid too large");
  hipLaunchKernelGGL((mfma_kernel<RT>), dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, s, P);
  BOOST_HIP(hipGetLastError());
  return launch_sums(P, n_pages, need_fixup, s);
}

template <int B>
int launch_b(GemvParams& P, int n_pages, bool need_fixup, const boost_ctx* ctx,
             hipStream_t s) {
  switch (k_splits(P.K)) {
    case 1: return launch<B, 1>(P, n_pages, need_fixup, ctx, s);
    case 2: return launch<B, 2>(P, n_pages, need_fixup, ctx, s);
    default: return launch<B, 4>(P, n_pages, need_fixup, ctx, s);
  }
}

}  // namespace

using namespace bst;

namespace {

int dispatch(GemvParams& P, const boost_tensor* W, int K, int B, const boost_ctx* ctx,
             hipStream_t s);

int check_sizes(int N, int K, int B) {
  if (N < 1 || K < 8 || K % 8) return fail(BOOST_EINVAL, "N=%d K=%d (K %% 8 == 0)", N, K);
  if (static_cast<uint64_t>(K) * 2 > kPage)
    return fail(BOOST_EINVAL, "row of %d elements exceeds a page", K);
  if (B < 1 || B > kMaxGemvBatch)
    return fail(BOOST_EINVAL, "B=%d outside [1, %d]", B, kMaxGemvBatch);
  return BOOST_OK;
}

// The decode GEMV behind both entry points: y, or with `slices` the split-K
// partial sums in fp32 in the layout of ws (S reported through n_slices).
int decode_gemv(boost_ctx* ctx, const boost_tensor* W, int N, int K, const void* x, int B,
                void* y, int y_dtype, float* slices, int64_t slice_floats, int* n_slices,
                void* stream) {
  if (!ctx || !W || !x || !y) return fail(BOOST_EINVAL, "null argument");
  if (ctx->device < 0) return fail(BOOST_ENODEV, "plan-only context");
  if (int rc = check_sizes(N, K, B)) return rc;
  if (y_dtype != BOOST_DTYPE_F32 && y_dtype != BOOST_DTYPE_BF16)
    return fail(BOOST_EINVAL, "y_dtype %d", y_dtype);
  if (static_cast<uint64_t>(N) * K * 2 != W->bytes)
    return fail(BOOST_EINVAL, "N*K*2=%llu but tensor holds %llu bytes",
                (unsigned long long)(static_cast<uint64_t>(N) * K * 2),
                (unsigned long long)W->bytes);
  if ((reinterpret_cast<uintptr_t>(x) & 15) || (reinterpret_cast<uintptr_t>(y) & 3))
    return fail(BOOST_EINVAL, "x must be 16-byte and y 4-byte aligned");
  GemvParams P{};
  P.page_table = W->d_page_table;
  P.hbm_pages = W->d_hbm_pages;
  P.host_pages = W->d_host_pages;
  P.hbm_base = W->hbm.base;
  P.host_base = W->host.base;
  P.lay_M = W->lay_M;
  P.lay_SP = W->lay_SP;
  P.n_hbm_pages = static_cast<int>(W->hbm_pages.size());
  P.n_host_pages = static_cast<int>(W->host_pages.size());
  P.address_order = ctx->gemv_schedule == BOOST_SCHED_ADDRESS;
  P.N = N;
  P.K = K;
  P.x = static_cast<const uint16_t*>(x);
  P.y = y;
  P.y_bf16 = y_dtype == BOOST_DTYPE_BF16;
  P.partial = W->d_partial;
  P.slices = slices;
  P.slice_floats = slice_floats;
  P.B = B;
  const int r = dispatch(P, W, K, B, ctx, static_cast<hipStream_t>(stream));
  if (r == BOOST_OK && n_slices) *n_slices = std::max(1, P.S);
  return r;
}

int dispatch(GemvParams& P, const boost_tensor* W, int K, int B, const boost_ctx* ctx,
             hipStream_t s) {
  const int n = static_cast<int>(W->n_pages);
  P.n_pages = n;
  P.tiers = W->d_tiers;
  const PlanInput in{P.N, K, B, n, rows_met(P, n), ctx->n_cu, ctx->gemm_ws_floats,
                     P.slices != nullptr, static_cast<uint64_t>(P.slice_floats)};
  const Route route = ctx->gemv_route.kernel ? forced_route(in, ctx->gemv_route) : plan(in);
  if (route.kernel == kAuto)
    return fail(BOOST_EINVAL, "N=%d K=%d B=%d does not fit the route that was set", P.N, K, B);
  if (route.kernel != kGemv) {
    // every row cut by a page boundary goes through split_fixup
    P.join = 0;
    bool fix = false;
    for (int b = 1; b < n && !fix; ++b) fix = (static_cast<int64_t>(b) * kPageElems) % K != 0;
    P.S = route.S;
    if (P.S > 1) P.ws = P.slices ? P.slices : ctx->gemm_ws;
    if (route.kernel == kRows16)
      return route.shape == 1 ? launch_mfma<1>(P, n, fix, ctx, s)
                              : launch_mfma<2>(P, n, fix, ctx, s);
    const int rows = 16 * kGemmShapes[route.shape].rtl;
    P.units_per_page = static_cast<int>((in.most + rows - 1) / rows) * P.S;
    switch (batch_tiles(B)) {
      case 1: return launch_gemm<1>(P, route, n, fix, ctx, s);
      case 2: return launch_gemm<2>(P, route, n, fix, ctx, s);
      case 4: return launch_gemm<4>(P, route, n, fix, ctx, s);
      case 8: return launch_gemm<8>(P, route, n, fix, ctx, s);
      default: return launch_gemm<16>(P, route, n, fix, ctx, s);
    }
  }
  // split_fixup is needed only where a cut row crosses a tier boundary
  P.join = 1;
  bool fix = false;
  if (kPageElems % K != 0)
    for (int b = 1; b < n && !fix; ++b)
      fix = (static_cast<int64_t>(b) * kPageElems) % K != 0 && W->tiers[b - 1] != W->tiers[b];
  switch (B) {
    case 1: return launch_b<1>(P, n, fix, ctx, s);
    case 2: return launch_b<2>(P, n, fix, ctx, s);
    default: return launch_b<3>(P, n, fix, ctx, s);
  }
}

}  // namespace

extern "C" {

int boost_gemv_set_schedule(boost_ctx* ctx, int schedule, int host_workers) {
  if (!ctx) return fail(BOOST_EINVAL, "null ctx");
  if (schedule != BOOST_SCHED_ADDRESS && schedule != BOOST_SCHED_CAP)
    return fail(BOOST_EINVAL, "schedule %d", schedule);
  if (host_workers < 0) return fail(BOOST_EINVAL, "host_workers %d", host_workers);
  ctx->gemv_schedule = schedule;
  ctx->gemv_host_workers = host_workers;
  return BOOST_OK;
}

int boost_gemv_set_route(boost_ctx* ctx, int kernel, int row_tiles, int pages, int slices) {
  if (!ctx) return fail(BOOST_EINVAL, "null ctx");
  if (kernel < kAuto || kernel > kGemm) return fail(BOOST_EINVAL, "kernel %d", kernel);
  if (kernel >= kRows16 &&
      (slices < 1 || slices > kMaxSlices || (slices & (slices - 1))))
    return fail(BOOST_EINVAL, "slices %d", slices);
  bool known = kernel < kRows16 || (kernel == kRows16 && pages == 1 && row_tiles >= 1 &&
                                    row_tiles <= 2);
  for (const GemmShape& u : kGemmShapes)
    known = known || (kernel == kGemm && u.rtl == row_tiles && u.g == pages);
  if (!known) return fail(BOOST_EINVAL, "no unit of %d row tiles and %d pages", row_tiles, pages);
  ctx->gemv_route = Forced{kernel, row_tiles, pages, slices};
  return BOOST_OK;
}

int boost_gemv_route(const boost_ctx* ctx, int N, int K, int B, int max_slices, int* kernel,
                     int* row_tiles, int* pages, int* slices) {
  if (!ctx || !kernel || !row_tiles || !pages || !slices)
    return fail(BOOST_EINVAL, "null argument");
  if (int rc = check_sizes(N, K, B)) return rc;
  if (max_slices < 0 || max_slices > BOOST_MAX_GEMV_SLICES)
    return fail(BOOST_EINVAL, "max_slices %d outside [0, %d]", max_slices, BOOST_MAX_GEMV_SLICES);
  uint64_t floats = 0;
  if (max_slices > 0)
    if (int rc = boost_gemv_slices_floats(N, K, B, max_slices, &floats)) return rc;
  GemvParams P{};
  P.N = N;
  P.K = K;
  const int64_t pages_ = (static_cast<int64_t>(N) * K + kPageElems - 1) / kPageElems;
  if (pages_ > 0x7fffffff) return fail(BOOST_EINVAL, "N=%d K=%d", N, K);
  const int n = static_cast<int>(pages_);
  const PlanInput in{N, K, B, n, rows_met(P, n), ctx->device < 0 ? 256 : ctx->n_cu,
                     ctx->device < 0 ? kGemmWsFloats : ctx->gemm_ws_floats, max_slices > 0, floats};
  const Route r = plan(in);
  *kernel = r.kernel;
  *row_tiles = r.kernel == kGemm ? kGemmShapes[r.shape].rtl : (r.kernel == kRows16 ? r.shape : 0);
  *pages = r.kernel == kGemv ? 0 : (r.kernel == kGemm ? kGemmShapes[r.shape].g : 1);
  *slices = r.S;
  return BOOST_OK;
}

int boost_decode_gemv(boost_ctx* ctx, const boost_tensor* W, int N, int K, const void* x,
                      int B, void* y, int y_dtype, void* stream) {
  return decode_gemv(ctx, W, N, K, x, B, y, y_dtype, nullptr, 0, nullptr, stream);
}

int boost_gemv_slices_floats(int N, int K, int B, int max_slices, uint64_t* floats) {
  if (!floats) return fail(BOOST_EINVAL, "null argument");
  if (N < 1 || K < 1 || B < 1 || max_slices < 1)
    return fail(BOOST_EINVAL, "N=%d K=%d B=%d max_slices=%d", N, K, B, max_slices);
  const uint64_t pages = (static_cast<uint64_t>(N) * K + kPageElems - 1) / kPageElems;
  *floats = static_cast<uint64_t>(max_slices) * B * (N + 2 * (pages + 1));
  return BOOST_OK;
}

int boost_decode_gemv_slices(boost_ctx* ctx, const boost_tensor* W, int N, int K,
                             const void* x, int B, float* slices, int max_slices,
                             int* n_slices, void* stream) {
  if (!slices || !n_slices) return fail(BOOST_EINVAL, "null argument");
  if (max_slices < 1 || max_slices > BOOST_MAX_GEMV_SLICES)
    return fail(BOOST_EINVAL, "max_slices %d outside [1, %d]", max_slices, BOOST_MAX_GEMV_SLICES);
  if (reinterpret_cast<uintptr_t>(slices) & 15)
    return fail(BOOST_EINVAL, "slices must be 16-byte aligned");
  uint64_t cap = 0;
  if (int rc = boost_gemv_slices_floats(N, K, B, max_slices, &cap)) return rc;
  *n_slices = 0;
  return decode_gemv(ctx, W, N, K, x, B, slices, BOOST_DTYPE_F32, slices,
                     static_cast<int64_t>(cap), n_slices, stream);
}

}  // extern "C"
